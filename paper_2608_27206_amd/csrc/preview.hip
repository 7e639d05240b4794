// APC's shallow feature preview (Section 3.2, "Shallow Feature Preview": the vision encoder's
// initial block, K = 1, at the original resolution): patch embedding, RMSNorm, window
// attention with residual, RMSNorm and SwiGLU MLP with residual, with caller-supplied weights.
// Its token embeddings feed pace_apc_density_features.
//
// Kernels:
//   preview_patchify  patch pixels (x/127.5 - 1) in the caller's token order, bf16, rows
//                     zero-padded to a multiple of 8 values
//   gemm_bf16_nt      C = A B^T on bf16 MFMA (32x32x16), fp32 accumulation, with the block's
//                     epilogues fused: + bias, + residual, or SwiGLU of interleaved gate/up
//                     columns; bf16 out
//   rmsnorm_bf16      one wave per row
// The attention step is pace_vit_attention over the windows.
#include <math.h>

#include <type_traits>

#include "pace_internal.h"

namespace pace {
namespace {

typedef __bf16 gbf16x8 __attribute__((ext_vector_type(8)));
typedef float gf32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest even (finite values)
  return static_cast<uint16_t>(u >> 16);
}

__device__ __forceinline__ uint32_t pack2(float a, float b) {   // two bf16, nearest even
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
// expf and the division to a rounding each: on the exponential and reciprocal units alone the
// error is 2^-18 at gates below -20 (the rounded product with log2 e), for 716 against 782 us of 42,196 x
// 6,848 x 1,280.
__device__ __forceinline__ float silu(float x) { return x / (1.0f + expf(-x)); }

// ---------------------------------------------------------------- patchify
// One thread per 16-byte chunk of X: eight neighbouring bytes of a patch row in one load, byte by
// byte where the chunk goes on in the next row (5 of 42 chunks at patch 14) or past the patch.
// Bound: HBM (25 MB read, 50 MB written at 4K: 80 us with one value per thread,
// 42 us).
__global__ __launch_bounds__(256) void preview_patchify(const uint8_t* __restrict__ img, int W, int P, int gw,
                                                        const int32_t* __restrict__ order, int N, int Kp,
                                                        uint16_t* __restrict__ X) {
  const long long idx = static_cast<long long>(blockIdx.x) * 256 + threadIdx.x;
  const int nch = Kp / 8, pb = 3 * P, kin = pb * P;
  if (idx >= static_cast<long long>(N) * nch) return;
  const int t = static_cast<int>(idx / nch), e0 = static_cast<int>(idx - static_cast<long long>(t) * nch) * 8;
  const int patch = order[t];
  const int py = patch / gw, px = patch - py * gw;
  const uint8_t* base = img + (static_cast<long long>(py) * P * W + px * P) * 3;
  const int r = e0 / pb, cb = e0 - r * pb;
  float v[8];
  if (cb + 8 <= pb && e0 < kin) {
    uint64_t b;
    __builtin_memcpy(&b, base + static_cast<long long>(r) * W * 3 + cb, 8);
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = static_cast<float>(static_cast<uint32_t>(b >> (8 * q)) & 255u) * (1.0f / 127.5f) - 1.0f;
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int e = e0 + q, rr = e / pb;
      v[q] = e < kin ? static_cast<float>(base[static_cast<long long>(rr) * W * 3 + (e - rr * pb)]) * (1.0f / 127.5f) - 1.0f : 0.f;
    }
  }
  reinterpret_cast<uint4*>(X)[idx] = make_uint4(pack2(v[0], v[1]), pack2(v[2], v[3]), pack2(v[4], v[5]), pack2(v[6], v[7]));
}

// ---------------------------------------------------------------- GEMM
// C[M, N] = A[M, K] B[N, K]^T.  WM x WN waves, each with MI x NI MFMA tiles of 32 x 32.  K goes in
// stages of 64 through a ring of ST LDS buffers filled by DMA (buffer to LDS, no registers), so that
// every row of a stage is one 128-byte line (in stages of 32 the loads were 64-byte requests, twice
// as many, and took 65% of the L2s' request slots).  A stage is four steps of K = 16; the
// fragments of each are read among the MFMAs of the one before, also across stages: a wave that
// holds a stage's last fragments meets the others, the stage's buffer takes the next request,
// and the last MFMAs run under the first reads of the following stage.  Rows past M or N and
// chunks past K load as zeros (range check, out-of-range offsets), so tails need no branches.
//   A stage row holds eight 16-byte chunks; chunk c of row r sits in slot c ^ ((r >> 1) & 7), so
// that the rows that a fragment read touches spread over all LDS banks.  The DMA writes lanes in
// order, so the swizzle is in the global addresses.
//   The product is formed as C^T (B's rows are the MFMA's A operand): a lane then holds four
// neighbouring columns of one row, which makes SwiGLU's gate and up neighbours in one lane; the
// tile leaves through LDS so that rows are stored in 16-byte chunks, and a residual tile comes
// the same way (read straight into the lanes it cost 20 us of a 64-us round of tiles).  Rows of other
// alignments go in units of 8, 4 or 2 bytes, neighbouring lanes taking neighbouring units (a lane's
// eight values one by one, and the residual by lane: 6,000 x 1,290 x 1,280 with residual 76.5 -> 56.3 us,
// 20,000 x 2,564 x 640 151.6 -> 98.1).
//   Bound: MFMA.  At 8,192^3 the matrix cores are busy 68% of the cycles and the clock falls to
// 1.6 GHz; at K = 1,280 47%, since a tile's first loads and the burst of stores (and residual
// loads) at the end of a round take a third of its time.  Measured against the 128 x 128
// register-staged kernel before it, 42,196 rows: N = K = 1,280 with residual 337 -> 197 us; N =
// 6,848, K = 1,280 with SwiGLU 1,211 -> 782 us (946 TFLOP/s); N = 1,280, K = 3,424 with residual
// 661 -> 401 us; 8,192^3 1,590 -> 868 us (1,267 TFLOP/s).  Stages of 32 in a ring of four: 205, 744, 446
// and 920 us.  Tried with stages of 32, TFLOP/s at 8,192^3 against 1,169: 4 x 4 MFMA tiles per wave
// with four waves 1,080 (one wave per SIMD does not hide its own LDS reads), two 128 x 256
// workgroups per CU with a ring of three 1,022, no fragments ahead of the barrier 1,144.
constexpr int kGK = 64;                      // K per stage: a row is one 128-byte line

enum { kEpiBias = 0, kEpiResidual = 1, kEpiSwiglu = 2 };

struct GemmParams {
  const uint16_t* A;
  const uint16_t* B[3];     // up to three products of the same A and shape (grid z)
  const float* bias[3];     // [N] or null
  const uint16_t* R;        // residual [M, N] (kEpiResidual)
  uint16_t* C[3];           // [M, N], or [M, N / 2] for kEpiSwiglu
  int M, N, K;
  int tiles_m, tiles_n;
  int mode;
  int width;                // elements per access to C and R: 8, 4, 2 or 1 as their alignment allows
  int res_dma;              // the residual tiles come by DMA (16-byte rows)
};

typedef __attribute__((address_space(3))) const char g_lds_char;
typedef int gi32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kGOut = 0x7FFFFFF0u;

__device__ __forceinline__ gi32x4 g_rsrc(const void* base, unsigned bytes) {
  const unsigned long long a = reinterpret_cast<unsigned long long>(base);
  gi32x4 r;
  r.x = __builtin_amdgcn_readfirstlane(static_cast<int>(a & 0xffffffffull));
  r.y = __builtin_amdgcn_readfirstlane(static_cast<int>((a >> 32) & 0xffffull));   // stride 0
  r.z = __builtin_amdgcn_readfirstlane(static_cast<int>(bytes));
  r.w = 0x00020000;
  return r;
}
// 64 lanes x 16 bytes from the buffer to lds .. lds + 1023; untracked by the compiler, awaited
// with g_wait.
__device__ __forceinline__ void g_dma16(gi32x4 r, unsigned lds, unsigned voff) {
  const unsigned m0 = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :: "v"(voff), "s"(r), "{m0}"(m0) : "memory");
}
template <int N>
__device__ __forceinline__ void g_wait() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
// the same, and the wave's LDS reads have returned
template <int N>
__device__ __forceinline__ void g_wait_lds() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N) : "memory"); }

// Workgroup barrier alone: the waits before it say what it orders.
__device__ __forceinline__ void g_barrier() { asm volatile("s_barrier" ::: "memory"); }

// What an access to W neighbouring elements moves.
template <int W> struct GemmUnit;
template <> struct GemmUnit<8> { typedef uint4 type; };
template <> struct GemmUnit<4> { typedef uint2 type; };
template <> struct GemmUnit<2> { typedef uint32_t type; };
template <> struct GemmUnit<1> { typedef uint16_t type; };
// f with W = 8, 4, 2 or 1 as a constant
template <typename F>
__device__ __forceinline__ void with_width(int width, F f) {
  if (width == 8) f(std::integral_constant<int, 8>{});
  else if (width == 4) f(std::integral_constant<int, 4>{});
  else if (width == 2) f(std::integral_constant<int, 2>{});
  else f(std::integral_constant<int, 1>{});
}

template <int MI, int NI, int WM, int WN, int ST>
__global__ __launch_bounds__(64 * WM * WN, 2) void gemm_bf16_nt(const GemmParams p) {
  constexpr int BM = 32 * MI * WM, BN = 32 * NI * WN;
  constexpr int NW = WM * WN, kGThreads = 64 * NW;
  constexpr int kStage = (BM + BN) * kGK;            // elements per stage
  constexpr int kInst = (BM + BN) / 8;               // wave-wide DMAs per stage, 8 rows each
  constexpr int kPW = kInst / NW;              // per wave
  static_assert(kInst % NW == 0, "every wave issues the same DMAs");
  constexpr int kLds = ST * kStage > BM * BN ? ST * kStage : BM * BN;
  __shared__ __align__(16) uint16_t lds[kLds];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, c32 = lane & 31;
  const int wm = (w / WN) * 32 * MI, wn = (w % WN) * 32 * NI;
  // XCD-contiguous order; groups of eight row tiles column by column, so that the workgroups
  // that run together on an XCD share a few rows of A and a few of B in its L2
  const int per = p.tiles_m * p.tiles_n;
  const int lb = remap_block_id(blockIdx.x, gridDim.x);
  const int z = lb / per;
  const int tl = lb - z * per;
  const int gsz = 8 * p.tiles_n, grp = tl / gsz, in = tl - grp * gsz;
  const int gm = min(8, p.tiles_m - 8 * grp);
  const int tn = in / gm, tm = 8 * grp + (in - tn * gm);
  const int bm = tm * BM, bn = tn * BN;
  const gi32x4 ra = g_rsrc(p.A, static_cast<unsigned>(static_cast<long long>(p.M) * p.K * 2));
  const gi32x4 rb = g_rsrc(p.B[z], static_cast<unsigned>(static_cast<long long>(p.N) * p.K * 2));

  // this lane's chunk of DMA i (wave w issues i = w, w + NW, ...; the first BM / 8 are A's rows)
  unsigned off[kPW];
  // row of the DMA's eight, first k of the chunk (NW is even: i's parity is w's)
  static_assert(NW % 2 == 0 && (BM / 8) % 2 == 0, "swizzle of odd DMAs");
  const int r8 = lane >> 3, kc = ((lane & 7) ^ (4 * (w & 1) + (r8 >> 1))) * 8;
#pragma unroll
  for (int u = 0; u < kPW; ++u) {
    const int i = w + NW * u;
    const bool isa = i < BM / 8;
    const int row = isa ? bm + i * 8 + r8 : bn + (i - BM / 8) * 8 + r8;
    // rows past the end lie past the buffer's range
    off[u] = row < (isa ? p.M : p.N) ? static_cast<unsigned>((static_cast<long long>(row) * p.K + kc) * 2) : kGOut;
  }
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<unsigned long long>((g_lds_char*)(const void*)lds));
  auto load = [&](int t, int buf) __attribute__((always_inline)) {
    const bool in_k = t * kGK + kc < p.K;
    const unsigned base = lds0 + buf * (kStage * 2);
#pragma unroll
    for (int u = 0; u < kPW; ++u) {
      const int i = w + NW * u;
      const unsigned o = in_k ? off[u] + static_cast<unsigned>(t) * (kGK * 2) : kGOut;
      g_dma16(i < BM / 8 ? ra : rb, base + i * 1024, o);
    }
  };
  // fragment reads: row r of the stage at byte 128 r, chunk c in slot c ^ ((r >> 1) & 7)
  const int sw = (c32 >> 1) & 7;
  auto frags = [&](int buf, int kk, gbf16x8* a, gbf16x8* b) __attribute__((always_inline)) {
    const uint16_t* st = lds + buf * kStage + c32 * kGK + (((2 * kk + g) ^ sw) * 8);
#pragma unroll
    for (int j = 0; j < NI; ++j) b[j] = *reinterpret_cast<const gbf16x8*>(st + (BM + wn + 32 * j) * kGK);
#pragma unroll
    for (int i = 0; i < MI; ++i) a[i] = *reinterpret_cast<const gbf16x8*>(st + (wm + 32 * i) * kGK);
  };
  gf32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = gf32x16{};
  auto mul = [&](const gbf16x8* a, const gbf16x8* b) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
  };
  // request: fragment reads spread among the MFMAs before the ones that use them
  auto spread = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < MI * NI; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (i < MI + NI) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
  };

  const int nk = (p.K + kGK - 1) / kGK;
#pragma unroll
  for (int s = 0; s < ST; ++s)
    if (s < nk) load(s, s);
  if (nk >= ST) g_wait<(ST - 1) * kPW>(); else g_wait<0>();
  g_barrier();
  gbf16x8 a0[MI], b0[NI], a1[MI], b1[NI];
  frags(0, 0, a0, b0);
  int cur = 0;   // buffer of stage t
  // Stage t: its first fragments are in a0 / b0.  Once a wave holds the last ones in registers it
  // meets the others; then stage t + 1 is in LDS, the buffer of stage t takes stage t + ST, and
  // the last MFMAs run under the first reads of stage t + 1.
  for (int t = 0; t + 1 < nk; ++t) {
    const int nxt = cur == ST - 1 ? 0 : cur + 1;
    frags(cur, 1, a1, b1);
    mul(a0, b0);
    spread();
    __builtin_amdgcn_sched_barrier(0);
    frags(cur, 2, a0, b0);
    mul(a1, b1);
    spread();
    __builtin_amdgcn_sched_barrier(0);
    frags(cur, 3, a1, b1);
    mul(a0, b0);
    spread();
    __builtin_amdgcn_sched_barrier(0);
    if (t + ST <= nk) g_wait_lds<(ST - 2) * kPW>(); else g_wait_lds<0>();
    g_barrier();
    if (t + ST < nk) load(t + ST, cur);
    frags(nxt, 0, a0, b0);
    mul(a1, b1);
    spread();
    __builtin_amdgcn_sched_barrier(0);
    cur = nxt;
  }
  // the last stage: only the chunks of 16 that K has
  const int last = (p.K - (nk - 1) * kGK + 15) / 16;
  if (last > 1) frags(cur, 1, a1, b1);
  mul(a0, b0);
  if (last > 1) {
    if (last > 2) frags(cur, 2, a0, b0);
    mul(a1, b1);
  }
  if (last > 2) {
    if (last > 3) frags(cur, 3, a1, b1);
    mul(a0, b0);
  }
  if (last > 3) mul(a1, b1);

  // epilogue: register 4 jj + ii of tile (i, j) is row wm + 32 i + c32, column
  // wn + 32 j + 8 jj + 4 g + ii.  The bf16 tile goes through LDS, once every wave has read its
  // last stage: 16-byte chunk ch of row r in slot ch ^ (r mod the chunks of a row), so that the
  // 32 rows of a write spread over all banks.  A residual tile comes in the same way first.
  __syncthreads();
  const int mode = p.mode;
  const bool glu = mode == kEpiSwiglu;
  constexpr int kCh = BN / 8;
  if (mode == kEpiResidual && p.res_dma) {
    constexpr int kRows = 512 / BN;   // tile rows per wave-wide DMA
    const gi32x4 rr = g_rsrc(p.R + static_cast<long long>(bm) * p.N, static_cast<unsigned>(min(BM, p.M - bm)) * p.N * 2u);
#pragma unroll
    for (int u = 0; u < BM / kRows / NW; ++u) {
      const int i = w + NW * u, r = i * kRows + lane / kCh;
      const int n = bn + (((lane % kCh) ^ (r & (kCh - 1))) * 8);
      g_dma16(rr, lds0 + i * 1024, n < p.N ? static_cast<unsigned>(r * p.N + n) * 2u : kGOut);
    }
    g_wait<0>();
    __syncthreads();
  } else if (mode == kEpiResidual) {
    with_width(p.width, [&](auto WC) __attribute__((always_inline)) {
      constexpr int W = decltype(WC)::value, kUnits = BN / W;
      typedef typename GemmUnit<W>::type T;
#pragma unroll 8
      for (int c = tid; c < BM * kUnits; c += kGThreads) {
        const int r = c / kUnits, cl = c % kUnits * W;
        T v{};
        if (bm + r < p.M && bn + cl < p.N)
          v = *reinterpret_cast<const T*>(p.R + static_cast<long long>(bm + r) * p.N + bn + cl);
        *reinterpret_cast<T*>(&lds[r * BN + (((cl >> 3) ^ (r & (kCh - 1))) << 3) + (cl & 7)]) = v;
      }
    });
    __syncthreads();
  }
  const auto rbias = range_rsrc(p.bias[z], p.bias[z] != nullptr ? static_cast<unsigned>(p.N) * 4u : 0u);
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4 bv[NI][4];
#pragma unroll
  for (int j = 0; j < NI; ++j)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj)
      bv[j][jj] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
          rbias, static_cast<unsigned>(bn + wn + 32 * j + 8 * jj + 4 * g) * 4u, 0, 0));
#pragma unroll
  for (int j = 0; j < NI; ++j)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int cl = wn + 32 * j + 8 * jj + 4 * g;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int rl = wm + 32 * i + c32;
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = acc[i][j][4 * jj + q] + bv[j][jj][q];
        if (glu) {
          const int cg = cl >> 1;
          *reinterpret_cast<uint32_t*>(&lds[rl * (BN / 2) + (((cg >> 3) ^ (rl & (kCh / 2 - 1))) << 3) + (cg & 7)]) =
              pack2(silu(v[0]) * v[1], silu(v[2]) * v[3]);
        } else {
          uint2* at = reinterpret_cast<uint2*>(&lds[rl * BN + (((cl >> 3) ^ (rl & (kCh - 1))) << 3) + (cl & 7)]);
          if (mode == kEpiResidual) {
            const uint2 u = *at;
            v[0] += __uint_as_float(u.x << 16); v[1] += __uint_as_float(u.x & 0xffff0000u);
            v[2] += __uint_as_float(u.y << 16); v[3] += __uint_as_float(u.y & 0xffff0000u);
          }
          *at = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        }
      }
    }
  __syncthreads();
  const int nc = glu ? p.N / 2 : p.N, n0 = glu ? bn / 2 : bn;   // columns of C, the tile's first
  const int cpr = glu ? kCh / 2 : kCh, cbits = __builtin_ctz(cpr);
  uint16_t* C = p.C[z];
  with_width(p.width, [&](auto WC) __attribute__((always_inline)) {
    constexpr int W = decltype(WC)::value, kLog = W == 8 ? 0 : W == 4 ? 1 : W == 2 ? 2 : 3;   // log2 of 8 / W
    typedef typename GemmUnit<W>::type T;
    const int ubits = cbits + kLog;
    for (int c = tid; c < BM << ubits; c += kGThreads) {
      const int r = c >> ubits, u = c & ((1 << ubits) - 1), ch = u >> kLog;
      const int m = bm + r, n = n0 + u * W;
      if (m >= p.M || n >= nc) continue;
      *reinterpret_cast<T*>(C + static_cast<long long>(m) * nc + n) =
          *reinterpret_cast<const T*>(&lds[(r * cpr + (ch ^ (r & (cpr - 1)))) * 8 + (u & (8 / W - 1)) * W]);
    }
  });
}

// ---------------------------------------------------------------- RMSNorm
struct NormAdd { __device__ float operator()(float a, float b) const { return a + b; } };

// y = x / sqrt(mean(x^2) + eps) * gamma, one wave per row, rows of D values (D % 8 == 0).
__global__ __launch_bounds__(256) void rmsnorm_bf16(const uint16_t* __restrict__ x, const float* __restrict__ gamma,
                                                    uint16_t* __restrict__ y, int M, int D, float eps) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  const uint4* xr = reinterpret_cast<const uint4*>(x + static_cast<long long>(row) * D);
  uint4* yr = reinterpret_cast<uint4*>(y + static_cast<long long>(row) * D);
  const int nch = D / 8;
  float ss = 0.f;
  for (int c = lane; c < nch; c += 64) {
    const uint4 v = xr[c];
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float a = __uint_as_float(u[q] << 16), b = __uint_as_float(u[q] & 0xFFFF0000u);
      ss += a * a + b * b;
    }
  }
  ss = wave_reduce_dpp(ss, NormAdd{});
  const float inv = 1.0f / sqrtf(ss / static_cast<float>(D) + eps);
  for (int c = lane; c < nch; c += 64) {
    const uint4 v = xr[c];
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
    uint32_t o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = c * 8 + 2 * q;
      const float a = __uint_as_float(u[q] << 16) * inv * gamma[e];
      const float b = __uint_as_float(u[q] & 0xFFFF0000u) * inv * gamma[e + 1];
      o[q] = static_cast<uint32_t>(to_bf16(a)) | (static_cast<uint32_t>(to_bf16(b)) << 16);
    }
    yr[c] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// What every product needs; nothing is launched otherwise.
pace_status_t check_gemm(const GemmParams& p, int nz) {
  PACE_REQUIRE(p.M >= 1 && p.N >= 1 && p.K >= 8 && p.K % 8 == 0,
               "pace_gemm_bf16: M=%d N=%d K=%d (K a positive multiple of 8)", p.M, p.N, p.K);
  PACE_REQUIRE(aligned16(p.A), "pace_gemm_bf16: A and B must be 16-byte aligned");
  for (int z = 0; z < nz; ++z) PACE_REQUIRE(aligned16(p.B[z]), "pace_gemm_bf16: A and B must be 16-byte aligned");
  PACE_REQUIRE(static_cast<long long>(p.M) * p.K * 2 < (1ll << 30) && static_cast<long long>(p.N) * p.K * 2 < (1ll << 30),
               "pace_gemm_bf16: an operand spans 1 GiB or more");
  return PACE_OK;
}

template <int MI, int NI, int WM, int WN, int ST>
void launch_tile(GemmParams p, int nz, hipStream_t stream) {
  p.tiles_m = (p.M + 32 * MI * WM - 1) / (32 * MI * WM);
  p.tiles_n = (p.N + 32 * NI * WN - 1) / (32 * NI * WN);
  const dim3 grid(static_cast<unsigned>(p.tiles_m) * p.tiles_n * nz);
  hipLaunchKernelGGL((gemm_bf16_nt<MI, NI, WM, WN, ST>), grid, dim3(64 * WM * WN), 0, stream, p);
}

// Tiles of 256 x 256 (one workgroup per CU) use the matrix cores best, but come in rounds of 256;
// tiles of 64 x 128 fill the chip from small products on.  With stages of 64, 42,196 x 1,280 x 1,280 takes 168 us
// in large tiles (four rounds of 42) and 215 in small ones (825 large tiles' area): a round costs as much
// as about 156 large tiles in small ones.  A launch of small tiles costs at least 0.3 of a round (11.6
// us at 1,024 rows).  The rows go to whichever of these is the shortest: large tiles alone, small ones alone,
// or the full rounds in large and the remaining rows in small tiles; large ones alone also if they
// cost 0.15 more (20,000 rows: two rounds 78.3 us, one and 0.9 of one in small tiles 84.3, as the second
// launch starts in the first one's idle end), and two launches only if they cost 0.1 less.  Over 168
// products (1 to 42,196 rows; N = 100 to 6,854; K = 592 to 3,424) the choice is within 7% of the best of
// the three.
pace_status_t launch_gemm(GemmParams p, int nz, hipStream_t stream) {
  const int nc = p.mode == kEpiSwiglu ? p.N / 2 : p.N;
  uintptr_t bits = 2 * static_cast<uintptr_t>(nc);
  for (int z = 0; z < nz; ++z) bits |= reinterpret_cast<uintptr_t>(p.C[z]);
  if (p.mode == kEpiResidual) bits |= reinterpret_cast<uintptr_t>(p.R);
  p.width = bits % 16 == 0 ? 8 : bits % 8 == 0 ? 4 : bits % 4 == 0 ? 2 : 1;
  p.res_dma = p.width == 8 && p.N < (1 << 20);   // a tile's rows of R within one buffer's range
  const long long rows = (p.M + 255) / 256, per_row = ((p.N + 255) / 256) * static_cast<long long>(nz);
  const long long small_cols = ((p.N + 127) / 128) * static_cast<long long>(nz);
  auto small_cost = [&](long long r) {   // of the rows from 256 r on; eight small tiles cover a large one
    const long long t = (p.M - 256 * r + 63) / 64 * small_cols;
    return t <= 0 ? 0.0 : fmax(0.3, static_cast<double>(t) / (8 * 156.0));
  };
  auto cost = [&](long long r) { return static_cast<double>((r * per_row + 255) / 256) + small_cost(r); };
  const long long full = rows * per_row / 256 * 256 / per_row;   // row tiles in full rounds
  long long best = 0;
  if (cost(full) + 0.1 < cost(best)) best = full;
  if (cost(rows) <= cost(best) + 0.15) best = rows;
  const int m0 = static_cast<int>(best * 256 < p.M ? best * 256 : p.M);
  if (m0 > 0) {
    GemmParams q = p;
    q.M = m0;
    launch_tile<4, 2, 2, 4, 2>(q, nz, stream);
  }
  if (m0 < p.M) {
    GemmParams q = p;
    q.M = p.M - m0;
    q.A += static_cast<long long>(m0) * p.K;
    if (q.R != nullptr) q.R += static_cast<long long>(m0) * p.N;
    for (int z = 0; z < nz; ++z) q.C[z] += static_cast<long long>(m0) * nc;
    launch_tile<2, 1, 1, 4, 3>(q, nz, stream);
  }
  return check_launch("gemm_bf16_nt");
}

}  // namespace
}  // namespace pace

using namespace pace;

extern "C" {

pace_status_t pace_gemm_bf16(const uint16_t* A, const uint16_t* B, const float* bias, const uint16_t* residual,
                             uint16_t* C, int M, int N, int K, int epilogue, hipStream_t stream) {
  PACE_REQUIRE(A && B && C, "pace_gemm_bf16: null device pointer");
  PACE_REQUIRE(epilogue >= 0 && epilogue <= 2, "pace_gemm_bf16: epilogue %d not in {0, 1, 2}", epilogue);
  PACE_REQUIRE(epilogue != 1 || residual != nullptr, "pace_gemm_bf16: residual epilogue without residual");
  PACE_REQUIRE(epilogue != 2 || N % 2 == 0, "pace_gemm_bf16: SwiGLU needs an even N");
  GemmParams p{};
  p.A = A; p.B[0] = B; p.bias[0] = bias; p.R = residual; p.C[0] = C;
  p.M = M; p.N = N; p.K = K;
  p.mode = epilogue;
  const pace_status_t st = check_gemm(p, 1);
  return st != PACE_OK ? st : launch_gemm(p, 1, stream);
}

size_t pace_apc_preview_workspace_size(int N, int dim, int ffn, int patch) {
  if (N <= 0 || dim <= 0 || ffn <= 0 || patch <= 0) return 0;
  const int kp = (3 * patch * patch + 7) / 8 * 8;
  Sizer s;
  s.take<uint16_t>(static_cast<size_t>(N) * kp);        // patch rows
  for (int i = 0; i < 7; ++i) s.take<uint16_t>(static_cast<size_t>(N) * dim);   // h0 u q k v o h1
  s.take<uint16_t>(static_cast<size_t>(N) * ffn);       // SwiGLU hidden
  return s.off;
}

pace_status_t pace_apc_preview(const uint8_t* img, int H, int W, int patch, const int32_t* token_patch,
                               const int32_t* cu_windows, int nwin, int max_window,
                               const pace_preview_weights* w, uint16_t* out, void* workspace,
                               size_t workspace_bytes, hipStream_t stream) {
  PACE_REQUIRE(img && token_patch && cu_windows && w && out, "pace_apc_preview: null pointer");
  PACE_REQUIRE(patch >= 1 && patch <= 16 && H >= patch && W >= patch && H % patch == 0 && W % patch == 0,
               "pace_apc_preview: H=%d W=%d must be multiples of patch=%d (1..16)", H, W, patch);
  const int gh = H / patch, gw = W / patch;
  const long long Nl = static_cast<long long>(gh) * gw;
  PACE_REQUIRE(Nl < (1 << 24), "pace_apc_preview: too many patches");
  const int N = static_cast<int>(Nl);
  const int D = w->dim, F = w->ffn;
  PACE_REQUIRE(D >= 80 && D % 80 == 0 && F >= 8 && F % 8 == 0,
               "pace_apc_preview: dim=%d must be a multiple of 80 and ffn=%d of 8", D, F);
  PACE_REQUIRE(nwin >= 1 && max_window >= 1 && max_window <= N && max_window < 1024,
               "pace_apc_preview: nwin=%d max_window=%d (windows are shorter than 1024 tokens)", nwin, max_window);
  PACE_REQUIRE(w->pe && w->g1 && w->wq && w->wk && w->wv && w->wo && w->g2 && w->wgu && w->wd,
               "pace_apc_preview: a weight pointer is null");
  PACE_REQUIRE(aligned16(out), "pace_apc_preview: out must be 16-byte aligned");
  const int kp = (3 * patch * patch + 7) / 8 * 8;
  const size_t need = pace_apc_preview_workspace_size(N, D, F, patch);
  if (workspace == nullptr || workspace_bytes < need)
    return set_error(PACE_ERR_WORKSPACE, "pace_apc_preview: workspace %zu < %zu bytes", workspace_bytes, need);
  pace_status_t st = check_offsets(cu_windows, nwin, N, max_window, "pace_apc_preview: cu_windows", stream);
  if (st != PACE_OK) return st;
  if (debug_checks()) {
    st = check_values(token_patch, N, nullptr, 0, N - 1, "pace_apc_preview: token_patch", stream);
    if (st != PACE_OK) return st;
  }
  Carver c(workspace, workspace_bytes);
  uint16_t* X = c.take<uint16_t>(static_cast<size_t>(N) * kp);
  uint16_t* h0 = c.take<uint16_t>(static_cast<size_t>(N) * D);
  uint16_t* u = c.take<uint16_t>(static_cast<size_t>(N) * D);
  uint16_t* q = c.take<uint16_t>(static_cast<size_t>(N) * D);
  uint16_t* k = c.take<uint16_t>(static_cast<size_t>(N) * D);
  uint16_t* v = c.take<uint16_t>(static_cast<size_t>(N) * D);
  uint16_t* o = c.take<uint16_t>(static_cast<size_t>(N) * D);
  uint16_t* h1 = c.take<uint16_t>(static_cast<size_t>(N) * D);
  uint16_t* hm = c.take<uint16_t>(static_cast<size_t>(N) * F);

  const long long total = static_cast<long long>(N) * (kp / 8);
  hipLaunchKernelGGL(preview_patchify, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, stream,
                     img, W, patch, gw, token_patch, N, kp, X);
  if ((st = check_launch("preview_patchify")) != PACE_OK) return st;
  if ((st = pace_gemm_bf16(X, w->pe, nullptr, nullptr, h0, N, D, kp, 0, stream)) != PACE_OK) return st;
  hipLaunchKernelGGL(rmsnorm_bf16, dim3((N + 3) / 4), dim3(256), 0, stream, h0, w->g1, u, N, D, 1e-6f);
  if ((st = check_launch("rmsnorm_bf16")) != PACE_OK) return st;
  // q, k and v in one launch: three times the tiles, so a smaller part of the last round is idle
  GemmParams g{};
  g.A = u;
  g.B[0] = w->wq; g.B[1] = w->wk; g.B[2] = w->wv;
  g.bias[0] = w->bq; g.bias[1] = w->bk; g.bias[2] = w->bv;
  g.C[0] = q; g.C[1] = k; g.C[2] = v;
  g.M = N; g.N = D; g.K = D;
  g.mode = kEpiBias;
  if ((st = check_gemm(g, 3)) != PACE_OK) return st;
  if ((st = launch_gemm(g, 3, stream)) != PACE_OK) return st;
  if ((st = pace_vit_attention(q, k, v, N, D / 80, 80, cu_windows, nwin, max_window, 1.0f / sqrtf(80.f), o,
                               nullptr, nullptr, nullptr, 0, stream)) != PACE_OK)
    return st;
  if ((st = pace_gemm_bf16(o, w->wo, w->bo, h0, h1, N, D, D, 1, stream)) != PACE_OK) return st;
  hipLaunchKernelGGL(rmsnorm_bf16, dim3((N + 3) / 4), dim3(256), 0, stream, h1, w->g2, u, N, D, 1e-6f);
  if ((st = check_launch("rmsnorm_bf16")) != PACE_OK) return st;
  if ((st = pace_gemm_bf16(u, w->wgu, w->bgu, nullptr, hm, N, 2 * F, D, 2, stream)) != PACE_OK) return st;
  return pace_gemm_bf16(hm, w->wd, w->bd, h1, out, N, D, F, 1, stream);
}

}  // extern "C"
