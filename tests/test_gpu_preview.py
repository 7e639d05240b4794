"""GPU parity of the APC preview block (pace_apc_preview, pace_gemm_bf16) against the float64
oracle (oracle/preview.py).

GEMM: every output within 2^-8 of |ref| (its bf16 rounding) plus 1e-3 of the output's RMS
(fp32 accumulation over K).  Block: the GPU stores ten intermediate activations in bf16
(relative rounding 2^-9 each), and each passes through products of depth up to 3420. Summed over
the chain that is about 2% for a single worst element and well under 1% in RMS. So the output's
RMS error is bounded by 1e-2 of the output RMS and its largest error by 6e-2 of it, and every
row's cosine with the oracle's must be >= 0.999. The APC scores computed from the GPU embeddings
agree with the oracle's scores of the oracle embeddings to 2e-3."""
import numpy as np
import pytest

from oracle import apc as oapc
from oracle import preview as opv
from paper_2608_27206_amd import workloads as wl
from tests.gpu_util import dev_bf16, dev_f32, dev_i32, dev_u8, host, host_bf16_to_f64, rho4, say

pytestmark = pytest.mark.gpu


def _silu(x):
    return x / (1.0 + np.exp(-x))


@pytest.mark.parametrize("M,N,K,epi", [(300, 200, 72, 0), (1024, 1280, 1280, 0), (129, 257, 8, 1),
                                       (513, 384, 592, 1), (200, 96, 1280, 2), (1, 2, 16, 2),
                                       # large tiles alone; full rounds of them and the remaining rows
                                       # in small ones (bias, residual, residual at a row length that
                                       # has no 16-byte chunks, SwiGLU); one and two stages of K
                                       (10500, 1280, 64, 0), (15460, 1280, 72, 1), (15461, 1276, 40, 1),
                                       (15460, 1280, 104, 2), (10241, 1290, 16, 2)])
def test_gemm_epilogues(M, N, K, epi):
    from paper_2608_27206_amd import pace
    import torch
    say(f"gemm M={M} N={N} K={K} epilogue={epi}")
    rs = np.random.default_rng(M * 7 + N + K)
    a = wl.f32_to_bf16_bits(rs.normal(size=(M, K)).astype(np.float32))
    b = wl.f32_to_bf16_bits((rs.normal(size=(N, K)) / np.sqrt(K)).astype(np.float32))
    bias = rs.normal(size=N).astype(np.float32) * 0.1
    res = wl.f32_to_bf16_bits(rs.normal(size=(M, N)).astype(np.float32))
    out = pace.gemm_bf16(dev_bf16(a), dev_bf16(b), dev_f32(bias), dev_bf16(res) if epi == 1 else None, epi)
    torch.cuda.synchronize()
    got = host_bf16_to_f64(out)
    ref = wl.bf16_bits_to_f64(a) @ wl.bf16_bits_to_f64(b).T + bias[None, :]
    if epi == 1:
        ref = ref + wl.bf16_bits_to_f64(res)
    if epi == 2:
        ref = _silu(ref[:, 0::2]) * ref[:, 1::2]
    tol = 2.0 ** -8 * np.abs(ref) + 1e-3 * np.sqrt(np.mean(ref ** 2))
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) - tol))


def _sampled_gemm(M, N, K, epi, rows, c_off=0, r_off=0, in_place=False):
    """Rows `rows` of a product against float64; C and the residual start c_off and r_off elements
    past a 16-byte boundary, and nothing around C is written."""
    from paper_2608_27206_amd import pace
    import torch
    say(f"gemm M={M} N={N} K={K} epilogue={epi} offsets {c_off} {r_off}")
    gen = torch.Generator(device="cuda").manual_seed(M + 3 * N + K)
    nc = N // 2 if epi == 2 else N
    normal = lambda *s: torch.randn(*s, generator=gen, device="cuda")   # noqa: E731
    a, b, bias = normal(M, K).bfloat16(), (normal(N, K) / K ** 0.5).bfloat16(), 0.1 * normal(N)
    res = normal(M * N + 16).bfloat16()[r_off:r_off + M * N].view(M, N) if epi == 1 else None
    buf = torch.full((M * nc + 32,), 7.0, dtype=torch.bfloat16, device="cuda")
    out = buf[8 + c_off:8 + c_off + M * nc].view(M, nc)
    rows = np.unique(np.clip(np.asarray(rows), 0, M - 1))
    sel = torch.from_numpy(rows).cuda()
    r64 = host_bf16_to_f64(res[sel]) if epi == 1 else 0.0
    if in_place:
        out.copy_(res)
        res = out
    pace.gemm_bf16(a, b, bias, res, epi, out=out)
    torch.cuda.synchronize()
    assert torch.all(buf[:8 + c_off] == 7.0) and torch.all(buf[8 + c_off + M * nc:] == 7.0)
    ref = host_bf16_to_f64(a[sel]) @ host_bf16_to_f64(b).T + host(bias).astype(np.float64)[None, :] + r64
    if epi == 2:
        ref = _silu(ref[:, 0::2]) * ref[:, 1::2]
    got = host_bf16_to_f64(out[sel])
    tol = 2.0 ** -8 * np.abs(ref) + 1e-3 * np.sqrt(np.mean(ref ** 2))
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) - tol))


@pytest.mark.parametrize("M,N,K,epi", [(10500, 1280, 200, 0), (10300, 1280, 136, 1), (15460, 1280, 592, 1),
                                       (10241, 1280, 1288, 2), (15460, 1284, 328, 2)])
def test_gemm_large_tiles_over_many_stages(M, N, K, epi):
    """The 256 x 256 tiles with K in more stages than their ring holds (even and odd numbers, tails of 8 to
    48 values), alone and with the remaining rows in small tiles: rows at both ends of the tiles, at
    the line between the two and at the end."""
    ends = np.concatenate([np.arange(0, M, 256), np.arange(255, M, 256), np.arange(128, M, 512)])
    _sampled_gemm(M, N, K, epi, np.concatenate([ends, np.arange(13050, 13060), np.arange(M - 66, M)]))


@pytest.mark.parametrize("N,c_off,r_off,width", [(264, 0, 0, 8), (264, 4, 0, 4), (264, 0, 4, 4), (268, 0, 0, 4),
                                                 (268, 2, 4, 2), (270, 0, 0, 2), (270, 0, 1, 1), (271, 0, 0, 1)])
@pytest.mark.parametrize("M", [70, 66000])
def test_gemm_row_alignment(M, N, c_off, r_off, width):
    """Rows of C and of the residual at every alignment (accesses of `width` elements), in small and
    in large tiles, with each epilogue; the residual also in place."""
    rows = np.concatenate([np.arange(70), np.arange(0, M, 1021), np.arange(M - 70, M)])
    for epi, in_place in ((0, False), (1, False), (1, r_off == c_off), (2, False)):
        if epi != 2 or N % 2 == 0:
            _sampled_gemm(M, N, 72, epi, rows, c_off, r_off, in_place)


def test_swiglu_in_single_precision():
    """SiLU(gate) up to 2^-21: expf's 2^-23, and 2^-24 each for 1 + e, the division and the product come to
    5 x 2^-24.  The products are zero, so gate and up are the fp32 biases; up puts each result 2^-21 to
    either side of the middle between two bf16 values, and the right one of the two has to come out."""
    from paper_2608_27206_amd import pace
    import torch
    rs = np.random.default_rng(5)
    n = 8192
    gate = np.concatenate([rs.uniform(-80, 20, n - 64), rs.normal(0, 1, 64)]).astype(np.float32)
    silu = gate.astype(np.float64) / (1.0 + np.exp(-gate.astype(np.float64)))
    mid = 1.0 + (2 * rs.integers(0, 128, n) + 1) * 2.0 ** -8
    side = np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    up = (mid * (1.0 + side * 1.2 * 2.0 ** -21) / np.abs(silu)).astype(np.float32)
    val = np.abs(silu) * up.astype(np.float64)
    ok = (np.abs(val / mid - 1.0) >= 2.0 ** -21) & (np.sign(val - mid) == side) & np.isfinite(up)
    assert ok.mean() > 0.99   # up's own rounding moves few of them closer
    bias = np.stack([gate, up], 1).reshape(-1)
    a, b = np.zeros((3, 8), np.uint16), np.zeros((2 * n, 8), np.uint16)
    got = host_bf16_to_f64(pace.gemm_bf16(dev_bf16(a), dev_bf16(b), torch.from_numpy(bias).cuda(), None, 2))
    want = np.sign(silu) * (mid + side * 2.0 ** -8)
    assert np.array_equal(got[:, ok], np.broadcast_to(want[ok], got[:, ok].shape)), np.mean(got[0, ok] != want[ok])


def _block_case(H, W, seed=11):
    from paper_2608_27206_amd import pace
    import torch
    img = wl.make_image(1, H, W)
    lay = wl.vit_layout(H // 14, W // 14)
    w = wl.preview_weights(seed)
    wdev = pace.preview_weights_to_device(w, torch.device("cuda"))
    out = pace.apc_preview(dev_u8(img), 14, dev_i32(lay.order), dev_i32(lay.cu_windows),
                           int(np.max(lay.window_sizes)), wdev)
    rho, d = pace.apc_density_features(out)
    torch.cuda.synchronize()
    w64 = {k: (wl.bf16_bits_to_f64(v) if v.dtype == np.uint16 else v.astype(np.float64)) for k, v in w.items()}
    ref = opv.preview_block(opv.patch_rows(img, 14, lay.order), w64, lay.cu_windows)
    return host_bf16_to_f64(out), ref, host(rho), host(d)


def _check_block(got, ref, name):
    rms = np.sqrt(np.mean(ref ** 2))
    err = got - ref
    rel_max = np.max(np.abs(err)) / rms
    rel_rms = np.sqrt(np.mean(err ** 2)) / rms
    cos = np.sum(got * ref, axis=1) / (np.linalg.norm(got, axis=1) * np.linalg.norm(ref, axis=1))
    say(f"preview {name}: max err / rms = {rel_max:.3g}, rms err / rms = {rel_rms:.3g}, "
        f"min row cosine = {cos.min():.6f}")
    assert rel_rms <= 1e-2
    assert rel_max <= 6e-2
    assert cos.min() >= 0.999


def test_preview_block_448():
    got, ref, rho, d = _block_case(448, 448)
    _check_block(got, ref, "448")
    dens = oapc.embedding_density(ref)
    say(f"rho gpu {rho} oracle {[dens['rho_g'], dens['rho_d'], dens['rho'], dens['phi']]}")
    np.testing.assert_allclose(rho4(rho), [dens["rho_g"], dens["rho_d"], dens["rho"], dens["phi"]], atol=2e-3)


def test_preview_block_ragged_windows():
    """A grid whose windows are cut at the right and bottom edges (partial windows)."""
    got, ref, rho, d = _block_case(196, 308, seed=12)
    _check_block(got, ref, "196x308")


@pytest.mark.parametrize("patch,gh,gw", [(1, 9, 7), (2, 6, 10), (3, 4, 6), (5, 3, 7), (8, 2, 3), (13, 3, 2), (16, 2, 4)])
def test_patch_rows_of_every_patch_size(patch, gh, gw):
    """Patch rows whose 16-byte chunks end inside, at and across a row of the patch: with zero
    output projections the block is its patch embedding, compared with float64 to the GEMM's
    tolerance."""
    from paper_2608_27206_amd import pace
    import torch
    rs = np.random.default_rng(patch)
    img = rs.integers(0, 256, size=(gh * patch, gw * patch, 3), dtype=np.uint8)
    kin, D = 3 * patch * patch, 80
    w = {"pe": wl.f32_to_bf16_bits(rs.normal(size=(D, kin)).astype(np.float32))}
    for k in ("wq", "wk", "wv", "wo"):
        w[k] = np.zeros((D, D), np.uint16)
    w["wg"], w["wu"], w["wd"] = np.zeros((8, D), np.uint16), np.zeros((8, D), np.uint16), np.zeros((D, 8), np.uint16)
    for k in ("bq", "bk", "bv", "bo", "bd"):
        w[k] = np.zeros(D, np.float32)
    w["bg"] = w["bu"] = np.zeros(8, np.float32)
    w["g1"] = w["g2"] = np.ones(D, np.float32)
    order = rs.permutation(gh * gw).astype(np.int32)
    say(f"preview patch={patch} grid={gh}x{gw}")
    out = pace.apc_preview(dev_u8(img), patch, dev_i32(order), dev_i32([0, gh * gw]), gh * gw,
                           pace.preview_weights_to_device(w, torch.device("cuda")))
    torch.cuda.synchronize()
    x = img.reshape(gh, patch, gw, patch, 3).transpose(0, 2, 1, 3, 4).reshape(gh * gw, kin)[order] / 127.5 - 1.0
    x = wl.bf16_bits_to_f64(wl.f32_to_bf16_bits(x.astype(np.float32)))
    ref = x @ wl.bf16_bits_to_f64(w["pe"]).T
    err = np.abs(host_bf16_to_f64(out) - ref) - (2.0 ** -8 * np.abs(ref) + 1e-3 * np.sqrt(np.mean(ref ** 2)))
    assert err.max() <= 0
