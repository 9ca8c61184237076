"""The matrix-core weight gradient at the sizes where its tiles can go wrong,
against a float64 sum on the CPU: dense (fp32, from three bf16 parts) and
masked (fp16 and fp32).  The bound per entry is gamma_n times the sum of the
absolute products, n the number of pixels (each of the n products is exact or
within 2^-24, one rounding; each addition rounds once; what the parts drop and
the slots' sums stay within the factor that the tests give)."""
import numpy as np
import pytest

from paper_2003_06513_amd import binding as B
from synthetic import inputs
from gpu_cases import dev, gamma, note, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    B.lib()


def _wgrad(x, g):
    """float64 dW [cout][cin][9] by the definition."""
    n, c, h, w = x.shape
    p = np.zeros((n, c, h + 2, w + 2))
    p[:, :, 1:-1, 1:-1] = x
    g2 = g.astype(np.float64).transpose(1, 0, 2, 3).reshape(g.shape[1], -1)
    out = np.empty((g.shape[1], c, 9))
    for q in range(9):
        t = p[:, :, q // 3:q // 3 + h, q % 3:q % 3 + w].transpose(1, 0, 2, 3).reshape(c, -1)
        out[:, :, q] = g2 @ t.T
    return out


# n, cin, cout, h, w: one to several groups of 8 columns with every remainder,
# rows split over tiles with halo groups, images inside and across tiles,
# ragged filters and channels, 32- and 64-wide blocks, one and many slots
SHAPES = [(1, 16, 1, 1, 1), (3, 17, 5, 2, 3), (5, 33, 40, 4, 4), (2, 16, 33, 7, 7), (4, 31, 70, 8, 8),
          (2, 40, 36, 9, 13), (1, 20, 65, 5, 16), (2, 16, 32, 6, 31), (1, 18, 34, 3, 61), (1, 32, 16, 5, 130),
          (1, 16, 20, 2, 300), (40, 16, 16, 4, 5), (9, 48, 24, 16, 15), (64, 512, 512, 4, 8), (2, 16, 16, 70, 9)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_dense_fp32(shape):
    torch = torch_mod()
    n, cin, cout, h, w = shape
    x, g = inputs.normal_activations(3, (n, cin, h, w)), inputs.normal_activations(4, (n, cout, h, w))
    dw, db = torch.empty((cout, cin, 3, 3), device="cuda"), torch.empty(cout, device="cuda")
    note("dense wgrad %s" % (shape,))
    ws = B.dense3x3_bwd_weight(dev(x), dev(g), dw, db)
    first = dw.clone()
    if ws is not None:
        ws.fill_(255)
    B.dense3x3_bwd_weight(dev(x), dev(g), dw, db, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(first, dw)
    err = np.abs(dw.cpu().numpy().reshape(cout, cin, 9) - _wgrad(x, g))
    bound = gamma(6 * n * h * w) * _wgrad(np.abs(x), np.abs(g)) + 1e-37
    assert (err <= bound).all(), float((err / bound).max())
    ref = g.astype(np.float64).sum((0, 2, 3))
    assert np.abs(db.cpu().numpy() - ref).max() <= gamma(n * h * w) * np.abs(g).sum((0, 2, 3)).max() + 1e-37


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("shape", SHAPES[2:10], ids=["x".join(map(str, s)) for s in SHAPES[2:10]])
def test_masked(shape, dtype):
    torch = torch_mod()
    n, cin, cout, h, w = shape
    x = inputs.normal_activations(5, (n, cin, h, w), dtype)
    g = inputs.normal_activations(6, (n, cout, h, w), dtype)
    wt = inputs.he_weights(7, cout, cin, dtype)
    masks = B.select_library(wt, 8)
    keep = inputs.keep_after_drop(cout * cin, 20)
    prep = B.prepare(dev(wt), masks, keep)
    dv = torch.empty(4 * keep, device="cuda")
    note("masked wgrad %s %s" % (shape, np.dtype(dtype).name))
    B.conv3x3_bwd_weight(prep.layer, prep.packed, dev(x), dev(g), dv)
    pk = prep.packed.to_host()
    pos = np.repeat(np.arange(cout), np.diff(pk["filter_ptr"]))
    bits = np.array([[b for b in range(9) if (int(c) >> b) & 1] for c in masks])[pk["pat_id"]]
    at = (pk["filter_perm"][pos][:, None], pk["cin_idx"][:, None], bits)
    err = np.abs(dv.cpu().numpy().reshape(-1, 4) - _wgrad(x, g)[at])
    bound = gamma(6 * n * h * w) * _wgrad(np.abs(x), np.abs(g))[at] + 1e-37
    assert (err <= bound).all(), float((err / bound).max())


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -122])
def test_values_that_bf16_parts_cannot_hold(scale):
    """Infinities and NaNs reach the entries that read them and no others
    (the zero columns beside the image must not make a NaN of an infinity);
    values near the smallest normal number keep their precision."""
    torch = torch_mod()
    n, cin, cout, h, w = 3, 40, 33, 6, 13
    x, g = inputs.normal_activations(3, (n, cin, h, w)), inputs.normal_activations(4, (n, cout, h, w))
    g *= np.float32(scale)
    if scale == 1.0:
        x[0, 1, 0, 0], x[1, 2, 5, 12], x[2, 3, 2, 12], x[0, 5, 3, 3] = np.inf, -np.inf, np.nan, 3.4e38
        g[1, 4, 5, 0] = np.inf
    dw = torch.empty((cout, cin, 3, 3), device="cuda")
    note("wgrad non-finite, scale %g" % scale)
    B.dense3x3_bwd_weight(dev(x), dev(g), dw)
    got = dw.cpu().numpy().reshape(cout, cin, 9).astype(np.float64)
    want = np.empty_like(got)
    with np.errstate(all="ignore"):
        for q in range(9):
            r, s = q // 3 - 1, q % 3 - 1
            i0, i1, j0, j1 = max(0, -r), min(h, h - r), max(0, -s), min(w, w - s)
            xs = x[:, :, i0 + r:i1 + r, j0 + s:j1 + s].astype(np.float64)
            gs = g[:, :, i0:i1, j0:j1].astype(np.float64)
            want[:, :, q] = (gs[:, :, None] * xs[:, None]).sum((0, 3, 4))
    # 3.4e38 times a few may pass the largest number: those entries may differ in kind
    big = np.zeros(got.shape, bool)
    big[:, 5] = scale == 1.0
    assert np.array_equal(np.isnan(got)[~big], np.isnan(want)[~big])
    assert np.array_equal(np.isinf(got)[~big], np.isinf(want)[~big])
    ok = np.isfinite(want) & ~big
    mag = _wgrad(np.where(np.isfinite(x), np.abs(x), 0), np.where(np.isfinite(g), np.abs(g), 0))
    assert (np.abs(got[ok] - want[ok]) <= gamma(6 * n * h * w) * mag[ok] + 300 * 2.0 ** -149).all()


# n, cin, cout, h, w: 32-wide blocks (rows whole and in parts, ragged), and
# 64-wide ones (at least 64 of them, and 4096 pixels)
NON_FINITE = [(40, 33, 70, 9, 13), (3, 48, 36, 20, 130), (64, 512, 500, 8, 8)]


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("shape", NON_FINITE, ids=["x".join(map(str, s)) for s in NON_FINITE])
def test_masked_non_finite(shape, dtype):
    """Infinities and NaNs, also at the edges of the image beside the zero
    padding, reach the entries that read them and no others; every kernel is
    kept, so every call takes the matrix cores."""
    torch = torch_mod()
    n, cin, cout, h, w = shape
    x = inputs.normal_activations(5, (n, cin, h, w), dtype)
    g = inputs.normal_activations(6, (n, cout, h, w), dtype)
    x[0, 1, 0, 0], x[n - 1, 2, h - 1, w - 1], x[1, 3, 2, w - 1] = np.inf, -np.inf, np.nan
    g[1, 4, h - 1, 0], g[0, 7, 0, w - 1], g[1, 8, 2, 3] = np.inf, -np.inf, np.nan
    wt = inputs.he_weights(7, cout, cin, dtype)
    masks = B.select_library(wt, 8)
    prep = B.prepare(dev(wt), masks, cout * cin)
    dv = torch.empty(4 * cout * cin, device="cuda")
    note("masked wgrad non-finite %s %s" % (shape, np.dtype(dtype).name))
    ws = B.conv3x3_bwd_weight(prep.layer, prep.packed, dev(x), dev(g), dv)
    assert ws.numel() % (36 * cout * cin) == 0  # slots of the dense gradient
    pk = prep.packed.to_host()
    pos = np.repeat(np.arange(cout), np.diff(pk["filter_ptr"]))
    bits = np.array([[b for b in range(9) if (int(c) >> b) & 1] for c in masks])[pk["pat_id"]]
    filters = [0, 4, 7, 8, cout - 1]
    got = np.zeros((cout, cin, 9))
    kept = np.zeros((cout, cin, 9), bool)
    at = (pk["filter_perm"][pos][:, None], pk["cin_idx"][:, None], bits)
    got[at], kept[at] = dv.cpu().numpy().reshape(-1, 4), True
    fin = lambda a: np.where(np.isfinite(a), np.abs(a.astype(np.float64)), 0)
    mag = _wgrad(fin(x), fin(g))
    for f in filters:
        want = np.empty((cin, 9))
        with np.errstate(all="ignore"):
            for q in range(9):
                r, s = q // 3 - 1, q % 3 - 1
                i0, i1, j0, j1 = max(0, -r), min(h, h - r), max(0, -s), min(w, w - s)
                xs = x[:, :, i0 + r:i1 + r, j0 + s:j1 + s].astype(np.float64)
                want[:, q] = (g[:, f, None, i0:i1, j0:j1].astype(np.float64) * xs).sum((0, 2, 3))
        k = kept[f]
        assert np.array_equal(np.isnan(got[f][k]), np.isnan(want[k]))
        assert np.array_equal(np.isinf(got[f][k]), np.isinf(want[k]))
        ok = k & np.isfinite(want)
        assert f or ok.any()
        assert (np.abs(got[f][ok] - want[ok]) <= gamma(6 * n * h * w) * mag[f][ok] + 1e-37).all()


@pytest.mark.parametrize("tiny", ["g", "x"])
@pytest.mark.parametrize("channel", [0, 3, 7, 33])
def test_tiny_values_against_large_ones(channel, tiny):
    """One filter's gradient (one channel's input) whose parts leave the range
    of bf16, against values that lift the sums back into it: the error stays
    that of fp32 sums."""
    n, cin, cout, h, w = 3, 40, 36, 6, 13
    x, g = inputs.normal_activations(3, (n, cin, h, w)), inputs.normal_activations(4, (n, cout, h, w))
    small, large = (g, x) if tiny == "g" else (x, g)
    small[:, channel] *= np.float32(2.0 ** -124)
    large *= np.float32(2.0 ** 60)
    torch = torch_mod()
    dw = torch.empty((cout, cin, 3, 3), device="cuda")
    note("wgrad tiny %s, channel %d" % (tiny, channel))
    B.dense3x3_bwd_weight(dev(x), dev(g), dw)
    err = np.abs(dw.cpu().numpy().reshape(cout, cin, 9) - _wgrad(x, g))
    bound = gamma(n * h * w) * _wgrad(np.abs(x), np.abs(g)) + n * h * w * 2.0 ** -105
    assert (err <= bound).all(), float((err / bound).max())


# 32-wide blocks (ragged, rows whole and in parts), and 64-wide ones (at least
# 64 of them and 4096 pixels in fp16; rows of one group in fp32), also ragged
ROUTED = [(40, 60, 70, 9, 13), (3, 48, 36, 20, 130), (256, 64, 64, 7, 8), (64, 512, 512, 8, 8), (40, 500, 460, 10, 13),
          (70, 460, 500, 9, 7)]


@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("shape", ROUTED, ids=["x".join(map(str, s)) for s in ROUTED])
def test_masked_on_matrix_cores(shape, dtype):
    """The masked gradient of calls that take the dense one (the workspace is
    whole slots of it), for some filters of each block."""
    torch = torch_mod()
    n, cin, cout, h, w = shape
    x = inputs.normal_activations(5, (n, cin, h, w), dtype)
    g = inputs.normal_activations(6, (n, cout, h, w), dtype)
    wt = inputs.he_weights(7, cout, cin, dtype)
    masks = B.select_library(wt, 8)
    keep = inputs.keep_after_drop(cout * cin, 20)
    prep = B.prepare(dev(wt), masks, keep)
    dv = torch.empty(4 * keep, device="cuda")
    note("masked wgrad routed %s %s" % (shape, np.dtype(dtype).name))
    ws = B.conv3x3_bwd_weight(prep.layer, prep.packed, dev(x), dev(g), dv)
    bias = -(-n * h * w // 8192) * 4 * cout if n * h * w > 8192 else 0
    assert (ws.numel() - bias) % (36 * cout * cin) == 0 and (ws.numel() - bias) % (16 * keep) != 0
    pk = prep.packed.to_host()
    pos = np.repeat(np.arange(cout), np.diff(pk["filter_ptr"]))
    bits = np.array([[b for b in range(9) if (int(c) >> b) & 1] for c in masks])[pk["pat_id"]]
    f = pk["filter_perm"][pos]
    some = [c for c in sorted({0, 5, 31, 32, 38, 63, 64, 200, cout - 1}) if c < cout]
    on = np.isin(f, some)
    at = (np.searchsorted(some, f[on])[:, None], pk["cin_idx"][on][:, None], bits[on])
    gs = np.ascontiguousarray(g[:, some])
    err = np.abs(dv.cpu().numpy().reshape(-1, 4)[on] - _wgrad(x, gs)[at])
    bound = gamma(6 * n * h * w) * _wgrad(np.abs(x), np.abs(gs))[at] + 1e-37
    assert on.any() and (err <= bound).all(), float((err / bound).max())
