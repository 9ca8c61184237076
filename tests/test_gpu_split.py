"""The fp32 convolution on the 16-bit matrix cores (three bf16 parts), dense
and pattern-sparse, at the sizes where its tiles can go wrong, against float64
sums; and values that bf16 parts cannot hold."""
import numpy as np
import pytest

from paper_2003_06513_amd import binding as B
from synthetic import inputs
from gpu_cases import check_output, dev, gamma, max_terms, note, oracle_ref, prepared_case, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    B.lib()


def _conv(x, w):
    """float64 sums over taps and channels by the definition."""
    n, c, h, wd = x.shape
    p = np.zeros((n, c, h + 2, wd + 2))
    p[:, :, 1:-1, 1:-1] = x
    y = 0.0
    for q in range(9):
        t = p[:, :, q // 3:q // 3 + h, q % 3:q % 3 + wd].transpose(1, 0, 2, 3).reshape(c, -1)
        y = y + w[:, :, q // 3, q % 3].astype(np.float64) @ t
    return y.reshape(w.shape[0], n, h, wd).transpose(1, 0, 2, 3)


# n, cin, cout, h, w: one pixel tile and many, rows of 4k and other columns,
# one to several strips, channels and filters that end inside a tile
DENSE = [(1, 16, 32, 1, 4), (1, 17, 40, 3, 5), (2, 33, 65, 7, 7), (3, 48, 70, 8, 8), (40, 16, 32, 4, 6),
         (1, 31, 64, 21, 33), (2, 64, 64, 32, 32), (1, 20, 130, 9, 67), (1, 16, 48, 2, 200), (130, 32, 64, 16, 16)]


@pytest.mark.parametrize("shape", DENSE, ids=["x".join(map(str, s)) for s in DENSE])
@pytest.mark.parametrize("offset", [0, 1])
def test_dense(shape, offset):
    torch = torch_mod()
    n, cin, cout, h, w = shape
    x, wt, b = inputs.normal_activations(1, (n, cin, h, w)), inputs.he_weights(2, cout, cin), inputs.bias_vector(3, cout)
    xd = torch.empty(x.size + offset, device="cuda")[offset:].view(x.shape)
    xd.copy_(dev(x))
    buf = torch.full((n * cout * h * w + 2048,), 1234.5, device="cuda")
    y = buf[1024:-1024].view(n, cout, h, w)
    ws = B.dense3x3_fwd_workspace(B.PSC_F32, cin, cout)
    note("split dense %s offset %d" % (shape, offset))
    B.dense3x3_fwd(xd, dev(wt), y, bias=dev(b), relu=bool(offset), ws=ws)
    first = y.clone()
    ws.fill_(255)
    B.dense3x3_fwd(xd, dev(wt), y, bias=dev(b), relu=bool(offset), ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(first, y)
    assert bool((buf[:1024] == 1234.5).all()) and bool((buf[-1024:] == 1234.5).all())
    ref = _conv(x, wt) + b[:, None, None]
    ref = np.maximum(ref, 0) if offset else ref
    # each of the 9 cin products is within 2^-24 (one rounding), and the 9 cin
    # additions, the bias among them, round like fp32's
    bound = gamma(9 * cin + 1) * (_conv(np.abs(x), np.abs(wt)) + np.abs(b)[:, None, None])
    assert (np.abs(y.cpu().numpy() - ref) <= bound).all()


# n, cin, cout, h, w, drop, stride, m
SPARSE = [(32, 64, 64, 30, 30, 60, 1, 8), (48, 33, 120, 33, 35, 20, 1, 12), (64, 40, 128, 32, 32, 20, 2, 6),
          (16, 20, 64, 33, 35, 0, 2, 56), (200, 48, 96, 10, 8, 0, 2, 8), (24, 64, 64, 56, 56, 0, 1, 8)]


@pytest.mark.parametrize("case", SPARSE, ids=["x".join(map(str, c)) for c in SPARSE])
def test_sparse(case):
    torch = torch_mod()
    n, cin, cout, h, w, drop, stride, m = case
    wt = inputs.he_weights(5, cout, cin)
    masks = B.select_library(wt, m)
    prep, packed = prepared_case(wt, masks, inputs.keep_after_drop(cout * cin, drop))
    assert B.conv3x3_on_matrix_cores(prep.layer, B.PSC_F32, n, h, w, False, stride)
    x, b = inputs.normal_activations(6, (n, cin, h, w)), inputs.bias_vector(7, cout)
    y = torch.empty((n, cout, (h - 1) // stride + 1, (w - 1) // stride + 1), device="cuda")
    note("split sparse %s" % (case,))
    B.conv3x3_fwd_strided(prep.layer, prep.packed, dev(x), y, stride, bias=dev(b), relu=True)
    first = y.clone()
    prep.packed.work.fill_(255)
    B.conv3x3_fwd_strided(prep.layer, prep.packed, dev(x), y, stride, bias=dev(b), relu=True)
    torch.cuda.synchronize()
    assert torch.equal(first, y)
    ref, s = oracle_ref(x, packed, masks, cout, bias=b, relu=True, stride=stride)
    check_output(y.cpu().numpy(), ref, s, np.float32, max_terms(packed), "split %s" % (case,))


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -120])
def test_values_that_bf16_parts_cannot_hold(scale):
    """Against the one-output-per-lane kernel: the same infinities and NaNs,
    finite outputs within the bound of both; inputs near the smallest normal
    number keep their precision."""
    torch = torch_mod()
    n, cin, cout, h, w, drop, stride, m = SPARSE[0]
    wt = inputs.he_weights(5, cout, cin)
    masks = B.select_library(wt, m)
    prep, packed = prepared_case(wt, masks, inputs.keep_after_drop(cout * cin, drop))
    x = inputs.normal_activations(6, (n, cin, h, w)) * np.float32(scale)
    if scale == 1.0:
        x[0, 0, 0, 0], x[3, 5, 29, 29], x[7, 9, 4, 29], x[8, 1, 0, 7], x[-1, -1, -1, -1] = \
            np.inf, -np.inf, np.nan, 3.3e38, np.inf
    xd = dev(x)
    y = torch.empty((n, cout, h, w), device="cuda")
    z = torch.empty_like(y)
    note("split non-finite, scale %g" % scale)
    B.conv3x3_fwd(prep.layer, prep.packed, xd, y)
    B.conv3x3_fwd(prep.layer, prep.packed, xd, z, algo=1)
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(y), torch.isnan(z)) and torch.equal(torch.isinf(y), torch.isinf(z))
    ok = torch.isfinite(z)
    # two fp32 sums of the same products, of outputs of the same size
    lim = 2 * gamma(max_terms(packed)) * 8 * (float(np.sqrt(max_terms(packed))) * scale if scale != 1.0 else 1.0)
    d = (y[ok] - z[ok]).abs()
    assert float((d / z[ok].abs().clamp(min=scale)).max()) <= max(lim, 1e-4 if scale == 1.0 else lim / scale)


def _by_definition(x, w):
    """Sums over the taps inside the image alone (nothing is multiplied by the
    padding), float64."""
    n, c, h, wd = x.shape
    y = np.zeros((n, w.shape[0], h, wd))
    for q in range(9):
        r, s = q // 3 - 1, q % 3 - 1
        i0, i1, j0, j1 = max(0, -r), min(h, h - r), max(0, -s), min(wd, wd - s)
        xs = x[:, None, :, i0 + r:i1 + r, j0 + s:j1 + s].astype(np.float64)
        y[:, :, i0:i1, j0:j1] += (xs * w[None, :, :, q // 3, q % 3, None, None].astype(np.float64)).sum(2)
    return y


@pytest.mark.parametrize("filters", [(7,), (1, 2, 3), (21, 30), (64,)], ids=str)
@pytest.mark.parametrize("kind", ["weight", "x", "tiny", "tiny weights, large x", "large weights, tiny x"])
def test_dense_values_that_bf16_parts_cannot_hold(kind, filters):
    """Any filter of a block alone brings the block to the fp32 sums: an
    infinite weight, an infinite input beside zero columns, weights whose
    parts leave the range of bf16, and those against inputs (and the other way
    round) that lift the sums back into it."""
    torch = torch_mod()
    n, cin, cout, h, w = DENSE[2]
    x, wt = inputs.normal_activations(1, (n, cin, h, w)), inputs.he_weights(2, cout, cin)
    for f in filters:
        if kind == "weight":
            wt[f, 5, 0, 0], wt[f, 6, 2, 2] = np.inf, -3e38
        elif kind == "tiny":
            wt[f] *= np.float32(2.0 ** -120)
        elif kind == "tiny weights, large x":
            wt[f] *= np.float32(2.0 ** -121)
        elif kind == "large weights, tiny x":
            wt[f] *= np.float32(2.0 ** 60)
        else:
            wt[f, 9] = 0.0                          # 0 * inf
    if kind == "x":
        x[0, 9, 3, 3], x[1, 2, 0, 0], x[0, 4, 6, 6], x[1, 0, 2, 6] = np.inf, -np.inf, np.nan, 3.3e38
    x *= np.float32({"tiny weights, large x": 2.0 ** 60, "large weights, tiny x": 2.0 ** -124}.get(kind, 1.0))
    y = torch.empty((n, cout, h, w), device="cuda")
    note("split dense %s %s" % (kind, filters))
    B.dense3x3_fwd(dev(x), dev(wt), y, ws=B.dense3x3_fwd_workspace(B.PSC_F32, cin, cout))
    got = y.cpu().numpy().astype(np.float64)
    with np.errstate(all="ignore"):
        want = _by_definition(x, wt)
        want[np.abs(want) > np.finfo(np.float32).max] *= np.inf
        fin = lambda a: np.where(np.isfinite(a), np.abs(a.astype(np.float64)), 0)
        mag = _by_definition(fin(x), fin(wt))
    sure = mag < 3e38                               # a sum near the largest number may differ in kind
    assert np.array_equal(np.isnan(got)[sure], np.isnan(want)[sure])
    assert np.array_equal(np.isinf(got)[sure], np.isinf(want)[sure])
    ok = sure & np.isfinite(want)
    assert (np.abs(got[ok] - want[ok]) <= gamma(9 * cin + 1) * mag[ok] + 2 * 9 * cin * 2.0 ** -149).all()


@pytest.mark.parametrize("lift", [1.0, 2.0 ** 60])
def test_sparse_filters_that_bf16_parts_cannot_hold(lift):
    """The same for packed weights, filter by filter, against the
    one-output-per-lane kernel."""
    torch = torch_mod()
    n, cin, cout, h, w, drop, stride, m = SPARSE[3]
    x = dev(inputs.normal_activations(6, (n, cin, h, w)) * np.float32(lift))
    for f in (0, 1, 6, 11, 35, 63):
        wt = inputs.he_weights(5, cout, cin)
        masks = B.select_library(wt, m)
        wt[f] *= np.float32(2.0 ** -120)
        prep, packed = prepared_case(wt, masks, inputs.keep_after_drop(cout * cin, drop))
        assert B.conv3x3_on_matrix_cores(prep.layer, B.PSC_F32, n, h, w, False, stride)
        y = torch.empty((n, cout, (h - 1) // stride + 1, (w - 1) // stride + 1), device="cuda")
        z = torch.empty_like(y)
        note("split sparse tiny filter %d" % f)
        B.conv3x3_fwd_strided(prep.layer, prep.packed, x, y, stride)
        B.conv3x3_fwd_strided(prep.layer, prep.packed, x, z, stride, algo=1)
        torch.cuda.synchronize()
        # two fp32 sums of the same 4 cin products and outputs of one size
        top = float(z[:, f].abs().max())
        assert top > 0 and float((y[:, f] - z[:, f]).abs().max()) <= 2 * gamma(4 * cin) * top + 8 * cin * 2.0 ** -149
