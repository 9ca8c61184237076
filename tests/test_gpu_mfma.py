"""The matrix-core convolution (fp16, algo 0 with the storage's scratch) at
the sizes where its tiles can go wrong: both parity gates against the oracle
(the products are exact and the sums fp32, so the gates of the vector kernels
hold), guard bands, a bitwise rerun, rows off their 8-byte boundaries, and
non-finite inputs, which must reach exactly the outputs whose kept weights
read them."""
import numpy as np
import pytest

from paper_2003_06513_amd import binding as B
from synthetic import inputs
from gpu_cases import check_output, dev, max_terms, note, oracle_ref, prepared_case, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    B.lib()


# n, cin, cout, h, w, drop, stride, m: one and several column strips, rows of
# 4k, 2k and odd columns, images that end inside a tile, ragged filters and
# channels, every tile (64, 128, 256 pixels; 4 and 8 waves), both strides
CASES = [
    (32, 64, 64, 28, 28, 50, 1, 8),       # 128 pixels
    (4, 33, 65, 57, 61, 0, 1, 12),        # 64 pixels, odd strips
    (200, 33, 65, 7, 9, 0, 1, 5),         # odd rows, many images a tile
    (300, 64, 96, 4, 4, 0, 1, 56),        # the smallest rows; every pattern
    (600, 16, 64, 5, 6, 0, 1, 8),         # rows of 2k columns
    (6, 100, 48, 70, 66, 0, 1, 8),        # 3 strips of 22 columns, 3 of 32 channels and 4 over
    (1, 64, 64, 112, 112, 60, 1, 8),      # 8 waves, 128 pixels
    (2, 128, 128, 56, 56, 60, 1, 8),      # 8 waves, 64 pixels
    (32, 64, 64, 56, 56, 60, 1, 8),       # 256 pixels
    (16, 64, 128, 33, 35, 20, 2, 8),      # stride 2, odd sizes
    (64, 64, 64, 32, 32, 20, 2, 8),       # stride 2, 4k columns
]


def _make(case, seed=5):
    n, cin, cout, h, w, drop, stride, m = case
    wt = inputs.he_weights(seed, cout, cin, np.float16)
    masks = B.select_library(wt, m)
    prep, packed = prepared_case(wt, masks, inputs.keep_after_drop(cout * cin, drop))
    assert B.conv3x3_on_matrix_cores(prep.layer, B.PSC_F16, n, h, w, False, stride)
    return prep, packed, masks, inputs.normal_activations(seed + 1, (n, cin, h, w), np.float16)


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
@pytest.mark.parametrize("offset", [0, 1])
def test_parity_guard_rerun(case, offset):
    torch = torch_mod()
    n, cin, cout, h, w, drop, stride, m = case
    prep, packed, masks, x = _make(case)
    bias, relu = (inputs.bias_vector(9, cout, np.float16), True) if offset else (None, False)
    oh, ow = (h - 1) // stride + 1, (w - 1) // stride + 1
    numel, guard = n * cout * oh * ow, 4096
    buf = torch.full((numel + 2 * guard,), 1234.5, dtype=torch.float16, device="cuda")
    y = buf[guard:guard + numel].view(n, cout, oh, ow)
    xd = torch.empty(x.size + offset, dtype=torch.float16, device="cuda")[offset:].view(x.shape)
    xd.copy_(dev(x))
    bd = None if bias is None else dev(bias)
    note("mfma %s offset %d" % (case, offset))
    B.conv3x3_fwd_strided(prep.layer, prep.packed, xd, y, stride, bias=bd, relu=relu)
    first = y.clone()
    prep.packed.work.fill_(255)
    y.fill_(-7.0)
    B.conv3x3_fwd_strided(prep.layer, prep.packed, xd, y, stride, bias=bd, relu=relu)
    torch.cuda.synchronize()
    assert torch.equal(first, y)
    assert bool((buf[:guard] == 1234.5).all()) and bool((buf[guard + numel:] == 1234.5).all())
    ref, s = oracle_ref(x, packed, masks, cout, bias=bias, relu=relu, stride=stride)
    check_output(y.cpu().numpy(), ref, s, np.float16, max_terms(packed), "mfma %s" % (case,))


@pytest.mark.parametrize("case", [CASES[1], CASES[7], CASES[9]], ids=["strips", "groups", "stride2"])
def test_non_finite_and_subnormal_inputs(case):
    """Against the one-output-per-lane kernel: the same infinities and NaNs;
    finite outputs within the rounding of both; subnormal inputs and weights
    count."""
    torch = torch_mod()
    n, cin, cout, h, w, drop, stride, m = case
    prep, packed, masks, x = _make(case)
    g = np.random.default_rng(3)
    for v in (np.inf, -np.inf, np.nan):
        for _ in range(3):
            x[g.integers(n), g.integers(cin), g.integers(h), g.integers(w)] = v
    x[0, 0, 0, 0] = x[-1, -1, -1, -1] = np.inf
    xd = dev(x)
    y = torch.empty((n, cout, (h - 1) // stride + 1, (w - 1) // stride + 1), dtype=torch.float16, device="cuda")
    z = torch.empty_like(y)
    note("mfma non-finite %s" % (case,))
    B.conv3x3_fwd_strided(prep.layer, prep.packed, xd, y, stride)
    B.conv3x3_fwd_strided(prep.layer, prep.packed, xd, z, stride, algo=1)
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(y), torch.isnan(z)) and torch.equal(torch.isinf(y), torch.isinf(z))
    ok = torch.isfinite(z)
    # two sums of at most 9 * cin terms of size < 6 in fp32, each rounded to fp16
    assert float((y[ok].float() - z[ok].float()).abs().max()) <= 2 * 2.0 ** -11 * float(z[ok].float().abs().max())
    # inputs in the subnormal range: the output is exactly representable in fp32
    xs = torch.full((n, cin, h, w), 2.0 ** -24, dtype=torch.float16, device="cuda")
    prep.packed.values.copy_(torch.sign(prep.packed.values.float()).half() * 512)
    B.conv3x3_fwd_strided(prep.layer, prep.packed, xs, y, stride)
    B.conv3x3_fwd_strided(prep.layer, prep.packed, xs, z, stride, algo=1)
    torch.cuda.synchronize()
    assert torch.equal(y, z) and float(z.abs().max()) > 0


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c)) for c in CASES])
def test_non_finite_classes(case, relu):
    """Every tile, with kept weights that are zero of either sign (0 * inf is
    NaN, a pruned weight's is nothing), few and many infinities of both signs
    in reach of one output, NaNs, and a bias: the class of every output is that
    of the one-output-per-lane kernel, and the finite ones agree."""
    torch = torch_mod()
    n, cin, cout, h, w, drop, stride, m = case
    prep, packed, masks, x = _make(case)
    g = np.random.default_rng(11)
    v = prep.packed.values
    v[torch.from_numpy(g.random(v.numel()) < 0.1).cuda()] = 0.0
    v[torch.from_numpy(g.random(v.numel()) < 0.1).cuda()] = -0.0
    k = max(1, x.size // 100000)
    for val in (np.inf, -np.inf, np.nan):
        x.reshape(-1)[g.integers(0, x.size, k)] = val
    x[n - 1, :2, h - 1, 1], x[0, :2, 0, 0] = np.inf, -np.inf
    x[n // 2, :, h // 2] = np.inf                   # a whole row of every channel
    xd, bd = dev(x), dev(inputs.bias_vector(9, cout, np.float16))
    y = torch.empty((n, cout, (h - 1) // stride + 1, (w - 1) // stride + 1), dtype=torch.float16, device="cuda")
    z = torch.empty_like(y)
    note("mfma classes %s relu %d" % (case, relu))
    B.conv3x3_fwd_strided(prep.layer, prep.packed, xd, y, stride, bias=bd, relu=relu)
    B.conv3x3_fwd_strided(prep.layer, prep.packed, xd, z, stride, bias=bd, relu=relu, algo=1)
    torch.cuda.synchronize()
    assert torch.equal(torch.isnan(y), torch.isnan(z))
    assert torch.equal(torch.where(torch.isinf(y), y, 0), torch.where(torch.isinf(z), z, 0))
    ok = torch.isfinite(z)
    assert bool(ok.any()) and float((y[ok].float() - z[ok].float()).abs().max()) <= 2 * 2.0 ** -11 * float(z[ok].float().abs().max())
