"""Connectivity selection at the sizes and key distributions where its paths
meet (one block up to 16384 kernels, two histograms and a list up to 2^20, the
radix passes above): the keep mask equals the oracle's bit for bit, with ties
inside the list, past its end, and everywhere."""
import numpy as np
import pytest

import oracle
from paper_2003_06513_amd import binding as B
from gpu_cases import dev, note, torch_mod

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    B.lib()


def _energy(kind, k, rng):
    if kind == "random":
        return rng.standard_normal(k) ** 2
    if kind == "equal":
        return np.full(k, 0.375)
    if kind == "few":                      # eight values: thousands of ties
        return rng.integers(0, 8, k).astype(np.float64)
    if kind == "close":                    # equal leading bits, distinct below
        return 1.0 + rng.integers(0, 1 << 20, k) * 2.0 ** -52
    if kind == "pairs":                    # every value twice
        return np.repeat(rng.standard_normal((k + 1) // 2) ** 2, 2)[:k]
    e = rng.standard_normal(k) ** 2        # "zeros": an already pruned layer, and an infinity
    e[rng.random(k) < 0.7] = 0.0
    e[k // 2] = np.inf
    return e


@pytest.mark.parametrize("kind", ["random", "equal", "few", "close", "pairs", "zeros"])
@pytest.mark.parametrize("shape", [(1, 2), (5, 13), (64, 64), (1, 4097), (128, 128), (127, 130), (512, 512),
                                   (1024, 1024), (1024, 1025)], ids=str)
def test_keep_mask(shape, kind):
    torch = torch_mod()
    k = shape[0] * shape[1]
    rng = np.random.default_rng(k)
    e = _energy(kind, k, rng)
    ed = dev(e)
    for keep in {1, k // 3, k // 2, k - 1} - {0}:
        L = B.Layer(shape[0], shape[1], [23, 282], keep, B.PSC_F32)
        got = torch.full((k,), 7, dtype=torch.uint8, device="cuda")
        ws = B.workspace(L, B.PSC_OP_SELECT)
        ws.fill_(255)
        note("select %s %s keep %d" % (shape, kind, keep))
        B.select(L, ed, got, ws)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.select(e, keep))
        B.select_noalloc(L, ed, got.fill_(7))
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.select(e, keep))
