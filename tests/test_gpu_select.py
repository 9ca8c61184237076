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


@pytest.mark.parametrize("keep", [1, 12000, 30000, 49151])
def test_ties_over_the_grid(keep):
    """More equal leading bits than the list holds, in every round and at
    every place where the rounds can end; repeated, and from two streams (each
    with its workspace) at a time."""
    torch = torch_mod()
    k = 48 * 1024 + 13                      # 13 chunks, the last one short
    rng = np.random.default_rng(keep)
    step = lambda b: 1.0 + rng.integers(0, 3, k) * 2.0 ** -b
    kinds = {"round%d" % i: step(b) for i, b in enumerate((22, 32, 42, 52))}
    kinds["mixed"] = np.where(rng.random(k) < 0.5, 1.0, 1.0 + rng.integers(0, 1 << 12, k) * 2.0 ** -52)
    kinds["small"] = np.where(rng.random(k) < 0.9, 0.0, 5e-324 * rng.integers(1, 9, k))
    L = B.Layer(1, k, [23, 282], keep, B.PSC_F32)
    for kind, e in kinds.items():
        want = oracle.select(e, keep)
        ed = dev(e)
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        ws = [B.workspace(L, B.PSC_OP_SELECT).fill_(255) for _ in streams]
        got = [torch.full((k,), 7, dtype=torch.uint8, device="cuda") for _ in streams]
        note("select rounds keep %d %s" % (keep, kind))
        torch.cuda.synchronize()
        for _ in range(5):
            for s, w, g in zip(streams, ws, got):
                B.select(L, ed, g, w, stream=s)
        torch.cuda.synchronize()
        for g in got:
            assert np.array_equal(g.cpu().numpy(), want), kind
