"""The scratch of the matrix-core convolution: a storage holds its arrays and
nothing else, each call has scratch of its own (two storages that share arrays
on two streams, calls on a side stream, capture), and a scratch that a caller
keeps with the storage gives the same bytes."""
import copy

import numpy as np
import pytest

from paper_2003_06513_amd import binding as B
from synthetic import inputs
from gpu_cases import dev, note, torch_mod


@pytest.mark.parametrize("dtype", [B.PSC_F32, B.PSC_F16])
def test_storage_holds_its_arrays_alone(dtype):
    torch = torch_mod()
    p = B.Packed(B.Layer(512, 512, [23, 282], 1000, dtype), device="cpu")
    held = sum(t.numel() * t.element_size() for t in vars(p).values() if isinstance(t, torch.Tensor))
    assert held == sum(getattr(p, f).numel() * getattr(p, f).element_size() for f in B.PACKED_FIELDS)


def _need_gpu():
    if not torch_mod().cuda.is_available():
        pytest.skip("no HIP device")
    B.lib()


def _case(dtype, seed):
    """A layer that runs on the matrix cores: fp16 stride 1, fp32 stride 2."""
    torch = torch_mod()
    stride = 1 if dtype == np.float16 else 2
    wt = inputs.he_weights(seed, 128, 64, dtype)
    prep = B.prepare(dev(wt), B.select_library(wt, 8), inputs.keep_after_drop(128 * 64, 20))
    x = dev(inputs.normal_activations(seed + 1, (64, 64, 32, 32), dtype))
    y = torch.empty((64, 128, 32 // stride, 32 // stride), dtype=x.dtype, device="cuda")
    assert B.conv3x3_on_matrix_cores(prep.layer, prep.layer.dtype, 64, 32, 32, False, stride)
    return prep, x, y, stride


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_copies_on_two_streams(dtype):
    _need_gpu()
    torch = torch_mod()
    prep, x, y, stride = _case(dtype, 11)
    other = copy.copy(prep.packed)              # the same arrays, other weights
    other.values = prep.packed.values * 2
    run = lambda p, o, s=None: B.conv3x3_fwd_strided(prep.layer, p, x, o, stride, stream=s)
    note("scratch, two copies, %s" % np.dtype(dtype).name)
    z = torch.empty_like(y)
    run(prep.packed, y)
    run(other, z)
    want, want2 = y.clone(), z.clone()
    torch.cuda.synchronize()
    assert not torch.equal(want, want2)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(50):
        run(prep.packed, y, streams[0])
        run(other, z, streams[1])
    torch.cuda.synchronize()
    assert torch.equal(y, want) and torch.equal(z, want2)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_kept_scratch_and_capture(dtype):
    """The same bytes with scratch of the call's own, with one kept with the
    storage (full of other bytes), and from a graph between whose replays
    another layer runs."""
    _need_gpu()
    torch = torch_mod()
    prep, x, y, stride = _case(dtype, 21)
    prep2, x2, y2, _ = _case(dtype, 31)
    run = lambda: B.conv3x3_fwd_strided(prep.layer, prep.packed, x, y, stride)
    note("scratch, capture, %s" % np.dtype(dtype).name)
    run()
    want = y.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    for _ in range(3):
        y.zero_()
        B.conv3x3_fwd_strided(prep2.layer, prep2.packed, x2, y2, stride)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
    prep.packed.work.fill_(255)
    y.zero_()
    run()
    torch.cuda.synchronize()
    assert torch.equal(y, want)


def test_admm_target_and_iteration_take_different_scratch(monkeypatch):
    """target() on the next batch may run beside an iteration: host only, with
    the library's calls left out."""
    torch = torch_mod()
    used = []

    def fwd(x, w, y, bias=None, relu=False, stream=None, ws=None):
        used.append(ws.data_ptr())
        if len(used) == 2:
            raise StopIteration

    monkeypatch.setattr(B, "dense3x3_fwd", fwd)
    monkeypatch.setattr(B, "_scratch", lambda b, stream: torch.empty(b, dtype=torch.uint8), raising=False)
    st = B.AdmmLayer(torch.zeros(32, 16, 3, 3), torch.zeros(32), [23, 282], 200)
    x = torch.zeros(1, 16, 4, 4)
    t = st.target(x)
    with pytest.raises(StopIteration):
        st.iteration(x, t, 1e-3, 1.0)
    assert used[0] != used[1]


@pytest.mark.gpu
def test_admm_target_beside_an_iteration():
    _need_gpu()
    torch = torch_mod()
    wt = inputs.he_weights(41, 64, 64)
    st = B.AdmmLayer(dev(wt), dev(inputs.bias_vector(42, 64)), B.select_library(wt, 8), 2000)
    x = dev(inputs.normal_activations(43, (32, 64, 32, 32)))
    note("scratch, target beside an iteration")
    target = st.target(x)
    want = target.clone()
    st.iteration(x, target, 1e-2, 1e-3)
    st.w.mul_(3)                                # far from W0
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    outs = [torch.empty_like(target) for _ in range(20)]
    torch.cuda.synchronize()
    for out in outs:
        st.iteration(x, target, 1e-2, 1e-3, stream=s1)
        st.target(x, out=out, stream=s2)
    torch.cuda.synchronize()
    assert all(torch.equal(out, want) for out in outs)
