"""Packing where the cursors of a filter's patterns pass from one 64-channel
step, and from one wave's quarter of the channels, to the next: one pattern in
every lane, every lane a pattern of its own, and channel counts on both sides
of a step and of a quarter; byte for byte against the oracle."""
import itertools

import numpy as np
import pytest

from synthetic import inputs
from gpu_cases import compare_prepared, gpu_prepare, note, torch_mod

pytestmark = pytest.mark.gpu

MASKS = [sum(1 << b for b in c) for c in itertools.combinations(range(9), 4)]     # all 126


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch_mod().cuda.is_available():
        pytest.skip("no HIP device")


@pytest.mark.parametrize("m", [1, 7, 126])
@pytest.mark.parametrize("cin", [1, 63, 65, 255, 257, 300, 1000])
def test_cursors(cin, m):
    for dtype, drop in ((np.float32, 0), (np.float16, 35)):
        wt = inputs.he_weights(cin + m, 9, cin, dtype)
        masks = np.array(sorted(MASKS[::len(MASKS) // m][:m]), dtype=np.uint16)
        keep = inputs.keep_after_drop(9 * cin, drop)
        note("pack cin %d m %d %s" % (cin, m, np.dtype(dtype).name))
        compare_prepared(gpu_prepare(wt, masks, keep), wt, masks, keep)
