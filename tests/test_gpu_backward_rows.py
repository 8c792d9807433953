"""The layer backward at slot counts around the 16-row halves and 32-row blocks
in which a wavefront gathers its slot rows and stores their input gradients,
and around the 128-row work items, against the CPU oracle (tolerances of
tests/test_gpu_backward.py)."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import announce, needs_gpu
from tests.test_gpu_backward import _compare, _counts, _gpu_backward

pytestmark = [pytest.mark.gpu, needs_gpu]

# slots of the experts 0, 1, ...; the rest choose the expert after them
EDGE_COUNTS = [0, 1, 4, 15, 16, 17, 31, 32, 33, 47, 48, 49, 127, 128, 129, 0, 257]


@pytest.mark.parametrize("dh,dff", [(128, 32), (128, 64), (128, 160), (64, 32), (64, 96)])
def test_edge_counts(dh, dff, oracle_instance):
    T, n_heads, Ne = sum(EDGE_COUNTS) + 3, 2, len(EDGE_COUNTS) + 1
    announce(f"backward rows d_h={dh} d_ff={dff}")
    shape = workloads.Shape(T, n_heads, dh, Ne, 1, dff, "bf16", backward=True)
    w = workloads.generate(shape, seed=11)
    rng = np.random.default_rng(13)
    first = np.repeat(np.arange(Ne), EDGE_COUNTS + [3]).astype(np.int32)
    idx = np.stack([rng.permutation(first) for _ in range(n_heads)], axis=1)[:, :, None]
    gate = (0.2 + 0.6 * rng.random((T, n_heads, 1))).astype(np.float32)
    got = _gpu_backward(w, idx, gate)
    want = oracle_instance.layer_backward(
        w.exact("X"), w.exact("W_router"), w.exact("W1"), w.exact("W3"), w.exact("W2"), idx,
        gate, w.exact("dY"))
    _compare(got, want, f"d_h={dh} d_ff={dff}", _counts(idx, Ne))
