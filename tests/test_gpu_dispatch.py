"""GPU parity at the sizes where the launch rules change kernel forms: the smallest calls that reach
each form, with remainders on both axes, against the fp64 oracle (bounds as in the parity tests)."""
import pytest
import torch

from test_gpu_parity_small import _run_pair

pytestmark = pytest.mark.gpu

# fp32: 1, 2 or 4 parts per tile, chosen by the number of workgroups.  The comment gives the parts of the
# (forward, backward).
F32_PARTS = [
    (130, 130, 150, 150, False),   # (2, 1)
    (260, 130, 150, 77, False),    # (1, 1), grouped heads
    (40, 20, 130, 161, False),     # (4, 4), grouped heads
    (40, 40, 130, 161, False),     # (4, 2)
    (520, 520, 130, 130, True),    # (2, 2): causal, 64-row blocks
    (130, 65, 33, 33, True),       # (2, 4): one row past a block
]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", F32_PARTS)
def test_f32_parts(shape, d):
    h_q, h_kv, s_q, s_k, causal = shape
    _run_pair(torch.float32, h_q, h_kv, s_q, s_k, d, causal)
