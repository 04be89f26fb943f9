"""Unwindowed intensities of few tasks with several 16-sample steps: the steps
of a task are spread over a workgroup's slots and summed at the end
(k_lag.hip).  Exact integers either way, so the outputs carry the one rounding
to FP32 of tests/test_gpu_lag.py."""
import pytest

from tests.test_gpu_lag import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ns", [16, 32, 64, 128])
@pytest.mark.parametrize("n_chan,n_pol,block,n_blk,pol_sum,keep", [
    (3, 1, 64, 1, False, 0),       # four steps, a slot each below 4 x 128
    (5, 2, 84, 1, True, 5),        # twelve steps, the last of each polarisation ragged
    (1, 1, 36 * 16, 2, False, 0),  # more steps than slots
    (700, 1, 48, 1, False, 9),     # one task a unit, more units than workgroups
    (1300, 1, 32, 1, False, 0),    # three tasks a unit in two rounds
])
def test_slots(n_ns, n_chan, n_pol, block, n_blk, pol_sum, keep):
    _check(n_ns, n_chan, n_pol, block, n_blk, pol_sum, keep)
