"""GPU: the matrix-core broad phase (from 1,024 link blocks on) where its
survivors overflow the list and the direct test takes over: 48 joints whose
links all reach each other, against the FP64 oracle."""
import numpy as np
import pytest

from paper_2603_05493_amd import synth
from tests import test_gpu_fused_limits as limits

pytestmark = pytest.mark.gpu


def _balled():
    rb = synth.random_tree(48, 2, seed=13)
    rb.fixed_p = synth._f32(np.asarray(rb.fixed_p) * 0.02)
    return rb


@pytest.mark.parametrize("B", [1, 67])
def test_list_overflow(oracle, B):
    limits.test_fused_iteration_at_table_limits(oracle, "balled49", _balled, B)
