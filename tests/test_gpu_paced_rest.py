"""Ordinary tiles that ride with a paced launch (taken, one per wave, by the workgroups that
have no piece in the last row) give the bits of the single-wave kernels."""
import gc

import numpy as np
import pytest

import parity_utils as PU
from test_gpu_paced import ROWS, SMALL, TILE, TWO_ROWS, _gossip, _groups, _workload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _free_gpu_memory():
    yield
    import torch
    gc.collect()
    torch.cuda.empty_cache()


# a full row and 172 pieces of the next one: what is left over rides by the library's rule
PART = (("a", (300 * TILE + 3,)), ("b", (128 * TILE + 5003,)), ("c", (2,)), ("d", (259,)))


@pytest.mark.parametrize("shapes,m,base,grad_dtype,policy,rest", [
    (PART, 8, "sgd_nesterov", "f32", "reset", None), (PART, 9, "adam", "bf16", "maintain", None),
    # forced: no piece at all for some XCDs; full rows, so every workgroup takes some
    (SMALL, 8, "adam", "f32", "reset", "1"), (TWO_ROWS, 8, "sgd_nesterov", "bf16", "maintain", "1"),
    (ROWS, 3, "sgd_nesterov", "f32", "maintain", "1"), (PART, 8, "adam", "bf16", "reset", "0")])
def test_rest_of_a_paced_launch(shapes, m, base, grad_dtype, policy, rest):
    w = _workload(shapes, m, base, grad_dtype, policy, tau=3)
    step = _gossip(w, [_groups(m), [0] * m, [int(v) for v in np.random.default_rng(m).integers(0, m, size=m)]])
    paced = None if shapes is PART else "2"
    PU.assert_same_bits(
        PU.run_library(w, ("arena", "flat"), step, SLOWMO_PACED=paced, SLOWMO_PACED_REST=rest),
        PU.run_library(w, ("arena", "flat"), step, SLOWMO_PACED="0"))
