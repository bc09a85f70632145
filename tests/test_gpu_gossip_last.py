"""Fused gossip step under "reset": the last step of an outer iteration does not store the buffers, also
where it is the first one; teams, walk and paced walk against the separate calls, bit for bit."""
import dataclasses
import gc

import pytest

from slowmo_inputs import workloads as W

import parity_utils as PU
from test_gpu_paced import ROWS
from test_gpu_teams import LONGER, _gossip

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _free_gpu_memory():
    yield
    import torch
    gc.collect()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("tau", [1, 2])
@pytest.mark.parametrize("m,shapes,base,grad_dtype,knobs", [
    (17, LONGER, "adam", "bf16", {}), (5, LONGER, "sgd_nesterov", "f32", {"SLOWMO_TEAM": "0"}),
    (3, LONGER, "adam", "f32", {"SLOWMO_TEAM": "0", "SLOWMO_KEPT": "1"}),
    (3, ROWS, "sgd_nesterov", "bf16", {"SLOWMO_PACED": "2", "SLOWMO_PACED_REST": "1"})])
def test_last_step_before_a_reset(m, shapes, base, grad_dtype, knobs, tau):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, m=m, policy="reset"), shapes=shapes,
                            tau=tau, rounds=2)
    PU.assert_same_bits(PU.run_library(w, ("separate", "flat"), _gossip(w, True), **knobs),
                        PU.run_library(w, ("separate", "flat"), _gossip(w, False)))
