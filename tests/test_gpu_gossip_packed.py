"""Fused gossip step on replicas packed back to back (not 16-byte aligned), in each of its three kernels,
against the two separate calls, bit for bit."""
import dataclasses
import gc

import pytest

from slowmo_inputs import workloads as W

import parity_utils as PU
from test_gpu_paced import ROWS, SMALL, TWO_ROWS
from test_gpu_teams import LONGER, SHORT, _gossip

pytestmark = pytest.mark.gpu

WALK = (("w", (700_001,)),) + LONGER      # past the 65 536 waves of the teams from 24 workers on


@pytest.fixture(autouse=True)
def _free_gpu_memory():
    yield
    import torch
    gc.collect()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("shapes,m,base,grad_dtype,policy,knobs", [
    (SHORT, 1, "sgd_nesterov", "f32", "maintain", {}), (SHORT, 4, "adam", "bf16", "maintain", {}),
    (LONGER, 17, "sgd_nesterov", "f32", "reset", {}), (SHORT, 33, "adam", "f32", "maintain", {}),
    (WALK, 24, "sgd_nesterov", "bf16", "maintain", {}), (LONGER, 3, "adam", "f32", "reset", {"SLOWMO_TEAM": "0"}),
    (WALK, 5, "sgd_nesterov", "f32", "maintain", {"SLOWMO_TEAM": "0", "SLOWMO_KEPT": "10"}),
    (SMALL, 8, "adam", "bf16", "maintain", {"SLOWMO_PACED": "2"}),
    (ROWS, 8, "sgd_nesterov", "f32", "reset", {"SLOWMO_PACED": "2"}),
    (ROWS, 3, "sgd_nesterov", "bf16", "maintain", {"SLOWMO_PACED": "2", "SLOWMO_PACED_REST": "1"})])
def test_one_kernel_on_packed_replicas(shapes, m, base, grad_dtype, policy, knobs):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, m=m, policy=policy),
                            shapes=(("first", (3,)),) + shapes, tau=5, rounds=2)
    PU.assert_same_bits(PU.run_library(w, ("flat", "flat"), _gossip(w, True), **knobs),
                        PU.run_library(w, ("flat", "flat"), _gossip(w, False)))


@pytest.mark.parametrize("layout,m", [("flat", 17), ("flat", 18), ("arena", 21), ("arena", 24)])
def test_both_sides_of_the_line_of_the_paced_walk(layout, m):
    """513 pieces, 512 of them paced, cut inside the last tensor: 101 MB that a step reads of each worker."""
    w = dataclasses.replace(W.ragged_mini(m=m), shapes=TWO_ROWS, tau=3, rounds=2)
    PU.assert_same_bits(PU.run_library(w, (layout, "flat"), _gossip(w, True)),
                        PU.run_library(w, (layout, "flat"), _gossip(w, True), SLOWMO_PACED="0"))


@pytest.mark.parametrize("m", [2, 3, 4, 5])
@pytest.mark.parametrize("peers", [[1, 0, 3, 2, 4], [0, 0, 1, 1, 0], [1, 1, 1, 1, 1]])
def test_one_launch_whatever_the_map(m, peers):
    """A second launch of the call would be refused."""
    from slowmo_inputs.gpu_problem import GpuProblem
    w = W.ragged_mini(m=m, policy="maintain")
    prob = GpuProblem(w, "cuda:0", param_layout="flat", grad_layout="flat")
    with PU.environment(SLOWMO_TEST_FAIL_LAUNCH="2"):
        opt = PU.make_gpu(w, prob)
    prob.fill_grads(0, 0)
    opt.local_mix_step(prob.grads[0], w.lr, [j % m for j in peers[:m]])
    opt.close()
