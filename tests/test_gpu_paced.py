"""Paced walks (one workgroup per CU, tiles of 16 384 elements, workgroups of an
XCD in step): bit for bit the results of the single-wave kernels."""
import dataclasses
import gc

import numpy as np
import pytest

from slowmo_inputs import workloads as W

import parity_utils as PU

pytestmark = pytest.mark.gpu

TILE = 16384


@pytest.fixture(autouse=True)
def _free_gpu_memory():
    yield
    import torch
    gc.collect()
    torch.cuda.empty_cache()


# below a tile, exactly one, one and a few, two and an odd rest, a tile that is not the first
SMALL = (("a", (TILE - 1,)), ("b", (TILE,)), ("c", (7,)), ("d", (TILE + 5,)), ("e", (2 * TILE + 4099,)))
# what the library paces by itself, from the worker counts below on: 300 pieces (256 of them paced), the
# rest with the short tensors more than a quarter of the list; 513 pieces (512 paced), cut inside the last
# tensor; 1100 (1024 paced)
ONE_ROW = (("a", (300 * TILE + 3,)),) + tuple((f"s{j}", (TILE - 1,)) for j in range(61))
TWO_ROWS = (("a", (200 * TILE + 1,)), ("b", (5,)), ("c", (150 * TILE,)), ("d", (163 * TILE + TILE - 1,)))
FOUR_ROWS = (("a", (1100 * TILE + 77,)),)
# more than one tile per CU: full rows, in which the workgroups pace each other, and a part of one
ROWS = (("a", (300 * TILE + 3,)), ("b", (301 * TILE,)))


def _workload(shapes, m, base, grad_dtype, policy, tau):
    return dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=m),
                               shapes=shapes, tau=tau, rounds=2,
                               tensor_wd=tuple(1e-4 * (j % 3) for j in range(len(shapes))),
                               tensor_lr_scale=tuple((1.0, 0.5, 2.0)[j % 3] for j in range(len(shapes))))


def _gossip(w, maps):
    def step(opt, grads, k):
        opt.local_mix_step(grads, w.lr, maps[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)
    return step


@pytest.mark.parametrize("shapes,m,base,grad_dtype,policy", [
    (SMALL, 1, "sgd_nesterov", "f32", "reset"),
    (SMALL, 2, "adam", "f32", "maintain"),
    (SMALL, 8, "sgd_nesterov", "bf16", "maintain"),
    (SMALL, 17, "adam", "bf16", "reset"),
    (ROWS, 4, "sgd_nesterov", "f32", "maintain"),
    (ROWS, 3, "adam", "bf16", "maintain"),
])
def test_gossip_step(shapes, m, base, grad_dtype, policy):
    """SLOWMO_PACED=2 (wherever the kernels allow, also on lists too short for it to pay)
    against 0 (never).  Permutations (one cycle, several, fixed points) and random maps:
    senders with several receivers take the saved values, and with more of them than are
    kept workers are stepped twice."""
    w = _workload(shapes, m, base, grad_dtype, policy, tau=5)
    rng = np.random.default_rng(m)
    maps = [[(i - 1) % m for i in range(m)], [i ^ 1 if i ^ 1 < m else i for i in range(m)],
            [0] * m, [int(v) for v in rng.integers(0, m, size=m)],
            [int(v) for v in rng.integers(0, m, size=m)]]
    step = _gossip(w, maps)
    PU.assert_same_bits(PU.run_library(w, ("separate", "flat"), step, SLOWMO_PACED="2"),
                        PU.run_library(w, ("separate", "flat"), step, SLOWMO_PACED="0"))


def _groups(*sizes):
    """Cycles of the given sizes side by side."""
    starts = np.cumsum((0,) + sizes[:-1])
    return [int(a + (i - 1) % n) for a, n in zip(starts, sizes) for i in range(n)]


@pytest.mark.parametrize("shapes,m,base,grad_dtype,policy,paced", [
    (ONE_ROW, 8, "adam", "bf16", "maintain", "2"),
    (ONE_ROW, 16, "sgd_nesterov", "f32", "reset", "2"),
    (TWO_ROWS, 9, "adam", "f32", "reset", "2"),
    (TWO_ROWS, 16, "sgd_nesterov", "bf16", "maintain", "2"),
    (ONE_ROW, 17, "adam", "bf16", "maintain", None),
    (ONE_ROW, 32, "sgd_nesterov", "f32", "reset", None),
    (TWO_ROWS, 17, "adam", "f32", "reset", None),
    (TWO_ROWS, 27, "sgd_nesterov", "bf16", "maintain", None),
    (FOUR_ROWS, 8, "adam", "f32", "maintain", None),
])
def test_gossip_steps_that_the_library_paces_by_itself(shapes, m, base, grad_dtype, policy, paced):
    """No variable set: whole rows of paced tiles, the pieces beyond them with the rest, and
    in one context maps that are paced (one cycle, a star, large groups) next to maps that
    are not (pairs).  Below the lines of the rule: all pieces paced, whatever the map."""
    maps = [_groups(m), _groups(*[2] * (m // 2) + [1] * (m % 2)), [0] * m,
            _groups(*[4] * (m // 4) + [1] * (m % 4)),
            [int(v) for v in np.random.default_rng(m).integers(0, m, size=m)]]
    w = _workload(shapes, m, base, grad_dtype, policy, tau=5)
    step = _gossip(w, maps)
    PU.assert_same_bits(PU.run_library(w, ("arena", "flat"), step, SLOWMO_PACED=paced),
                        PU.run_library(w, ("arena", "flat"), step, SLOWMO_PACED="0"))


@pytest.mark.parametrize("shapes,m,base,grad_dtype,launches", [
    (ONE_ROW, 16, "adam", "bf16", 1), (ONE_ROW, 17, "adam", "bf16", 2), (ONE_ROW, 32, "sgd_nesterov", "f32", 2),
    (TWO_ROWS, 16, "adam", "f32", 1), (TWO_ROWS, 17, "adam", "f32", 2), (TWO_ROWS, 26, "sgd_nesterov", "bf16", 1),
    (TWO_ROWS, 27, "sgd_nesterov", "bf16", 2), (FOUR_ROWS, 7, "adam", "f32", 1), (FOUR_ROWS, 8, "adam", "f32", 2)])
def test_what_the_library_paces_by_itself(shapes, m, base, grad_dtype, launches):
    """The rest of a paced list is a second launch here, which is made to fail."""
    import contextlib
    import paper_1910_00643_amd as P
    from slowmo_inputs.gpu_problem import GpuProblem
    w = _workload(shapes, m, base, grad_dtype, "maintain", tau=2)
    prob = GpuProblem(w, "cuda:0", param_layout="arena", grad_layout="flat")
    with PU.environment(SLOWMO_TEST_FAIL_LAUNCH="2"):
        opt = PU.make_gpu(w, prob)
    prob.fill_grads(0, 0)
    with pytest.raises(P.SlowMoError) if launches == 2 else contextlib.nullcontext():
        opt.local_mix_step(prob.grads[0], w.lr, _groups(m))
    opt.close()


def test_workgroups_that_stop_waiting_for_each_other():
    """With a limit of one poll almost every workgroup gives up its first wait and runs on
    out of step, in one launch after the other: the pace is a matter of speed only."""
    w = _workload(ROWS, 4, "sgd_nesterov", "f32", "maintain", tau=3)
    step = _gossip(w, [_groups(4), [0, 0, 0, 0], _groups(2, 2)])
    PU.assert_same_bits(
        PU.run_library(w, ("arena", "flat"), step, SLOWMO_PACED="2", SLOWMO_TEST_PACE_SPINS="1"),
        PU.run_library(w, ("arena", "flat"), step, SLOWMO_PACED="0"))
