"""How a sweep over the tiles goes through the caches (streaming or plain accesses, tiles
that are kept in the last-level cache, the direction of the sweep) changes no bit of any
result.  By itself the library chooses by sizes far above these."""
import dataclasses
import gc

import pytest

from slowmo_inputs import workloads as W

import parity_utils as PU

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _free_gpu_memory():
    yield
    import torch
    gc.collect()
    torch.cuda.empty_cache()


# kept tiles come in units of 16 384 elements: one short of a unit, one, a few more, some
LENGTHS = (16383, 16384, 16387, 3, 49152, 1, 70001, 257)
MAPS = ([1, 2, 0], [0, 0, 1], [2, 0, 1])
STREAMING = {"SLOWMO_LOCAL_NT": "1", "SLOWMO_OUTER_NT": "1", "SLOWMO_WRITE_THROUGH": "0",
             "SLOWMO_KEPT": "0", "SLOWMO_TURN": "0"}


def _separate(w):
    def step(opt, grads, k):
        opt.local_step(grads, w.lr)
        if k == w.tau - 1:
            opt.outer_step(w.lr)
    return step


def _fused(w):
    def step(opt, grads, k):
        if k == w.tau - 1:
            opt.local_outer_step(grads, w.lr)
        else:
            opt.local_step(grads, w.lr)
    return step


def _gossip(w):
    def step(opt, grads, k):
        opt.local_mix_step(grads, w.lr, MAPS[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)
    return step


# the walks from worker to worker, and teams where the library takes them on lists of this length
@pytest.mark.parametrize("team", ["0", None])
@pytest.mark.parametrize("layout", ["arena", "flat"])
@pytest.mark.parametrize("base,grad_dtype,policy,calls,average", [
    ("sgd_nesterov", "f32", "reset", _fused, True), ("sgd_nesterov", "bf16", "maintain", _separate, True),
    ("adam", "bf16", "maintain", _fused, True), ("adam", "f32", "average", _separate, True),
    ("sgd_nesterov", "f32", "maintain", _separate, False), ("adam", "bf16", "reset", _gossip, True)])
def test_accesses_and_directions(base, grad_dtype, policy, calls, average, layout, team):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=3), tau=3,
                            exact_average=average,
                            shapes=tuple((f"t{n}", (n,)) for n in LENGTHS))
    want = PU.run_library(w, (layout, "padded"), calls(w), SLOWMO_TEAM="0", **STREAMING)
    for other in ({"SLOWMO_LOCAL_NT": "0"}, {"SLOWMO_LOCAL_NT": "0", "SLOWMO_OUTER_NT": "0"}, {"SLOWMO_LOCAL_NT": "0", "SLOWMO_WRITE_THROUGH": "1"},
                  {"SLOWMO_WRITE_THROUGH": "1", "SLOWMO_KEPT": "1"},
                  {"SLOWMO_WRITE_THROUGH": "1", "SLOWMO_KEPT": "1000"},
                  # whole workers kept, and a part of the first one: where big tiles are in use
                  {"SLOWMO_WRITE_THROUGH": "1", "SLOWMO_KEPT": "3", "SLOWMO_BIG_TILES": "1"},
                  {"SLOWMO_WRITE_THROUGH": "1", "SLOWMO_KEPT": "1", "SLOWMO_BIG_TILES": "1"}):
        PU.assert_same_bits(want, PU.run_library(w, (layout, "padded"), calls(w),
                                                 **{**STREAMING, "SLOWMO_TURN": "1", "SLOWMO_TEAM": team, **other}))


def test_debias_of_a_list_that_stays_in_the_caches():
    import torch
    from slowmo_inputs.gpu_problem import GpuProblem
    w = dataclasses.replace(W.ragged_mini(m=3, policy="maintain"), tau=3,
                            shapes=tuple((f"t{n}", (n,)) for n in LENGTHS))
    prob = GpuProblem(w, "cuda:0", param_layout="flat", grad_layout="flat")
    with PU.environment(SLOWMO_LOCAL_NT="0"):
        opt = PU.make_gpu(w, prob)
    prob.fill_grads(0, 0)
    opt.local_mix_step(prob.grads[0], w.lr, MAPS[1])
    z = [[torch.full((n,), 7.0, device="cuda:0") for n in LENGTHS] for _ in range(w.m)]
    opt.debias(z)
    weights = opt.pushsum_weights()
    for i in range(w.m):
        for x, t in zip(prob.params[i], z[i], strict=True):
            assert torch.equal(t, x / torch.tensor(weights[i], device="cuda:0"))
    opt.close()


KEPT = {"SLOWMO_LOCAL_NT": "1", "SLOWMO_OUTER_NT": "1", "SLOWMO_WRITE_THROUGH": "1", "SLOWMO_TURN": "1"}


@pytest.mark.parametrize("megabytes", ["1", "1000"])
@pytest.mark.parametrize("layout", ["arena", "flat"])
def test_debias_of_kept_tiles(layout, megabytes):
    """A part of the units and all of them: z = x / w in every element."""
    import torch
    from slowmo_inputs.gpu_problem import GpuProblem
    w = dataclasses.replace(W.ragged_mini(m=3, policy="maintain"), tau=3,
                            shapes=tuple((f"t{n}", (n,)) for n in LENGTHS))
    prob = GpuProblem(w, "cuda:0", param_layout=layout, grad_layout="flat")
    with PU.environment(SLOWMO_KEPT=megabytes, **KEPT):
        opt = PU.make_gpu(w, prob)
    prob.fill_grads(0, 0)
    opt.local_mix_step(prob.grads[0], w.lr, MAPS[1])
    z = [[torch.full((n,), 7.0, device="cuda:0") for n in LENGTHS] for _ in range(w.m)]
    opt.debias(z)
    weights = opt.pushsum_weights()
    assert len(set(weights)) > 1
    for i in range(w.m):
        for x, t in zip(prob.params[i], z[i], strict=True):
            assert torch.equal(t, x / torch.tensor(weights[i], device="cuda:0"))
    opt.close()


@pytest.mark.parametrize("layout", ["arena", "flat"])
@pytest.mark.parametrize("base,grad_dtype,average", [("sgd_nesterov", "f32", True), ("adam", "bf16", False)])
def test_gossip_kernel_on_kept_tiles(base, grad_dtype, average, layout):
    """The gossip step by itself reads and writes kept tiles like the others."""
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy="maintain", m=3), tau=3,
                            exact_average=average, shapes=tuple((f"t{n}", (n,)) for n in LENGTHS))

    def step(opt, grads, k):
        opt.local_step(grads, w.lr)
        opt.mix_step(MAPS[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)

    PU.assert_same_bits(PU.run_library(w, (layout, "padded"), step, **STREAMING),
                        PU.run_library(w, (layout, "padded"), step, SLOWMO_KEPT="1", **KEPT))


@pytest.mark.parametrize("policy", ["reset", "maintain"])
@pytest.mark.parametrize("calls", [_separate, _fused, _gossip])
def test_one_step_rounds_by_the_rule(calls, policy):
    """tau = 1, 36 and 50 MB with 11 workers: each call pattern has lines of its own there, and
    an outer step goes by the step before it."""
    maps = [(i + 3) % 11 for i in range(11)]

    def gossip(w):
        def step(opt, grads, k):
            opt.local_mix_step(grads, w.lr, maps)
            opt.outer_step(w.lr)
        return step

    for elements in (270_001, 380_003):
        w = dataclasses.replace(W.ragged_mini(policy=policy, m=11), tau=1,
                                shapes=(("a", (elements,)), ("b", (16387,)), ("c", (3,))))
        step = gossip(w) if calls is _gossip else calls(w)
        PU.assert_same_bits(PU.run_library(w, ("arena", "flat"), step, **STREAMING),
                            PU.run_library(w, ("arena", "flat"), step))
