"""The end of a tensor: the last lane of a tile takes its vector at the last four
elements, so it shares some with its neighbour, and a tile of fewer than four goes by
single elements.  Every element evolves by itself, so lists of short tensors give bit for
bit what the same elements give as one tensor."""
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


# one lane alone, one lane and a few, a full tile less or more a few, two tiles
LENGTHS = list(range(1, 10)) + list(range(251, 262)) + [511, 512, 513, 515]
MAPS = ([1, 2, 3, 4, 0], [0, 0, 1, 1, 4], [3, 3, 3, 3, 3])


def _last(w):
    def step(opt, grads, k):
        if k == w.tau - 1:
            opt.local_outer_step(grads, w.lr)
        else:
            opt.local_step(grads, w.lr)
    return step


def _outer(w):
    def step(opt, grads, k):
        opt.local_step(grads, w.lr)
        if k == w.tau - 1:
            opt.outer_step(w.lr)
    return step


def _gossip(w):
    def step(opt, grads, k):
        opt.local_mix_step(grads, w.lr, MAPS[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)
    return step


def _gossip_separate(w):
    def step(opt, grads, k):
        opt.local_step(grads, w.lr)
        opt.mix_step(MAPS[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)
    return step


@pytest.mark.parametrize("layouts", [("flat", "flat"), ("arena", "padded"), ("arena", "flat")])
@pytest.mark.parametrize("base,grad_dtype,policy,calls,average", [
    ("sgd_nesterov", "f32", "reset", _last, True), ("adam", "bf16", "maintain", _last, True),
    ("sgd_nesterov", "bf16", "average", _last, True), ("adam", "f32", "average", _outer, True),
    ("sgd_nesterov", "f32", "maintain", _gossip, True), ("adam", "bf16", "maintain", _gossip, True),
    ("sgd_nesterov", "bf16", "maintain", _gossip_separate, True),
    ("adam", "bf16", "maintain", _outer, False)])
def test_short_tensors_equal_the_same_elements_in_one(base, grad_dtype, policy, calls, average, layouts):
    import torch
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=5), tau=3,
                            exact_average=average)
    many = dataclasses.replace(w, shapes=tuple((f"t{n}", (n,)) for n in LENGTHS))
    one = dataclasses.replace(w, shapes=(("all", (sum(LENGTHS),)),))
    a = PU.run_library(many, layouts, calls(w))
    b = PU.run_library(one, ("separate", "separate"), calls(w))
    assert a.keys() == b.keys()
    for key in a:
        per = len(LENGTHS)
        joined = [torch.cat([t.reshape(-1) for t in a[key][i:i + per]]) for i in range(0, len(a[key]), per)]
        PU.assert_same_bits({key: joined}, {key: [t.reshape(-1) for t in b[key]]})


@pytest.mark.parametrize("layout", ["flat", "arena"])
def test_debias_of_short_tensors(layout):
    import torch
    from slowmo_inputs.gpu_problem import GpuProblem
    w = dataclasses.replace(W.ragged_mini(m=5, policy="maintain"), tau=3,
                            shapes=tuple((f"t{n}", (n,)) for n in LENGTHS))
    prob = GpuProblem(w, "cuda:0", param_layout=layout, grad_layout="flat")
    opt = PU.make_gpu(w, prob)
    prob.fill_grads(0, 0)
    opt.local_mix_step(prob.grads[0], w.lr, MAPS[1])
    stores = [torch.full((sum(LENGTHS),), 7.0, device="cuda:0") for _ in range(w.m)]
    z = [list(s.split(LENGTHS)) for s in stores]
    opt.debias(z)
    weights = opt.pushsum_weights()
    assert min(weights) != max(weights)
    for i in range(w.m):
        for x, t in zip(prob.params[i], z[i]):
            assert torch.equal(t, x / torch.tensor(weights[i], device="cuda:0"))
    opt.close()


@pytest.mark.parametrize("layout", ["arena", "flat"])
@pytest.mark.parametrize("base,grad_dtype,policy,average", [
    ("sgd_nesterov", "f32", "reset", True), ("sgd_nesterov", "bf16", "maintain", False),
    ("adam", "bf16", "maintain", True), ("adam", "f32", "maintain", False)])
def test_stores_that_are_written_through(base, grad_dtype, policy, average, layout):
    """By itself the library writes through only on lists larger than these."""
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=3), tau=3,
                            exact_average=average)
    w = dataclasses.replace(w, shapes=w.shapes + tuple((f"t{n}", (n,)) for n in LENGTHS))
    PU.assert_same_bits(*(PU.run_library(w, (layout, "padded"), _outer(w), SLOWMO_WRITE_THROUGH=v)
                          for v in ("1", "0")))
