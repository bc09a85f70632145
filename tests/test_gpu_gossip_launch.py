"""The mixing order of a gossip step travels in the kernel's arguments up to 32 workers and as
a table beyond, and one launch runs all connected groups of workers: both sides of the limit,
from one group to one pair of workers per group (64 of them)."""
import dataclasses

import numpy as np
import pytest

from slowmo_inputs import workloads as W

import parity_utils as PU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused_mix", [False, True])
@pytest.mark.parametrize("m,mix", [(32, "expgraph"), (32, "random"), (33, "random"), (64, "expgraph"), (64, "random"), (65, "random"), (128, "expgraph")])
def test_limit_of_the_inline_order_every_element(m, mix, fused_mix):
    """128 workers on the exponential graph: hops 1 to 64, 1 to 64 groups; 32: 1 to 16."""
    from slowmo_inputs.gpu_problem import GpuProblem
    w = dataclasses.replace(W.ragged_mini(m=m, policy="maintain"), mix=mix, tau=7, rounds=1,
                            shapes=(("a", (300,)), ("b", (3,)), ("c", (1030,))))
    prob = GpuProblem(w, "cuda:0", grad_layout="separate")
    opt = PU.make_gpu(w, prob)
    PU.compare_run(w, prob, opt, np.arange(w.d, dtype=np.int64), w.rounds, bitwise_f32=True,
                   fused_mix=fused_mix)
    opt.close()


@pytest.mark.parametrize("m", [3, 32, 33, 64, 65])
def test_debias_into_more_destinations_than_are_remembered(m):
    """The weights change with every gossip step and the destinations take turns, six sets of them;
    up to 32 workers only new destinations are uploaded."""
    import torch
    from slowmo_inputs.gpu_problem import GpuProblem
    w = dataclasses.replace(W.ragged_mini(m=m, policy="maintain"), mix="random", tau=14, rounds=1,
                            shapes=(("a", (300,)), ("b", (3,))))
    prob = GpuProblem(w, "cuda:0", grad_layout="separate")
    opt = PU.make_gpu(w, prob)
    sets = [[[torch.zeros_like(t) for t in p] for p in prob.params] for _ in range(6)]
    for k in range(w.tau):
        prob.fill_grads(0, k)
        opt.local_mix_step(prob.grads[0], w.lr, W.in_peers(w, k).tolist())
        z = sets[k % 6 if k != 1 else 0]
        opt.debias(z)
        weights = opt.pushsum_weights()
        assert len(set(weights)) > 1
        for i in range(m):
            for zt, xt in zip(z[i], prob.params[i], strict=True):
                # a division by an fp32 tensor rounds once, as the kernel's
                assert torch.equal(zt, xt / torch.tensor(weights[i], dtype=torch.float32, device=xt.device))
    opt.close()


@pytest.mark.parametrize("peers", [[1, 0, 3, 2], [0, 0, 2, 2], [1, 0, 3, 2, 4, 5, 6], [0, 1, 5, 3, 6, 2, 4, 0]])
def test_one_launch_for_all_groups(peers):
    """However few workers move: a second launch of the call would be refused."""
    from slowmo_inputs.gpu_problem import GpuProblem
    w = W.ragged_mini(m=len(peers), policy="maintain")
    prob = GpuProblem(w, "cuda:0")
    with PU.environment(SLOWMO_TEST_FAIL_LAUNCH="2"):
        opt = PU.make_gpu(w, prob)
    opt.mix_step(peers)
    opt.close()


@pytest.mark.parametrize("m", [4, 33])
@pytest.mark.parametrize("elements", [9000, 640_000 - 256, 640_001, 1_300_001])
def test_maps_that_move_few_workers(m, elements):
    """Walks and teams, on both sides of their lines for four and for two workers, against a walk per group."""
    rest = list(range(4, m))
    maps = [[3, 0, 1, 2] + rest, [1, 0, 2, 3] + rest, [1, 0, 3, 2] + rest, [0, 0, 0, 0] + rest]
    w = dataclasses.replace(W.ragged_mini(m=m, policy="maintain"), tau=4, rounds=2, shapes=(("a", (elements,)), ("b", (3,))))

    def step(opt, grads, k):
        opt.local_step(grads, w.lr)
        opt.mix_step(maps[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)

    PU.assert_same_bits(PU.run_library(w, ("separate", "flat"), step),
                        PU.run_library(w, ("separate", "flat"), step, SLOWMO_TEST_GROUP_LAUNCHES="1"))
