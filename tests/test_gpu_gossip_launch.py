"""The mixing order of a gossip step travels in the kernel's arguments up to 64 workers and as
a table beyond, and one launch runs all connected groups of workers: both sides of the limit,
from one group to one pair of workers per group (64 of them)."""
import dataclasses

import numpy as np
import pytest

from slowmo_inputs import workloads as W

import parity_utils as PU

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused_mix", [False, True])
@pytest.mark.parametrize("m,mix", [(64, "expgraph"), (64, "random"), (65, "random"), (128, "expgraph")])
def test_limit_of_the_inline_order_every_element(m, mix, fused_mix):
    """128 workers on the exponential graph: hops 1 to 64, 1 to 64 groups; 64: 1 to 32."""
    from slowmo_inputs.gpu_problem import GpuProblem
    w = dataclasses.replace(W.ragged_mini(m=m, policy="maintain"), mix=mix, tau=7, rounds=1,
                            shapes=(("a", (300,)), ("b", (3,)), ("c", (1030,))))
    prob = GpuProblem(w, "cuda:0", grad_layout="separate")
    opt = PU.make_gpu(w, prob)
    PU.compare_run(w, prob, opt, np.arange(w.d, dtype=np.int64), w.rounds, bitwise_f32=True,
                   fused_mix=fused_mix)
    opt.close()
