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
