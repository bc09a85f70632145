"""Paced walks (one workgroup per CU, tiles of 16 384 elements, workgroups of an
XCD in step): bit for bit the results of the single-wave kernels."""
import dataclasses
import gc
import os

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


def _run(w, paced, grad_layout, step):
    """Two outer iterations with SLOWMO_PACED = `paced` (0: never, 2: wherever the
    kernels allow, also on lists too short for it to pay)."""
    from slowmo_inputs.gpu_problem import GpuProblem
    prob = GpuProblem(w, "cuda:0", grad_layout=grad_layout)
    os.environ["SLOWMO_PACED"] = paced
    try:
        opt = PU.make_gpu(w, prob)
    finally:
        os.environ.pop("SLOWMO_PACED", None)
    for r in range(2):
        for k in range(w.tau):
            prob.fill_grads(0, r * w.tau + k)
            step(w, opt, prob.grads[0], k)
    st = PU.gpu_state(w, prob, opt, np.arange(w.d, dtype=np.int64))
    opt.close()
    return st


def _same(w, a, b):
    keys = ("x", "x0", "u") + (("h",) if w.policy != "reset" else ())
    for key in keys + (("v",) if w.base == "adam" and w.policy != "reset" else ()):
        assert np.array_equal(a[key], b[key]), key


# below a tile, exactly one, one and a few, two and an odd rest, a tile that is not the first
SMALL = (("a", (TILE - 1,)), ("b", (TILE,)), ("c", (7,)), ("d", (TILE + 5,)), ("e", (2 * TILE + 4099,)))
# more than one tile per CU: full rows, in which the workgroups pace each other, and a part of one
ROWS = (("a", (300 * TILE + 3,)), ("b", (301 * TILE,)))


def _workload(shapes, m, base, grad_dtype, policy, tau):
    return dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=m),
                               shapes=shapes, tau=tau, rounds=2,
                               tensor_wd=tuple(1e-4 * (j % 3) for j in range(len(shapes))),
                               tensor_lr_scale=tuple((1.0, 0.5, 2.0)[j % 3] for j in range(len(shapes))))


@pytest.mark.parametrize("shapes,m,base,grad_dtype,policy", [
    (SMALL, 1, "sgd_nesterov", "f32", "reset"),
    (SMALL, 2, "adam", "f32", "maintain"),
    (SMALL, 8, "sgd_nesterov", "bf16", "maintain"),
    (SMALL, 17, "adam", "bf16", "reset"),
    (ROWS, 4, "sgd_nesterov", "f32", "maintain"),
    (ROWS, 3, "adam", "bf16", "maintain"),
])
def test_gossip_step(shapes, m, base, grad_dtype, policy):
    """Permutations (one cycle, several, fixed points) and random maps: senders with
    several receivers take the saved values, and with more of them than are kept
    workers are stepped twice."""
    w = _workload(shapes, m, base, grad_dtype, policy, tau=5)
    rng = np.random.default_rng(m)
    maps = [[(i - 1) % m for i in range(m)], [i ^ 1 if i ^ 1 < m else i for i in range(m)],
            [0] * m, [int(v) for v in rng.integers(0, m, size=m)],
            [int(v) for v in rng.integers(0, m, size=m)]]

    def step(w, opt, grads, k):
        opt.local_mix_step(grads, w.lr, maps[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)

    _same(w, _run(w, "2", "flat", step), _run(w, "0", "flat", step))
