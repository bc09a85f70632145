"""Tensors packed back to back: the vector path takes any element alignment, and
the fused calls no longer need 16-byte aligned pointers.  Bit for bit against
the same run through the two separate kernels."""
import dataclasses
import gc
import os

import numpy as np
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


def _run(w, layouts, knob, step):
    """Two outer iterations of `step` with the library's knob set to 0 or unset."""
    from slowmo_inputs.gpu_problem import GpuProblem
    prob = GpuProblem(w, "cuda:0", param_layout=layouts[0], grad_layout=layouts[1])
    if knob:
        os.environ[knob] = "0"
    try:
        opt = PU.make_gpu(w, prob)
    finally:
        if knob:
            os.environ.pop(knob, None)
    for r in range(2):
        for k in range(w.tau):
            prob.fill_grads(0, r * w.tau + k)
            step(w, opt, prob.grads[0], k)
    st = PU.gpu_state(w, prob, opt, np.arange(w.d, dtype=np.int64))
    opt.close()
    return st


def _same(w, a, b):
    for key in ("x", "x0", "u") + (("h",) if w.policy != "reset" else ()) + \
            (("v",) if w.base == "adam" and w.policy != "reset" else ()):
        assert np.array_equal(a[key], b[key]), key


@pytest.mark.parametrize("base,grad_dtype,policy,layouts", [
    ("sgd_nesterov", "bf16", "maintain", ("flat", "flat")),
    ("adam", "bf16", "maintain", ("separate", "flat")),
    ("adam", "f32", "average", ("flat", "flat")),
    ("adam", "bf16", "average", ("flat", "separate")),
])
def test_fused_last_step_on_unaligned_pointers(base, grad_dtype, policy, layouts):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=3), tau=2)

    def step(w, opt, grads, k):
        if k == w.tau - 1:
            opt.local_outer_step(grads, w.lr)
        else:
            opt.local_step(grads, w.lr)

    _same(w, _run(w, layouts, None, step), _run(w, layouts, "SLOWMO_FUSE_LAST", step))


@pytest.mark.parametrize("base,grad_dtype", [("sgd_nesterov", "f32"), ("adam", "bf16")])
def test_fused_gossip_step_with_unaligned_gradients(base, grad_dtype):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy="maintain", m=5), tau=2)
    maps = ([1, 2, 3, 4, 0], [0, 0, 1, 1, 4])

    def step(w, opt, grads, k):
        opt.local_mix_step(grads, w.lr, maps[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)

    layouts = ("separate", "flat")
    _same(w, _run(w, layouts, None, step), _run(w, layouts, "SLOWMO_FUSE_MIX", step))
