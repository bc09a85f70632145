"""Tensors packed back to back: the vector path takes any element alignment, and
the fused calls no longer need 16-byte aligned pointers.  Bit for bit against
the same run through the two separate kernels."""
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


def _rounds(w):
    def step(opt, grads, k):
        if k == w.tau - 1:
            opt.local_outer_step(grads, w.lr)
        else:
            opt.local_step(grads, w.lr)
    return step


@pytest.mark.parametrize("base,grad_dtype,policy,layouts", [
    ("sgd_nesterov", "bf16", "maintain", ("flat", "flat")),
    ("adam", "bf16", "maintain", ("separate", "flat")),
    ("adam", "f32", "average", ("flat", "flat")),
    ("adam", "bf16", "average", ("flat", "separate")),
])
def test_fused_last_step_on_unaligned_pointers(base, grad_dtype, policy, layouts):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=3), tau=2)
    PU.assert_same_bits(PU.run_library(w, layouts, _rounds(w), SLOWMO_FUSE_LAST=None),
                        PU.run_library(w, layouts, _rounds(w), SLOWMO_FUSE_LAST="0"))


@pytest.mark.parametrize("base,grad_dtype,policy", [
    ("sgd_nesterov", "f32", "reset"), ("sgd_nesterov", "bf16", "reset"), ("adam", "bf16", "maintain"),
    ("adam", "f32", "reset")])
def test_fused_last_step_on_big_tiles_with_unaligned_gradients(base, grad_dtype, policy):
    """Big tiles ask for aligned replicas only: the tensors of 70 001 and 131 077 elements
    have one and two of them, with gradients at any element."""
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=3), tau=2)
    layouts = ("separate", "flat")
    PU.assert_same_bits(PU.run_library(w, layouts, _rounds(w), SLOWMO_BIG_TILES="1"),
                        PU.run_library(w, layouts, _rounds(w), SLOWMO_FUSE_LAST="0"))


@pytest.mark.parametrize("base,grad_dtype", [("sgd_nesterov", "f32"), ("adam", "bf16")])
def test_fused_gossip_step_with_unaligned_gradients(base, grad_dtype):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy="maintain", m=5), tau=2)
    maps = ([1, 2, 3, 4, 0], [0, 0, 1, 1, 4])

    def step(opt, grads, k):
        opt.local_mix_step(grads, w.lr, maps[k])
        if k == w.tau - 1:
            opt.outer_step(w.lr)

    layouts = ("separate", "flat")
    PU.assert_same_bits(PU.run_library(w, layouts, step, SLOWMO_FUSE_MIX=None),
                        PU.run_library(w, layouts, step, SLOWMO_FUSE_MIX="0"))
