"""Teams, a wave per worker on every tile of a short list, against the walk from worker to worker
(SLOWMO_TEAM=0), bit for bit: tensors whose ends fall on every side of a tile's edge, worker counts
around one and two workers per wave, teams of all workers and of one connected group."""
import dataclasses
import gc

import numpy as np
import pytest

from slowmo_inputs import workloads as W

import parity_utils as PU

pytestmark = pytest.mark.gpu

# one lane alone, one lane and a few, a full tile less or more a few, two tiles
LENGTHS = list(range(1, 10)) + list(range(251, 262)) + [511, 512, 513, 515]
SHORT = tuple((f"t{j}", (n,)) for j, n in enumerate(LENGTHS))
LONGER = SHORT + (("long", (60_001,)),)      # beyond the line of the teams of one group


@pytest.fixture(autouse=True)
def _free_gpu_memory():
    yield
    import torch
    gc.collect()
    torch.cuda.empty_cache()


def _maps(m):
    cycle = [(i - 1) % m for i in range(m)]
    pairs = [i ^ 1 if i ^ 1 < m else i for i in range(m)]
    return [cycle, pairs, np.random.default_rng(m).integers(0, m, size=m).tolist(), [0] * m,
            list(range(m))]


def _gossip(w, fused):
    def step(opt, grads, k):
        peers = _maps(w.m)[k]
        if fused:
            opt.local_mix_step(grads, w.lr, peers)
        else:
            opt.local_step(grads, w.lr)
            opt.mix_step(peers)
        if k == w.tau - 1:
            opt.outer_step(w.lr)
    return step


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("m,shapes,base,grad_dtype,policy", [
    (2, LONGER, "sgd_nesterov", "f32", "reset"), (5, SHORT, "adam", "bf16", "maintain"),
    (16, SHORT, "sgd_nesterov", "bf16", "maintain"), (16, LONGER, "adam", "f32", "reset"),
    (17, LONGER, "sgd_nesterov", "f32", "reset"), (32, SHORT, "adam", "f32", "maintain"),
    (32, LONGER, "sgd_nesterov", "bf16", "average"), (33, SHORT, "sgd_nesterov", "f32", "reset")])
def test_gossip_by_teams(m, shapes, base, grad_dtype, policy, fused):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, m=m, policy=policy),
                            shapes=shapes, tau=5, rounds=2)
    for layouts in (("separate", "separate"), ("flat", "flat")) if not fused else (("separate", "flat"),):
        PU.assert_same_bits(PU.run_library(w, layouts, _gossip(w, fused)),
                            PU.run_library(w, layouts, _gossip(w, fused), SLOWMO_TEAM="0"))


# the accesses that the library would take on lists past the caches, and those on lists inside them
ACCESSES = pytest.mark.parametrize("nt", ["0", "1"])


@ACCESSES
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("m,base,grad_dtype", [(5, "adam", "bf16"), (17, "sgd_nesterov", "f32"),
                                               (32, "adam", "f32")])
def test_gossip_by_teams_streaming_or_not(m, base, grad_dtype, fused, nt):
    """One and two workers per wave; nothing kept, which a team would not take."""
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, m=m, policy="maintain"),
                            shapes=LONGER, tau=5, rounds=2)
    PU.assert_same_bits(
        PU.run_library(w, ("separate", "flat"), _gossip(w, fused), SLOWMO_LOCAL_NT=nt, SLOWMO_KEPT="0"),
        PU.run_library(w, ("separate", "flat"), _gossip(w, fused), SLOWMO_TEAM="0"))


def _outer(w, fused):
    def step(opt, grads, k):
        if fused and k == w.tau - 1:
            opt.local_outer_step(grads, w.lr)
        else:
            opt.local_step(grads, w.lr)
            if k == w.tau - 1:
                opt.outer_step(w.lr)
    return step


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("m,base,grad_dtype,policy,tau", [
    (3, "adam", "bf16", "average", 2), (4, "sgd_nesterov", "f32", "reset", 2),
    (5, "adam", "f32", "maintain", 1), (16, "sgd_nesterov", "bf16", "average", 2),
    (17, "adam", "f32", "average", 1), (31, "sgd_nesterov", "f32", "maintain", 2),
    (32, "adam", "f32", "average", 2), (32, "adam", "bf16", "reset", 1)])
def test_outer_step_by_teams(m, base, grad_dtype, policy, tau, fused):
    """Two workers per wave from 17 on; three rows of LDS per worker with Adam's averages (96 KiB
    with 32 workers)."""
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, m=m, policy=policy),
                            shapes=LONGER, tau=tau, rounds=2)
    for layouts in (("separate", "separate"), ("flat", "flat")):
        PU.assert_same_bits(PU.run_library(w, layouts, _outer(w, fused)),
                            PU.run_library(w, layouts, _outer(w, fused), SLOWMO_TEAM="0"))


@ACCESSES
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("m,base,grad_dtype,policy", [
    (5, "adam", "bf16", "maintain"), (17, "sgd_nesterov", "f32", "average"), (32, "adam", "f32", "average"),
    (32, "sgd_nesterov", "bf16", "reset")])
def test_outer_step_by_teams_streaming_or_not(m, base, grad_dtype, policy, fused, nt):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, m=m, policy=policy),
                            shapes=LONGER, tau=2, rounds=2)
    PU.assert_same_bits(
        PU.run_library(w, ("separate", "flat"), _outer(w, fused), SLOWMO_OUTER_NT=nt, SLOWMO_KEPT="0"),
        PU.run_library(w, ("separate", "flat"), _outer(w, fused), SLOWMO_TEAM="0"))


@pytest.mark.parametrize("tiles", [768, 769, 1024, 1025])
@pytest.mark.parametrize("policy", ["reset", "maintain"])
def test_both_sides_of_the_line_of_the_teams(tiles, policy):
    w = dataclasses.replace(W.ragged_mini(m=5, policy=policy), tau=2, rounds=2,
                            shapes=(("a", (256 * tiles - 300,)), ("b", (1,)),))
    PU.assert_same_bits(PU.run_library(w, ("separate", "flat"), _outer(w, True)),
                        PU.run_library(w, ("separate", "flat"), _outer(w, True), SLOWMO_TEAM="0"))
