"""Big tiles of 14 and 12 vectors per lane: the same bits as the ordinary tiles, with tensors
of exactly one tile, a few elements less or more, two tiles, and none."""
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


@pytest.mark.parametrize("vectors", [14, 12])
@pytest.mark.parametrize("base,grad_dtype,policy,tau,fused", [
    ("sgd_nesterov", "f32", "reset", 2, True), ("sgd_nesterov", "bf16", "reset", 1, True),
    ("adam", "bf16", "reset", 2, True), ("adam", "f32", "reset", 1, True),
    ("adam", "bf16", "reset", 1, True), ("sgd_nesterov", "f32", "maintain", 2, False)])
def test_smaller_big_tiles(base, grad_dtype, policy, tau, fused, vectors):
    tile = 4096 * vectors
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, policy=policy, m=5), tau=tau,
                            shapes=tuple((f"t{n}", (n,)) for n in (tile, tile + 5, 3, 2 * tile, tile - 1)))

    def step(opt, grads, k):
        if k < tau - 1 or not fused:
            opt.local_step(grads, w.lr)
        if k == tau - 1:
            opt.local_outer_step(grads, w.lr) if fused else opt.outer_step(w.lr)

    PU.assert_same_bits(*(PU.run_library(w, ("separate", "separate"), step, SLOWMO_BIG_TILES=b,
                                         SLOWMO_TEST_BIG_VPT=str(vectors)) for b in ("0", "1")))
