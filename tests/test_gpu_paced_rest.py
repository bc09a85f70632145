"""Ordinary tiles that ride with a paced launch (taken, one per wave, by the workgroups that
have no piece in the last row) give the bits of the single-wave kernels."""
import gc

import numpy as np
import pytest

import parity_utils as PU
from test_gpu_paced import ROWS, SMALL, TILE, TWO_ROWS, _gossip, _groups, _workload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _free_gpu_memory():
    yield
    import torch
    gc.collect()
    torch.cuda.empty_cache()


# a full row and 172 pieces of the next one: what is left over rides by the library's rule
PART = (("a", (300 * TILE + 3,)), ("b", (128 * TILE + 5003,)), ("c", (2,)), ("d", (259,)))
# 31 of the 32 CUs of each XCD have a piece in the last row, the waves of the others six tiles each
LAST_CU = (("a", (504 * TILE,)), ("b", (63 * 256,)), ("c", (62 * 256 + 77,))) + tuple(
    (f"s{j}", (64 * 256 - 1 - j,)) for j in range(4))


@pytest.mark.parametrize("shapes,m,base,grad_dtype,policy,rest", [
    (PART, 8, "sgd_nesterov", "f32", "reset", None), (PART, 9, "adam", "bf16", "maintain", None),
    (PART, 17, "sgd_nesterov", "f32", "reset", None), (LAST_CU, 18, "adam", "bf16", "maintain", None),
    (LAST_CU, 8, "adam", "f32", "maintain", None), (LAST_CU, 8, "sgd_nesterov", "bf16", "reset", "0"),
    # forced: no piece at all for some XCDs; full rows, so every workgroup takes some
    (SMALL, 8, "adam", "f32", "reset", "1"), (TWO_ROWS, 8, "sgd_nesterov", "bf16", "maintain", "1"),
    (ROWS, 3, "sgd_nesterov", "f32", "maintain", "1"), (PART, 8, "adam", "bf16", "reset", "0")])
def test_rest_of_a_paced_launch(shapes, m, base, grad_dtype, policy, rest):
    w = _workload(shapes, m, base, grad_dtype, policy, tau=3)
    step = _gossip(w, [_groups(m), [0] * m, [int(v) for v in np.random.default_rng(m).integers(0, m, size=m)]])
    # (by the library's own rule from 17 workers on)
    paced = None if m >= 17 else "2"
    PU.assert_same_bits(
        PU.run_library(w, ("arena", "flat"), step, SLOWMO_PACED=paced, SLOWMO_PACED_REST=rest),
        PU.run_library(w, ("arena", "flat"), step, SLOWMO_PACED="0"))


@pytest.mark.parametrize("m", [17, 32])
@pytest.mark.parametrize("shapes", [PART, LAST_CU])
@pytest.mark.parametrize("rest,launches", [(None, 1), ("1", 1), ("0", 2)])
def test_riding_tiles_take_no_launch(shapes, rest, launches, m):
    """By the library's rule the step is one launch; a second one, made to fail, comes only where
    the tiles are launched by themselves."""
    import paper_1910_00643_amd as P
    from slowmo_inputs.gpu_problem import GpuProblem
    w = _workload(shapes, m, "sgd_nesterov", "f32", "reset", tau=3)
    prob = GpuProblem(w, "cuda:0", param_layout="arena", grad_layout="flat")
    with PU.environment(SLOWMO_PACED_REST=rest, SLOWMO_TEST_FAIL_LAUNCH="2"):
        opt = PU.make_gpu(w, prob)
    prob.fill_grads(0, 0)
    if launches == 1:
        opt.local_mix_step(prob.grads[0], w.lr, _groups(m))
    else:
        with pytest.raises(P.SlowMoError):
            opt.local_mix_step(prob.grads[0], w.lr, _groups(m))
    opt.close()
