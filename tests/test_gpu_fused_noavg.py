"""Last local step and outer step without the average in one kernel, against the two kernels
(SLOWMO_FUSE_LAST=0), bit for bit, in each of its instances by accesses to memory."""
import dataclasses
import gc

import pytest

from slowmo_inputs import workloads as W

import parity_utils as PU
from test_gpu_teams import LONGER, SHORT, _outer

pytestmark = pytest.mark.gpu

STREAM = {"SLOWMO_LOCAL_NT": "1", "SLOWMO_OUTER_NT": "1"}
PLAIN = {"SLOWMO_LOCAL_NT": "0", "SLOWMO_OUTER_NT": "0"}


@pytest.fixture(autouse=True)
def _free_gpu_memory():
    yield
    import torch
    gc.collect()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("layout", ["separate", "flat"])
@pytest.mark.parametrize("m,shapes,base,grad_dtype,policy,tau,knobs", [
    (1, SHORT, "sgd_nesterov", "f32", "reset", 1, {}), (3, LONGER, "adam", "bf16", "reset", 1, PLAIN),
    (5, LONGER, "sgd_nesterov", "bf16", "maintain", 1, STREAM), (3, SHORT, "adam", "f32", "maintain", 2, PLAIN),
    (4, LONGER, "sgd_nesterov", "f32", "reset", 3, {"SLOWMO_LOCAL_NT": "0", "SLOWMO_OUTER_NT": "1"}),
    (2, LONGER, "adam", "bf16", "maintain", 2, {"SLOWMO_KEPT": "1", "SLOWMO_WRITE_THROUGH": "1", **STREAM}),
    (2, LONGER, "sgd_nesterov", "f32", "reset", 2, {"SLOWMO_KEPT": "1", "SLOWMO_WRITE_THROUGH": "1", **STREAM}),
    (3, LONGER, "adam", "f32", "maintain", 1, {"SLOWMO_WRITE_THROUGH": "1", **PLAIN}),
    (4, LONGER, "sgd_nesterov", "bf16", "reset", 1,
     {"SLOWMO_LOCAL_NT": "0", "SLOWMO_OUTER_NT": "1", "SLOWMO_WRITE_THROUGH": "1"}),
    (3, LONGER, "adam", "bf16", "reset", 2, {"SLOWMO_WRITE_THROUGH": "0", **STREAM})])
def test_fused_step_without_the_average(layout, m, shapes, base, grad_dtype, policy, tau, knobs):
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, m=m, policy=policy), tau=tau, rounds=2,
                            shapes=shapes, exact_average=False,
                            tensor_wd=tuple(1e-4 * (j % 3) for j in range(len(shapes))),
                            tensor_lr_scale=tuple((1.0, 0.5, 2.0)[j % 3] for j in range(len(shapes))))
    PU.assert_same_bits(PU.run_library(w, (layout, "flat"), _outer(w, True), **knobs),
                        PU.run_library(w, (layout, "flat"), _outer(w, True), SLOWMO_FUSE_LAST="0", **knobs))
