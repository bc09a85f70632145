"""The benchmark counts the bytes of big tiles by the library's own rules: both are asked for the
same lists; and it runs, and counts, one kernel where the library has one."""
import dataclasses
import os
import random
import subprocess
import types

import pytest

import bench
from slowmo_inputs import shapes, workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1910_00643_amd", "csrc")


def test_rules_agree(tmp_path):
    exe = str(tmp_path / "plan_big")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, "-o", exe,
                    os.path.join(ROOT, "tests", "plan_big_driver.cpp"),
                    os.path.join(CSRC, "slowmo_plan.cpp")], check=True)
    rng = random.Random(5)
    lists = [shapes.numels(s()) for s in (shapes.ragged_mini, shapes.resnet18, shapes.resnet50,
                                          shapes.transformer_big)]
    for _ in range(2000):
        n = rng.choice([1, 2, 5, 40])
        lists.append([int(10 ** rng.uniform(5, 8) / n) for _ in range(n)])
    lists = [(rng.choice([256, 256, 304, 104]), x) for x in lists]
    text = "".join(f"{cus} {len(x)} {' '.join(map(str, x))}\n" for cus, x in lists)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
    chosen = set()
    for (cus, x), got in zip(lists, out):
        chosen.add(int(got))
        assert bench.big_tile(types.SimpleNamespace(numel=x), cus) == 4096 * int(got), (cus, x)
    assert chosen == {0, 12, 14, 16}
    rules = iter(out[len(lists):])
    for policy in ("reset", "maintain", "average"):
        for m in (7, 8, 15, 16, 32):
            w = types.SimpleNamespace(numel=[1 << 24], policy=policy, m=m, exact_average=True)
            assert f"{bench.big_elements(w, True) > 0:d} {bench.big_elements(w, False) > 0:d}" == next(rules)


@pytest.mark.parametrize("average", [True, False])
@pytest.mark.parametrize("policy", ["reset", "maintain"])
@pytest.mark.parametrize("base,grad_dtype", [("sgd_nesterov", "f32"), ("adam", "bf16")])
@pytest.mark.parametrize("tau", [1, 3])
def test_fused_last_step_without_the_average(base, grad_dtype, policy, tau, average):
    """Every replica read and written once less than in the two kernels, with the average and without."""
    w = dataclasses.replace(W.ragged_mini(base=base, grad_dtype=grad_dtype, m=5, policy=policy), tau=tau,
                            exact_average=average)
    assert bench.fusable(w)
    assert bench.round_bytes(w) - bench.round_bytes(w, fused=True) == 8 * w.m * w.d
