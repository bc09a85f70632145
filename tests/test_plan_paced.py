"""The mixing orders of the paced gossip kernel, replayed in place on the CPU."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_orders_for_the_paced_walk(tmp_path):
    exe = str(tmp_path / "plan_paced")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", os.path.join(HERE, "plan_paced_driver.cpp"),
                    os.path.join(HERE, "..", "paper_1910_00643_amd", "csrc", "slowmo_plan.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr
