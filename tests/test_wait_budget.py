"""The bounded wait for hidden vectors in the single-kernel layer (csrc/oea_wait.h), on the CPU: all staging steps of a
wavefront share one budget, and a step behind one that gave up does not wait again."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_02237_amd", "csrc")


def test_one_budget_for_all_steps(tmp_path):
    exe = str(tmp_path / "wait_budget")
    subprocess.check_call(["g++", "-O1", "-Wall", "-std=c++17", "-D__host__=", "-D__device__=", "-I", CSRC, "-o", exe,
                           os.path.join(ROOT, "tests", "wait_budget_main.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "wait budget: ok" in r.stdout, r.stdout


def test_the_layer_draws_its_budget_once():
    """The budget is made ahead of the staging loop, and nothing in the loop counts polls of its own."""
    text = open(os.path.join(CSRC, "oea_fused.hip")).read()
    begin = text.index("auto mid_b = [&]")
    body = text[begin:text.index("OEA_TL(12);", begin)]
    assert body.index("WaitBudget") < body.index("for (int base = 0;")
    loop = body[body.index("for (int base = 0;"):]
    assert "WaitBudget" not in loop and "budget.again()" in loop and not re.search(r"spins\s*=\s*0", loop)
