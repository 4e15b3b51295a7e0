"""Kernels whose waves share LDS, run on the CPU under wave orders a GPU shows
only now and then (tests/emulate): a wave held back at each barrier it has been
let through, a wave ahead of all others.  A read or write that no barrier
separates from another wave's makes waves meet at different barriers or end
with other results."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EMU = os.path.join(ROOT, "tests", "emulate")


def _run(name: str, kernels: str, out: str) -> str:
    src = os.path.join(ROOT, "paper_2609_35587_amd", "csrc", kernels)
    exe = os.path.join(out, name)
    subprocess.run(["g++", "-std=c++20", "-O1", "-Wno-unknown-pragmas", "-Wno-attributes", "-isystem", EMU,
                    f'-DKERNELS="{src}"', os.path.join(EMU, name + ".cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    return r.stdout


def test_topk_waves_agree_whatever_their_order(tmp_path):
    assert _run("topk", "select.hip", str(tmp_path)).strip().endswith("topk ok")
