"""The planner's row layout on the CPU, with the waves of its workgroup in several orders between the barriers: whatever it reads
and writes in LDS and in memory has to be ordered by a barrier, not by which wave happens to be ahead."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2403_07339_amd", "csrc")


def test_row_layout_does_not_depend_on_the_order_of_the_waves(tmp_path):
    text = open(os.path.join(CSRC, "plan.hip")).read()
    start = text.index("__device__ void rows_layout(")
    (tmp_path / "rows_layout.inc").write_text(text[start:text.index("\n}\n", start) + 3])
    exe = str(tmp_path / "rows_layout")
    for cmd in (["g++", "-O1", "-g", "-std=c++17", "-I", str(tmp_path), "-I", CSRC, "-I", "/opt/rocm/include", "-o", exe,
                 os.path.join(ROOT, "tests", "host", "rows_layout_driver.cpp")], [exe]):
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
        assert r.returncode == 0, r.stdout[-4000:]
    assert r.stdout.strip().endswith(" 0 failures"), r.stdout
