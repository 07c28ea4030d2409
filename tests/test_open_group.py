"""A float4 group that the settling pass looks up (csrc/qa_open_group.h, compiled for the CPU) may be the last of a row
whose length is not a multiple of 4: nothing beyond the row's last component belongs to the call."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_listed_groups_are_read_up_to_the_end_of_the_row_only(tmp_path):
    """Every length around 4 .. 256, the page behind the row unreadable."""
    exe = str(tmp_path / "open_group")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I" + os.path.join(ROOT, "paper_2208_05631_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "open_group.cpp"), "-o", exe], check=True)
    done = subprocess.run([exe], capture_output=True, text=True)
    assert done.returncode == 0, (done.returncode, done.stdout)
