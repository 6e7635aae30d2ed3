"""The session kernel's commit (counters, page tables, free list) on the host:
it is done once per launch, by the workgroup that is the last to have read
the old counters, and leaves nothing behind for the next launch.  A wait with
a time limit would not do: when it ran out, the count of workgroups that had
read would stay behind, the next launch would commit before its own
workgroups had read, and they would see the session one token further on.
"""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_10582_amd", "csrc")


def test_every_launch_commits_once_after_all_reads(tmp_path):
    exe = tmp_path / "arrive"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, os.path.join(ROOT, "tests", "arrive_threads.cpp"),
                    "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_no_workgroup_of_the_session_kernel_waits_for_another():
    src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "md_rows.hip")).read())
    for word in ("memrealtime", "s_sleep", "kWordWaitTicks", "while ("):
        assert word not in src, word
    assert "arrive_last" in src
