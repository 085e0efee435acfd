"""The persistent kernels' scheduler compiled for the host, a workgroup as one
thread per wavefront: whichever wavefront is late to read a word that the
workgroup shares, all of them get the same ticket and the same outcome of a
wait, also when the word is used again at once, and leave a batch together when
an error comes up.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2504_19171_amd", "csrc")


@pytest.fixture(scope="module")
def sched_words(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("sched") / "sched_words")
    cmd = ["g++", "-O1", "-std=c++17", "-pthread", "-w", "-I", os.path.join(HERE, "host"), "-I", CSRC,
           os.path.join(HERE, "host", "sched_words.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    return exe


@pytest.mark.parametrize("late", [-1, 0, 1, 2, 3])
def test_late_wavefront_gets_the_same_words(sched_words, late):
    res = subprocess.run([sched_words, str(late)], capture_output=True, text=True, timeout=20)
    assert res.returncode == 0, res.stdout + res.stderr
