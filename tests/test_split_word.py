"""The operations of a split tile's parts on their common word (csrc/split_word.hpp), compiled for the host and run in random
orders against a memory in which a store may arrive late."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("split") / "split_word_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(HERE, "..", "paper_2305_13450_amd", "csrc"),
                           os.path.join(HERE, "split_word_check.cpp"), "-o", exe])
    return exe


def test_every_slice_is_finished_once_in_any_order(check):
    r = subprocess.run([check, "4000"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


def test_the_model_sees_a_clear_that_the_post_does_not_wait_for(check):
    # side launches outlive their chain: without the wait a late clear wipes out the next chain's counts
    r = subprocess.run([check, "4000", "no-drain"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 1 and "seed" in r.stdout
