"""Host build of the allocator's searches for a free block (find_set and
claim_free_block in csrc/smmo_device.hpp): while the summary bits of windows
that were claimed to the last block are still set, a search finds the blocks of
the later windows, and does not report an exhausted heap.  Compiled for the
host with a stand-in for HIP (a wavefront of one lane); no GPU."""

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def run(tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Wno-unused-variable", "-Wno-unknown-pragmas",
                           "-I", os.path.join(HERE, "one_lane"), "-I", os.path.join(os.path.dirname(HERE), "include"),
                           "-o", exe, os.path.join(HERE, name + ".cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, check=True, timeout=60).stdout.split()
    return {k: int(v) for k, v in zip(out[::2], out[1::2])}


def test_a_window_behind_is_not_an_exhausted_heap(tmp_path):
    assert run(tmp_path, "search_host") == {"missed": 0, "exhausted": 1, "once": 1}
