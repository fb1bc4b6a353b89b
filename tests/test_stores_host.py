"""Which calls leave their stores to the L2: the rule of kv_engine.hpp at its edges, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_which_calls_leave_their_stores_to_the_l2(tmp_path):
    exe = str(tmp_path / "host_stores")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                    "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(ROOT, "tests", "host_stores.cpp"),
                    "-o", exe], check=True)
    mib = 8 << 20
    cases = [
        # bytes per vector, piece, layer-first, block bytes, slots in runs of, out, in
        ((16, 64, 1, 1024, 1, 8192, 8192), 1),           # 8 MiB of pieces of half a line, scattered
        ((16, 64, 1, 1024, 1000, 8192, 8192), 1),        # and of consecutive slots
        ((16, 128, 1, 2048, 1, 4096, 4096), 1),
        ((16, 128, 1, 2048, 1, 4095, 4095), 0),          # a block less than 8 MiB
        ((16, 144, 1, 2304, 1, 4096, 4096), 1),
        ((16, 144, 1, 2304, 2, 4096, 4096), 0),          # every second slot follows the one before: a run
        ((16, 1008, 1, 16128, 1, 1024, 1024), 1),
        ((16, 1024, 1, 16384, 1, 1024, 1024), 0),        # 1 KiB at a time
        ((16, 32768, 1, 2 << 20, 1, 128, 128), 0),
        ((16, 128, 0, 128, 1, mib // 128, mib // 128), 1),    # block-first, a block is a line
        ((16, 160, 0, 160, 1, mib // 160 + 1, mib // 160 + 1), 0),
        ((16, 2 << 20, 0, 2 << 20, 1, 128, 128), 0),
        ((16, 400, 1, 6400, 1, 2000, 0), 0),             # one way
        ((16, 400, 1, 6400, 1, 0, 2000), 0),
        ((16, 400, 1, 6400, 1, 0, 0), 0),
        ((16, 400, 1, 6400, 1, 2000, 4000), 1),          # twice as much in, and more
        ((16, 400, 1, 6400, 1, 2000, 4001), 0),
        ((16, 400, 1, 6400, 1, 2000, 1001), 1),          # less than twice as much out, and twice
        ((16, 400, 1, 6400, 1, 2000, 1000), 0),
        ((16, 64, 1, 1024, 1, 16384, 2049), 1),          # pieces of a line: less than eight times as much out
        ((16, 64, 1, 1024, 1, 16384, 2048), 0),
        ((8, 200, 1, 3200, 1, 3000, 3000), 1),        # 8-byte vectors: runs, too, below 512 bytes
        ((8, 200, 1, 3200, 1000, 3000, 3000), 1),
        ((16, 208, 1, 3328, 1000, 3000, 3000), 0),
        ((8, 520, 1, 8320, 1, 2000, 2000), 1),
        ((8, 520, 1, 8320, 1000, 2000, 2000), 0),
    ]
    run = subprocess.run([exe], input="".join(" ".join(map(str, c)) + "\n" for c, _ in cases), capture_output=True,
                         text=True, check=True, timeout=60)
    assert [int(x) for x in run.stdout.split()] == [want for _, want in cases]
