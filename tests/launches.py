"""What the engine launches for a call, without a GPU: builds and asks tests/host_launches.cpp."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


# Up to how many rounds of a launch's waves the waves take fixed shares: one way, both ways.
ONE_WAY, BOTH_WAYS = 24, 8

# The most blocks that a rotation, a swap-out and a swap-in of the default shapes move by fixed shares, in a
# block-first pool and in a layer-first one; blocks of six layers in segments of (dim, tokens) bf16 values.
SHARES = {(128, 16): ((22, 32, 48), (22, 32, 48)), (65, 8): ((78, 125, 219), (88, 140, 242)),
          (60, 7): ((153, 244, 297), (136, 218, 272)), (20, 5): ((428, 456, 854), (204, 326, 612)),
          (18, 5): ((159, 253, 317), (158, 254, 318)), (9, 5): ((159, 253, 317), (158, 254, 318))}

# (waves, steps of a block) of rotations, swap-outs and swap-ins of the default shapes: blocks of one layer in
# segments of so many vectors, block-first.
ROUNDS = {128: ((68, 2), (36, 2), (44, 2)), 80: ((144, 3), (76, 3), (134, 3))}


def round_lengths(vecs):
    """Block counts just below, at and just above a full round of each kind's waves, from one round to
    the first launch that draws its steps, one way and both."""
    return sorted({max(1, r * waves // steps + d) for waves, steps in ROUNDS[vecs] for r in (1, 2, 3, BOTH_WAYS, ONE_WAY) for d in (0, 1)})


def configured_lengths(wgs, lanes, vecs):
    """Block counts around one round of configured waves, around both limits of the fixed share, and where
    more draws are of four steps; blocks of two layers in segments of `vecs` vectors, a vector per lane."""
    waves, steps = wgs * lanes // 64, -(-4 * vecs // 64)
    return sorted({max(1, r * waves // steps + d) for r in (1, BOTH_WAYS, 14, ONE_WAY, 33) for d in (-1, 0, 1, 3)})


def build(folder):
    """The program, built in `folder`.  Only the host's half of the HIP source is compiled; what it
    would hand to the HIP runtime (the kernels' image) is left unresolved and never looked at."""
    obj, exe = os.path.join(folder, "host_launches.o"), os.path.join(folder, "host_launches")
    subprocess.run([HIPCC, "--offload-host-only", "-x", "hip", "-fPIC", "-std=c++17", "-O1", "-w", "-c",
                    os.path.join(ROOT, "tests", "host_launches.cpp"), "-o", obj], check=True)
    subprocess.run(["g++", obj, "-o", exe, "-Wl,--unresolved-symbols=ignore-all"], check=True)
    return exe


def move(n_out, n_in, dim, layers=1, heads=1, tokens=1, elem=2, path=0, host_layout=0, chunk_layers=0, max_copy_wgs=0, wg_lanes=0,
         vecs_per_lane=0, cache_at=0, pool_at=0):
    return (f"move {path} {host_layout} {layers} {heads} {dim} {tokens} {elem} {chunk_layers} {max_copy_wgs} {wg_lanes} "
            f"{vecs_per_lane} {cache_at} {pool_at} {n_out} {n_in}")


def read(n, dim, layers=1, heads=1, tokens=1, elem=2, max_wgs=0):
    return f"read {layers} {heads} {dim} {tokens} {elem} {max_wgs} {n}"


def launches(exe, calls):
    """For each call its launches, each a dict of what the program says."""
    run = subprocess.run([exe], input="".join(c + "\n" for c in calls), capture_output=True, text=True, check=True, timeout=120)
    every = []
    for part in run.stdout.split("\n\n")[:len(calls)]:
        lines = [line.split() for line in part.strip().splitlines()]
        every.append([{"kernel": w[0], **{k: int(v) for k, v in (x.split("=") for x in w[1:])}} for w in lines])
    assert len(every) == len(calls)
    return every
