"""What the engine launches for a call, without a GPU: builds and asks tests/host_launches.cpp."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


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
