"""Build the test probe libraries (libkdemathprobe.so for gfx950, libhashclaimprobe.so with host code only) in-tree."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIBS = {"kde_math_probe.hip": os.path.join(HERE, "libkdemathprobe.so"),
        "hash_claim_probe.hip": os.path.join(HERE, "libhashclaimprobe.so")}
sys.path.insert(0, os.path.dirname(os.path.dirname(HERE)))


def build(verbose: bool = False) -> list:
    from paper_2606_20374_amd.build import HIPCC, HIP_FLAGS
    for src, lib in LIBS.items():
        tmp = lib + ".tmp"
        cmd = [HIPCC, *HIP_FLAGS, "-shared", os.path.join(HERE, src), "-o", tmp]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError(f"probe build failed:\n{res.stderr}")
        os.replace(tmp, lib)
    return list(LIBS.values())


if __name__ == "__main__":
    print(build(verbose=True))
