"""Build the HIP library (csrc/*.hip -> libarith_sampling.so) for gfx950 with hipcc.

hipcc cross-compiles without a GPU.  The .so stays in-tree next to this file.
"""
import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libarith_sampling.so")
SOURCES = ["as_api.hip", "as_step.hip", "as_threshold.hip", "as_wide.hip", "as_model.hip", "as_interval.hip", "as_fused.hip",
           "as_small.hip", "as_rows.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def stale():
    if not os.path.exists(OUT):
        return True
    t = os.path.getmtime(OUT)
    deps = sources() + [os.path.join(CSRC, "as_common.hpp"), os.path.join(CSRC, "as_row.hpp"), os.path.join(CSRC, "as_tile.hpp"), os.path.join(CSRC, "as_pairs.hpp"),
                        os.path.join(CSRC, "as_workspace.hpp"),
                        os.path.join(HERE, "..", "include", "arith_sampling.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def build(force=True, extra=()):
    if not force and not stale():
        return OUT
    # one compiler per source, side by side; then the link
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in sources()]
        flags = [f for f in FLAGS if f != "-shared"] + list(extra)
        with concurrent.futures.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            for _ in pool.map(lambda so: subprocess.run(["hipcc"] + flags + ["-c", so[0], "-o", so[1]], check=True),
                              zip(sources(), objs)):
                pass
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-fPIC", "-shared"] + objs + ["-o", OUT], check=True)
    return OUT


if __name__ == "__main__":
    print(build(force=True, extra=sys.argv[1:]))
