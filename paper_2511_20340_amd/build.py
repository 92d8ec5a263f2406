"""Build libspecformer.so (HIP, gfx950 only) in-tree with hipcc."""
import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libspecformer.so")
SOURCES = ["api.hip", "attention.hip", "gemm.hip", "gemm_tiles_narrow.hip",
           "gemm_tiles_wide.hip", "gemm_tiles_tall.hip", "gemm_stream.hip", "gemm_block.hip", "gemm_panel.hip",
           "gemm_panel_narrow.hip", "gemm_f32.hip", "elementwise.hip", "accept.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-result"]


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)]
    deps.append(os.path.join(os.path.dirname(HERE), "include", "specformer.h"))
    return any(os.path.getmtime(p) > t for p in deps)


def _compile(flags, out) -> str:
    """Compile every source on its own, a few at a time, and link them into the shared library `out`."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

    def run(cmd):
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
        return res.stdout + res.stderr
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        with concurrent.futures.ThreadPoolExecutor(min(len(SOURCES), os.cpu_count() or 1, 8)) as pool:
            logs = list(pool.map(lambda so: run([hipcc] + flags + ["-c", os.path.join(CSRC, so[0]), "-o", so[1]]),
                                 zip(SOURCES, objs)))
        logs.append(run([hipcc] + flags + ["-shared"] + objs + ["-o", out]))
    return "\n".join(l for l in "".join(logs).splitlines() if "packed-fp32-ops" not in l)


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and not stale():
        return LIB
    log = _compile(FLAGS, LIB)
    if verbose and log.strip():
        print(log, file=sys.stderr)
    return LIB


def build_host_sanitized(out: str) -> str:
    """The same library with AddressSanitizer + UBSan on the HOST side only (argument checking, workspace
    planning, launch glue); device code is built as usual.  For the CPU-only ABI tests."""
    flags = [f for f in FLAGS if f != "-O3"] + ["-O1", "-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host",
                                                "-fsanitize=undefined", "-Xarch_host", "-fno-omit-frame-pointer"]
    _compile(flags, out)
    return out


if __name__ == "__main__":
    print(build(force=True, verbose=True))
