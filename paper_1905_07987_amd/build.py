"""Build libadg.so (HIP, gfx950) in the package directory.

Every translation unit under ``csrc/`` is compiled with hipcc for gfx950 in
parallel, then linked into ``paper_1905_07987_amd/libadg.so``.  Packed FP32
instructions are disabled for all device code.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libadg.so")
ARCH = "gfx950"

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC)
                  if f.endswith((".hip", ".cpp")) and f != "gen_tables.cpp")


def _compile(src: str, extra: list[str]) -> tuple[str, str]:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = ["hipcc", "-x", "hip", "-c", src, "-o", obj] + FLAGS + extra
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{p.stderr[-6000:]}")
    return obj, p.stderr


def generate_tables() -> str:
    """Compile and run gen_tables (host only) to write csrc/tables_gen.hpp."""
    exe = os.path.join(BUILD, "gen_tables")
    cmd = ["g++", "-O2", "-std=c++17", "-o", exe, os.path.join(CSRC, "gen_tables.cpp"),
           os.path.join(CSRC, "basis.cpp")]
    subprocess.run(cmd, check=True)
    out = os.path.join(CSRC, "tables_gen.hpp")
    subprocess.run([exe, out], check=True)
    return out


# Headers compiled again at run time by hiprtc for user-supplied PDEs, under
# the names their #include directives use.
RTC_HEADERS = [("kernels.hpp", "csrc/kernels.hpp"), ("adg_internal.hpp", "csrc/adg_internal.hpp"),
               ("pde.hpp", "csrc/pde.hpp"), ("tables_gen.hpp", "csrc/tables_gen.hpp"),
               ("predict64.hpp", "csrc/predict64.hpp"), ("predict_line.hpp", "csrc/predict_line.hpp"),
               ("basis.hpp", "csrc/basis.hpp"), ("adjoint.hpp", "csrc/adjoint.hpp"),
               ("user_pde.hpp", "csrc/user_pde.hpp"), ("../../include/adg.h", "../include/adg.h")]


def generate_rtc_headers() -> str:
    """Write _build/rtc_headers.cpp: the header texts as byte arrays."""
    out = os.path.join(BUILD, "rtc_headers.cpp")
    lines = ["// Generated by build.py: header texts for hiprtc; do not edit.", "namespace adg {"]
    for i, (_, rel) in enumerate(RTC_HEADERS):
        data = open(os.path.join(HERE, rel), "rb").read() + b"\0"
        body = ",".join(str(b) for b in data)
        lines.append(f"static const char kText{i}[] = {{{body}}};")
    lines.append(f"extern const int kRtcHeaderCount = {len(RTC_HEADERS)};")
    lines.append("extern const char* const kRtcHeaderNames[] = {" +
                 ", ".join(f'"{name}"' for name, _ in RTC_HEADERS) + "};")
    lines.append("extern const char* const kRtcHeaderTexts[] = {" +
                 ", ".join(f"kText{i}" for i in range(len(RTC_HEADERS))) + "};")
    lines.append("}  // namespace adg")
    open(out, "w").write("\n".join(lines) + "\n")
    return out


def build(jobs: int | None = None, extra: list[str] | None = None, verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    generate_tables()
    extra = list(extra or [])
    srcs = sources() + [generate_rtc_headers()]
    jobs = jobs or min(len(srcs), max(1, (os.cpu_count() or 4)))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        results = list(ex.map(lambda s: _compile(s, extra), srcs))
    if verbose:
        for _, log in results:
            if log:
                sys.stderr.write(log)
    objs = [o for o, _ in results]
    tmp = LIB + ".tmp"
    cmd = ["hipcc", "-shared", f"--offload-arch={ARCH}", "-fPIC", "-o", tmp] + objs + ["-lhiprtc"]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError(f"link failed:\n{p.stderr[-4000:]}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    extra = sys.argv[1:]
    print(build(extra=extra, verbose=bool(extra)))
