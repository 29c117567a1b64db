"""Builds libbg.so for gfx950 in-tree: one object per kernel (kind, multiplicity, precision,
lane form; kernels fully unrolled per n), the persistent multi-class kernel, and the C-ABI
layer, compiled in parallel with hipcc, then linked shared.  The C-ABI layer embeds a hash
of the sources (source_hash), which the binding checks before it uses the library.

Usage: python -m paper_1002_3446_amd.build [--jobs J]
"""
from __future__ import annotations

import argparse
import concurrent.futures as cf
import hashlib
import os
import subprocess
import sys
import time

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
HEADER = os.path.join(PKG, "..", "include", "bg.h")
OUT_DIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libbg.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    # packed FP32 instructions stay disabled (only scalar FP32 VALU forms are emitted)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # LLVM's CodeGenPrepare pass is quadratic on the recursion's straight-line code (half the
    # compile time of a unit) and changes nothing in its machine code: skipped
    "-mllvm", "-disable-cgp",
]


def source_hash() -> str:
    """sha256 (first 16 hex digits) over the kernel sources in csrc/ (sorted by name), the
    C header and this file (the compiler flags of every unit): the identity a built library
    carries and the binding checks."""
    h = hashlib.sha256()
    for f in sorted(os.listdir(CSRC)):
        if f.endswith((".hip", ".hpp")):
            h.update(f.encode())
            h.update(open(os.path.join(CSRC, f), "rb").read())
    h.update(open(HEADER, "rb").read())
    h.update(open(os.path.abspath(__file__), "rb").read())
    return h.hexdigest()[:16]


def _compile(src: str, obj: str, defines: list[str]) -> tuple[str, float]:
    cmd = [HIPCC, *FLAGS, *defines, "-c", src, "-o", obj]
    t0 = time.time()
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {obj}:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj, time.time() - t0


KINDS = (0, 1, 2)  # 0 generate, 1 amp2, 2 gradient


def has_one_lane(n: int, p: int) -> bool:
    return n <= 9 if p == 32 else n <= 6


def has_lane_pairs(n: int, p: int) -> bool:
    return n >= 9 if p == 32 else n >= 6


def one_or_pair(n: int, p: int) -> bool:
    """FP64 n = 7, 8: one lane per event, two in short calls."""
    return p == 64 and n in (7, 8)


def has_lane_quads(n: int, p: int) -> bool:
    return p == 64 and n >= 10


def has_real_pol(n: int, p: int) -> bool:
    return n <= 12 if p == 32 else n <= 8


def has_wtensor(n: int, p: int) -> bool:
    return (n == 8 or n >= 10) if p == 32 else n in (6, 10)


def unit_flags(n: int, p: int, k: int, f: int) -> list[str]:
    """Extra compiler flags of one kernel unit.  The generation and bg_amp2 units whose recursion
    fills the register file are built without LLVM's pre-RA machine scheduler: its reordering for
    latency raises register pressure, which costs more (scratch spill, AGPR copies) than the
    latency it hides.  With against without, us: two FP32 lanes, 5 10^5 events, n = 10 518 / 511,
    n = 11 743 / 720, 10^6 events n = 12 2053 / 2012 (n = 9 373 / 372: keeps it); four FP64 lanes,
    2^18 events, n = 11 611 / 598, n = 12 1023 / 868 (n = 10 420 / 430: keeps it); two FP64 lanes
    from n = 9.  The one-lane recursions and the gradients keep it too: n = 8 FP32 5.51 / 5.55 ms
    per 2^24 events, FP64 n = 7 bg_amp2 99 / 101 per 5 10^5, gradient n = 8 FP32 2169 / 2192.
    The four-lane units' matrix sums write vector registers: into accumulation registers, as the
    compiler would place them, every sum costs two copies."""
    flags = []
    if k < 2 and (p == 64 and (f == 2 and n >= 9 or f == 5 and n >= 11) or p == 32 and f == 2 and n >= 10):
        flags += ["-mllvm", "-enable-misched=0"]
    if k < 2 and p == 64 and f == 5:
        flags += ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]
    return flags


def units_for(ns, precs=(32, 64), kinds=KINDS):
    """(source, object, defines, expected cost) of every unit; the costliest start first."""
    units = [(os.path.join(CSRC, "bg_capi.hip"), os.path.join(OUT_DIR, "bg_capi.o"),
              [f'-DBG_SOURCE_HASH="{source_hash()}"'], 0),
             (os.path.join(CSRC, "bg_finalize.hip"), os.path.join(OUT_DIR, "bg_finalize.o"), [], 0),
             (os.path.join(CSRC, "bg_hist.hip"), os.path.join(OUT_DIR, "bg_hist.o"), [], 0),
             (os.path.join(CSRC, "bg_probe.hip"), os.path.join(OUT_DIR, "bg_probe.o"), [], 0)]
    if set(range(4, 13)) <= set(ns) and 32 in precs:
        units.append((os.path.join(CSRC, "bg_multi.hip"), os.path.join(OUT_DIR, "bg_multi_p32.o"),
                      # without the pre-RA scheduler, as unit_flags: its large-n paths spill less (n = 4..12 with
                      # 2^26 / 2^n events each, one persistent launch: 1838 / 1587 us; 2^20 / 2^n: 569 / 548)
                      ["-mllvm", "-enable-misched=0"], 1000))
    for n in ns:
        for p in precs:
            for k in kinds:
                if k == 2:
                    forms = (1,)
                else:
                    one = has_one_lane(n, p) or one_or_pair(n, p)
                    forms = tuple(f for f, ok in ((1, one), (2, has_lane_pairs(n, p)),
                                                  (3, k == 0 and has_real_pol(n, p)),
                                                  (4, has_wtensor(n, p)),
                                                  (5, k < 2 and has_lane_quads(n, p))) if ok)
                for f in forms:
                    obj = os.path.join(OUT_DIR, f"bg_n{n:02d}_p{p}_k{k}_f{f}.o")
                    cost = n ** 3 * (2 if p == 64 else 1) * (4 if k == 2 else 1)
                    units.append((os.path.join(CSRC, "bg_inst.hip"), obj,
                                  [f"-DBG_N={n}", f"-DBG_PREC={p}", f"-DBG_KIND={k}", f"-DBG_FORM={f}"]
                                  + unit_flags(n, p, k, f), cost))
    units.sort(key=lambda u: -u[3])
    return units


def build(jobs: int | None = None, verbose: bool = True, ns=range(4, 13)) -> str:
    """Compiles every unit for the multiplicities ns and links libbg.so (always a full build)."""
    os.makedirs(OUT_DIR, exist_ok=True)
    jobs = jobs or min(8, os.cpu_count() or 1)
    units = units_for(list(ns))
    t0 = time.time()
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        done = list(ex.map(lambda u: _compile(u[0], u[1], u[2]), units))
    if verbose:
        slow = sorted(done, key=lambda d: -d[1])[:3]
        print(f"compiled {len(done)} units in {time.time() - t0:.0f} s (slowest: "
              + ", ".join(f"{os.path.basename(o)} {t:.0f} s" for o, t in slow) + ")", file=sys.stderr)
    return _link([d[0] for d in done], verbose)


def _link(objs, verbose) -> str:
    tmp = LIB + ".tmp"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB} (sources {source_hash()})", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("--jobs", type=int, default=None)
    ap.add_argument("--ns", type=str, default="4,5,6,7,8,9,10,11,12",
                    help="comma-separated multiplicities to build (others report BG_ENOTSUP)")
    a = ap.parse_args()
    build(a.jobs, ns=[int(x) for x in a.ns.split(",")])
