"""Build libhjpd.so for gfx950 with hipcc (in-tree).

Translation units are compiled in parallel: the C-ABI layer, the
linear-tanh unit and the kernel-instantiation units, one or two per (family
shape, dtype).  All device code is compiled with packed FP32 instructions disabled,
and the linked library is kept only if isa_check finds nothing in it.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

if __package__:
    from . import isa_check
else:  # run as a script
    import isa_check

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libhjpd.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

# (lookup suffix, family type, real type)
INSTANCES = [
    ("cnorm2_f32", "CNorm<2>", "float"), ("cnorm2_f64", "CNorm<2>", "double"),
    ("cnorm3_f32", "CNorm<3>", "float"), ("cnorm3_f64", "CNorm<3>", "double"),
    ("cnorm4_f32", "CNorm<4>", "float"), ("cnorm4_f64", "CNorm<4>", "double"),
    ("cnorm10_f32", "CNorm<10>", "float"), ("cnorm10_f64", "CNorm<10>", "double"),
    ("quad_f32", "Quad", "float"), ("quad_f64", "Quad", "double"),
    ("pursuit_f32", "Pursuit", "float"), ("pursuit_f64", "Pursuit", "double"),
    ("isaacs_f32", "Isaacs", "float"), ("isaacs_f64", "Isaacs", "double"),
]

# The FP64 four-node tiles of the two widest families are units of their own,
# compiled with the constants of the sine and cosine left beside their uses
# instead of moved out of the iteration: those registers are short, and with the
# constants moved out the allocator misplaced register copies in three of these
# kernels (isa_check.py).  Same arithmetic and bits.  Against the tiles compiled
# as the rest: quadrotor 8x4 2.25 -> 2.03 ms and 64x4 5.3 -> 3.75 ms (2,000
# points, 150 iterations; before the misplaced copies came in), d = 10 16x4 1.97
# -> 2.03 ms (10,007 points, 200 iterations); for the narrower tiles it costs up
# to 3 %.
K4_FLAGS = ["-DHJPD_K_LO=4", "-mllvm", "-disable-machine-licm"]
UNIT_FLAGS = {}
for _name, _fam, _real in [i for i in INSTANCES if i[0] in ("quad_f64", "cnorm10_f64")]:
    INSTANCES.append((_name + "_k4", _fam, _real))
    UNIT_FLAGS[_name] = ["-DHJPD_K_HI=3", "-DHJPD_K4=%s_k4" % _name]
    UNIT_FLAGS[_name + "_k4"] = K4_FLAGS


def _run(cmd):
    p = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in p.stderr.splitlines() if "packed-fp32-ops' is not a recognized feature" not in l
                    and "is not a recognized feature for this target" not in l)
    if p.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), err))
    return err


def build(jobs: int | None = None, verbose: bool = False) -> str:
    """Compile every unit and link libhjpd.so; returns the library path."""
    os.makedirs(BUILD, exist_ok=True)
    os.makedirs(LIBDIR, exist_ok=True)
    cmds, objs = [], []
    for name, fam, real in INSTANCES:
        o = os.path.join(BUILD, "inst_%s.o" % name)
        cmds.append([HIPCC, *FLAGS, *UNIT_FLAGS.get(name, []), "-DHJPD_FAM=%s" % fam, "-DHJPD_REAL=%s" % real, "-DHJPD_NAME=%s" % name,
                     "-c", os.path.join(CSRC, "hjpd_inst.hip"), "-o", o])
        objs.append(o)
    for unit in ("hjpd_api", "hjpd_lintanh", "hjpd_calib"):
        o = os.path.join(BUILD, unit + ".o")
        cmds.append([HIPCC, *FLAGS, "-c", os.path.join(CSRC, unit + ".hip"), "-o", o])
        objs.append(o)
    jobs = jobs or min(8, os.cpu_count() or 4)
    with cf.ThreadPoolExecutor(jobs) as ex:
        for msg in ex.map(_run, cmds):
            if verbose and msg.strip():
                print(msg, file=sys.stderr)
    tmp = LIB + ".tmp%d" % os.getpid()
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    bad = isa_check.misplaced(tmp, HIPCC, jobs)
    if bad:
        os.remove(tmp)
        raise RuntimeError("kernels with register copies before an EXEC restore (isa_check.py): %s" % ", ".join(sorted(bad)))
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
