"""Host build of the elimination's block kernels (k_getrf.hip, k_trsm.hip) for
tests, as emu.py does for the batched solver's."""
import os
import shutil
import struct
import subprocess
import tempfile

import numpy as np

from . import emu

EXE = os.path.join(emu.OUT_DIR, "emu_blocks")
SOURCES = ["k_getrf.hip", "k_trsm.hip"]
LN, UN, UT, LT = range(4)


def build(exe=EXE, csrc=emu.CSRC, sources=SOURCES, driver="emu_blocks.cpp", watch=()):
    """Compile unless the executable is newer than every input (watch: sources
    that the driver includes)."""
    cc = emu.clang()
    if cc is None:
        raise RuntimeError("clang++ not found")
    os.makedirs(os.path.dirname(exe), exist_ok=True)
    srcs = [os.path.join(csrc, s) for s in sources]
    ours = [os.path.join(emu.HERE, "emu_runtime.cpp"), os.path.join(emu.HERE, driver)]
    inputs = srcs + ours + [os.path.join(csrc, s) for s in watch]
    inputs += [os.path.join(csrc, h) for h in os.listdir(csrc) if h.endswith(".h")]
    inputs += [os.path.join(emu.HERE, "include", "hip", "hip_runtime.h"), os.path.abspath(__file__)]
    if os.path.exists(exe) and all(os.path.getmtime(f) < os.path.getmtime(exe) for f in inputs):
        return exe
    cmd = [cc, "-std=c++17", "-O2", "-g", "-fsanitize=address", "-fno-omit-frame-pointer",
           "-ffp-contract=off", "-Wno-psabi",
           f"-I{os.path.join(emu.HERE, 'include')}",
           f"-I{os.path.join(emu.ROOT, 'include')}", f"-I{csrc}", "-x", "c++", *srcs, *ours, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("host build failed:\n" + r.stderr[-4000:])
    return exe


def run(exe, payload, env=None, timeout=120):
    """The executable's output for an input file's bytes."""
    with tempfile.TemporaryDirectory() as d:
        fin, fout = os.path.join(d, "in"), os.path.join(d, "out")
        with open(fin, "wb") as f:
            f.write(payload)
        e = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1:"
                 "detect_stack_use_after_return=0", **(env or {}))
        r = subprocess.run([exe, fin, fout], capture_output=True, text=True, timeout=timeout, env=e)
        if r.returncode:
            raise RuntimeError(f"host build exited with {r.returncode}:\n{r.stderr[-4000:]}")
        with open(fout, "rb") as f:
            return f.read()


def call(exe, op, A, B=None, C=None, order=0):
    """One operation of emu_blocks.cpp on copies of the arrays. Returns
    (A, B, C, info); C: what follows B in the output (one-dimensional for the
    inverses)."""
    dt = A.dtype
    B = np.zeros((0, 0), dt) if B is None else B
    m = A.shape[1]
    n = B.shape[0] if op in (30, 31) else B.shape[1]
    head = struct.pack("<5q", op, m, n, A.shape[0], B.shape[0])
    parts = [A, B] + ([C] if C is not None else [])
    raw = run(exe, head + b"".join(np.asfortranarray(a).tobytes(order="F") for a in parts),
              env={"EMU_ORDER": str(order)})
    out, off = [], 0
    for a in parts:
        out.append(np.frombuffer(raw, dt, a.size, off).reshape(a.shape, order="F").copy())
        off += a.nbytes
    rest = np.frombuffer(raw[off:-4], dt).copy()
    return out[0], out[1], (out[2] if C is not None else rest), struct.unpack("<i", raw[-4:])[0]
