"""libburgers.so on a HIP runtime without a GPU (fake_hip.cpp), for host-code tests in a process of their own:
``run(code, tmp)`` executes `code` there with `lib` (the library), `fake` (the runtime's counters) and `B` (the
binding's argument types) defined."""
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
sys.path.insert(0, {root!r})
import numpy as np
import paper_2601_12204_amd as B
import workloads as W
fake = ctypes.CDLL({runtime!r}, mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(B.library_path())
for name in {counters!r}:
    getattr(fake, name).restype = ctypes.c_long
vp, i64 = ctypes.c_void_p, ctypes.c_int64
MAIN = vp(0x1000)                # the caller's stream

def problems(ps):
    return (B.CProblem * len(ps))(*[B.to_cproblem(p) for p in ps])

def create(ps, dtype=B.F64):
    ctx = vp()
    assert lib.burgers_create(problems(ps), i64(len(ps)), dtype, MAIN, ctypes.byref(ctx)) == 0
    return ctx

def state(ps):
    return np.zeros(int(B.packed_offsets(ps)[-1]))
"""
COUNTERS = ["fake_streams_made", "fake_streams_live", "fake_events_made", "fake_events_live", "fake_launches",
            "fake_streams_used"]


def build(tmp) -> str:
    """Compile the runtime, with the symbol versions that the library asks for."""
    sys.path.insert(0, ROOT)
    from paper_2601_12204_amd import library_path
    names = subprocess.run(["nm", "-D", "--undefined-only", library_path()], check=True, capture_output=True,
                           text=True).stdout
    versions = {}
    for name, version in re.findall(r"U (\w*hip\w+)@([\w.]+)", names):
        versions.setdefault(version, []).append(name)
    script = os.path.join(tmp, "versions")
    with open(script, "w") as f:
        for version, members in sorted(versions.items()):
            f.write(f"{version} {{ global: {'; '.join(members)}; }};\n")
        f.write("fake { global: fake_*; };\n")
    out = os.path.join(tmp, "libamdhip64.so.7")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7",
                    f"-Wl,--version-script={script}", "-o", out, os.path.join(HERE, "fake_hip.cpp")], check=True)
    return out


def run(code: str, tmp) -> str:
    prelude = PRELUDE.format(root=ROOT, runtime=build(str(tmp)), counters=COUNTERS)
    done = subprocess.run([sys.executable, "-c", prelude + code], capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stdout + done.stderr
    return done.stdout
