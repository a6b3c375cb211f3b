"""What a call of the C ABI would launch, without a GPU: a child process loads the
recording stand-in of fake_hip.cpp ahead of the library and calls it with
addresses that nothing reads.

As a program: ``launches.py STAND_IN LIBRARY`` with a list of calls on standard
input, each {"reset": [cus, failing attribute queries, failing occupancy
queries]}, {"round": pctree_shape fields} or {"attention": pctree_attn_shape
fields}; prints, per call, the status and the launches.
"""
from __future__ import annotations

import ctypes
import json
import os
import re
import subprocess
import sys


def record(calls, library, workdir):
    """[{"status", "kernels": [(name, grid, block, lds)]}] of every call in turn."""
    here = os.path.dirname(os.path.abspath(__file__))
    stand_in = os.path.join(str(workdir), "fake_hip.so")
    if not os.path.exists(stand_in):
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1",
                        "-I/opt/rocm/include", os.path.join(here, "fake_hip.cpp"), "-o", stand_in],
                       check=True)
    out = subprocess.run([sys.executable, os.path.abspath(__file__), stand_in, library],
                         input=json.dumps(calls), capture_output=True, text=True, check=True)
    return json.loads(out.stdout)


def _kernel(name):
    """'attn_kernel<64>' from a mangled '_ZN..11attn_kernelILi64EEvNS_8AttnArgsE'."""
    m = re.search(r"\d+([a-z_]+_kernel)(I(?:L\w\d+E)+E)?", name)
    args = re.findall(r"L\w(\d+)E", m.group(2) or "")
    return m.group(1) + (f"<{','.join(args)}>" if args else "")


def _main(stand_in, library):
    fake = ctypes.CDLL(stand_in, ctypes.RTLD_GLOBAL)  # found before the runtime's own
    lib = ctypes.CDLL(library)
    fake.fake_launch.restype = ctypes.c_char_p
    lib.pctree_workspace_bytes.restype = ctypes.c_size_t
    lib.pctree_attention_workspace_bytes.restype = ctypes.c_size_t
    A, vp = 0x1000000, ctypes.c_void_p
    results = []
    for call in json.load(sys.stdin):
        status = 0
        n0 = fake.fake_launches()
        if "reset" in call:
            fake.fake_reset(*call["reset"])
            n0 = 0
        elif "round" in call:
            shape = (ctypes.c_int32 * 8)(*call["round"])
            inp, tree = (vp * 6)(*[A] * 6), (vp * 7)(*[A] * 7)
            status = lib.pctree_build_tree(shape, inp, tree, None, vp(A),
                                           ctypes.c_size_t(lib.pctree_workspace_bytes(shape)), None)
        else:
            class AttnShape(ctypes.Structure):
                _fields_ = [("n", ctypes.c_int32 * 6), ("scale", ctypes.c_float)]
            s = AttnShape((ctypes.c_int32 * 6)(*call["attention"]), 0.125)
            ws = lib.pctree_attention_workspace_bytes(ctypes.byref(s))
            status = lib.pctree_tree_attention(ctypes.byref(s), *[vp(A)] * 8, ctypes.c_size_t(ws),
                                               None)
        kernels = []
        for i in range(n0, fake.fake_launches()):
            g, b, lds = ctypes.c_uint(), ctypes.c_uint(), ctypes.c_size_t()
            name = fake.fake_launch(i, ctypes.byref(g), ctypes.byref(b), ctypes.byref(lds)).decode()
            kernels.append((_kernel(name), g.value, b.value, lds.value))
        results.append({"status": status, "kernels": kernels})
    json.dump(results, sys.stdout)


if __name__ == "__main__":
    _main(sys.argv[1], sys.argv[2])
