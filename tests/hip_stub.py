"""The built library over hip_stub.cpp's recording HIP runtime, on a machine without a GPU. Run as a
program (a process of its own, where no other HIP runtime is loaded): reads a list of calls as JSON
from stdin and prints for each its status and what it launched and allocated.

    {"new": name, "w": workload, "n_envs": n}           sim_create and sim_reset of context `name`
    {"call": function, "ctx": name, "args": [..]}       an entry point; "args" are numbers, pointers
                                                        (any value: nothing is read) or "traj:T"
    {"device": d}                                       the current device from here on
"""
import ctypes as C
import importlib.util
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2607_05272_amd")


def build(out):
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I", "/opt/rocm/include", os.path.join(HERE, "hip_stub.cpp"), "-o", out],
                   check=True)
    return out


def run(stub, calls):
    """[(status, log lines split into words)] of `calls`, in a process of its own."""
    r = subprocess.run([sys.executable, os.path.abspath(__file__), stub], input=json.dumps(calls),
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return [(rc, [l.split() for l in log]) for rc, log in json.loads(r.stdout.splitlines()[-1])]


def main(stub_path):
    stub = C.CDLL(stub_path, mode=C.RTLD_GLOBAL)
    stub.stub_log.restype = C.c_char_p
    spec = importlib.util.spec_from_file_location("_lib", os.path.join(PKG, "_lib.py"))
    L = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(L)
    lib, ctx, out = L.load(), {}, []
    for c in json.load(sys.stdin):
        stub.stub_clear()
        rc = 0
        if "device" in c:
            stub.stub_device(c["device"])
        elif "new" in c:
            w, h = c["w"], C.c_void_p()
            cfg = L.make_cfg(w, c["n_envs"])
            rc = lib.sim_create(C.byref(cfg), C.c_void_p(8), C.byref(h)) or lib.sim_reset(h, 1)
            has = ["actions", "logp", "reward"] + ["reward_shadow"] * w["shadow"] + \
                ["value"] * w["value_head"]
            ctx[c["new"]] = h, L.SimTraj(**{f: (i + 1) << 40 for i, f in enumerate(has)})
        else:
            h, traj = ctx[c["ctx"]]
            args = [C.byref(traj) if a == "traj" else a for a in c["args"]]
            rc = getattr(lib, c["call"])(h, *args)
        out.append((rc, stub.stub_log().decode().splitlines()))
    print(json.dumps(out))


if __name__ == "__main__":
    main(sys.argv[1])
