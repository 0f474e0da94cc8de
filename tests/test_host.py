"""Host-side behaviour that needs no GPU: the binding refuses to work without its shared
library (no fallback path exists), bench.py refuses more than one GPU with a message, and the
entry points the build and smoke checks call exist."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_binding_fails_loudly_without_the_library(tmp_path):
    code = (
        "import sys; sys.path.insert(0, %r)\n"
        "from paper_2607_05272_amd import _lib\n"
        "_lib.LIB_PATH = %r\n"
        "_lib._lib = None\n"
        "try:\n"
        "    _lib.load()\n"
        "except ImportError as e:\n"
        "    print('raised', e)\n"
        "    sys.exit(0)\n"
        "sys.exit(3)\n" % (ROOT, str(tmp_path / "missing.so")))
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "not built" in r.stdout


def test_bench_kernel_classes_name_their_kernels_and_sources():
    """The HBM traffic that bench.py reports for a kernel class is counted over the kernels whose
    names hold the class's pattern and dropped when the class's sources change: every pattern is
    the start of a kernel's name in those sources, and they hold every device header that they
    include (all classes share devmath.hpp and params.hpp)."""
    sys.path.insert(0, ROOT)
    import bench
    csrc = os.path.join(ROOT, "paper_2607_05272_amd", "csrc")
    text = {f: open(os.path.join(csrc, f)).read() for f in os.listdir(csrc)}
    kernel = re.compile(r"__global__[^;{]*?void\s+(\w+)\(")
    for cls, files in bench.KERNEL_SOURCE.items():
        inc = {h for f in files for h in re.findall(r'#include "(\w+\.hpp)"', text[f])}
        assert inc - {"devmath.hpp", "params.hpp"} <= set(files), cls
        if cls in bench.KERNEL_OF:
            names = [n for f in files for n in kernel.findall(text[f])]
            assert any(n.startswith(bench.KERNEL_OF[cls]) for n in names), (cls, names)
    # kernels that the runtime times under a class
    for cls, file in (("rollout", "rollout_wide.hip"), ("ppo", "ppo_fused.hip")):
        assert file in bench.KERNEL_SOURCE[cls]


def test_bench_traffic_is_of_whole_batch_launches():
    """Halves of a batch, which a rollout launches side by side, are not averaged with whole ones."""
    sys.path.insert(0, ROOT)
    import bench
    row = lambda i, grid, v: {"Counter_Name": "FETCH_SIZE", "Kernel_Name": "learned_k<4>",  # noqa: E731
                              "Dispatch_Id": str(i), "Grid_Size": str(grid), "Counter_Value": str(v)}
    rows = [row(0, 512, 5.0), row(1, 512, 6.0), row(2, 1024, 10.0), row(3, 1024, 12.0)]
    assert bench._per_dispatch(rows, "FETCH_SIZE", lambda k: "learned_k" in k) == (11.0, 2)


def test_bench_refuses_several_gpus():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr


def test_graft_entry_points_exist():
    sys.path.insert(0, ROOT)
    import __graft_entry__ as g
    assert callable(g.build) and callable(g.smoke)
