"""The keys that problem-specialised kernels are found by: what every call
looks up is no longer than the generated source, and what is kept on disk
covers the device headers that the kernel is compiled from, and no others."""
import glob
import os
import shutil
import struct
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r"""
import sys
import numpy as np
sys.path.insert(0, sys.argv[1])
import paper_1705_03666_amd as pdd
from workloads import configs as CF
w = CF.c4()
r = pdd.branching_eval(w.problem, np.zeros((2, w.problem.ndim)), 100, 3, precision="fp32", specialize="on")
import torch
torch.cuda.synchronize()
print(float(r["mean"][0]), flush=True)
"""


def test_keys(tmp_path):
    from paper_1705_03666_amd import build as B
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not available")
    objs = [os.path.join(B.BUILD, "specialize.o"), os.path.join(B.BUILD, B.RTC_SOURCE.replace(".cpp", ".o"))]
    if not all(os.path.exists(o) for o in objs):
        B.build(verbose=False)
    obj, exe = str(tmp_path / "spec_key_check.o"), str(tmp_path / "spec_key_check")
    flags = [f for f in B.FLAGS if not f.startswith("--offload-arch")]
    subprocess.check_call([B._hipcc()] + flags + ["-c", os.path.join(HERE, "spec_key_check.cpp"), "-o", obj])
    subprocess.check_call([B._hipcc(), obj] + objs + ["-lhiprtc", "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    rows = {f[0]: f[1:] for f in (line.split() for line in r.stdout.splitlines())}
    for source, table, *_ in rows.values():
        assert int(table) <= int(source) + 16
    common = {"pdd_internal.hpp", "pdd_device.hpp"}
    assert set(rows["branch"][2:]) == common | {"branch_kernels.hpp"}
    assert set(rows["walk"][2:]) == common | {"walk_kernels.hpp", "walk_stream.hpp"}


@pytest.mark.gpu
def test_a_branching_entry_does_not_hold_the_walks(tmp_path):
    """The key of the entry that a branching call writes (magic, four lengths,
    key, symbol, code object)."""
    print("spec keys: a branching call in a process of its own", flush=True)
    env = dict(os.environ, PDD_JIT_CACHE=str(tmp_path))
    p = subprocess.run([sys.executable, "-c", CHILD, ROOT], env=env, capture_output=True, text=True, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    entry, = glob.glob(str(tmp_path / "*.pddjit"))
    with open(entry, "rb") as f:
        d = f.read()
    key = d[40:40 + struct.unpack("<Q", d[8:16])[0]].decode()
    assert "k_branch(const BranchParams" in key
    assert "stream_walk(" not in key and "k_walk_adj(" not in key
