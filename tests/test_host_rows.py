"""Host-side replay of the row-by-row factorisation schedule and of the split
block storage (``tests/native/rows_check.cpp``), built with the sanitizers."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from gen.grids import SPECS, make_network
from paper_2606_07099_amd.pf import symbolic_analyze, ybus_from_branches

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_07099_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("rows") / "rows_check")
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "native", "rows_check.cpp"),
           os.path.join(CSRC, "symbolic.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return out


def _write(path, bus_type, f, t, r, x, bc):
    with open(path, "w") as fh:
        fh.write(f"{len(bus_type)} {len(f)}\n" + " ".join(str(int(v)) for v in bus_type) + "\n")
        for k in range(len(f)):
            fh.write("%d %d %.17g %.17g %.17g\n" % (f[k], t[k], r[k], x[k], bc[k]))
    return str(path)


def _run(checker, net, *args, status=0):
    r = subprocess.run([checker, net, *map(str, args)], capture_output=True, text=True, timeout=600)
    assert r.returncode == status, r.stdout + r.stderr
    return r.stdout


@pytest.mark.parametrize("name", list(SPECS))
def test_row_schedule_on_every_grid(checker, tmp_path, name):
    net = make_network(SPECS[name])
    p = _write(tmp_path / "net.txt", net.bus_type, net.f, net.t, net.r, net.x, net.bc)
    indptr, indices, _, _ = ybus_from_branches(net.n_bus, net.f, net.t, net.r, net.x, net.bc)
    longest = symbolic_analyze(net.n_bus, net.bus_type, indptr, indices)[0]["max_row_blocks"]
    # slice width, threads per workgroup, row buffer blocks of one scenario,
    # metadata words: the library's launch shapes, narrow workgroups, a
    # workgroup that is no power of two, and buffers that hold few rows
    for tail, args in ((32, (1, 1024, 2500, 12288)), (16, (1, 1024, 2500, 12288)), (32, (16, 1024, 440, 6144)),
                       (16, (16, 1024, 200, 6144)), (16, (8, 1024, 265, 6144)), (32, (2, 256, 120, 6144)),
                       (32, (4, 192, 90, 1600)), (16, (16, 64, 100, 1600))):
        if args[2] < longest:
            assert "row buffers" in _run(checker, p, tail, *args, status=3)
        else:
            assert "violations 0" in _run(checker, p, tail, *args)


def test_rows_that_do_not_fit_are_refused(checker, tmp_path):
    """A star's hub eliminates all its leaves: its row outgrows the buffers,
    then the metadata; a path's rows fit the smallest of both."""
    n = 400
    hub = _write(tmp_path / "star.txt", [2] + [0] * (n - 1), [1] * (n - 2) + [0], list(range(2, n)) + [1],
                 np.full(n - 1, 0.01), np.full(n - 1, 0.05), np.zeros(n - 1))
    assert "violations 0" in _run(checker, hub, 0, 1, 1024, 400, 12288)
    assert "row buffers" in _run(checker, hub, 0, 1, 1024, 300, 12288, status=3)
    assert "metadata" in _run(checker, hub, 0, 1, 1024, 400, 1600, status=3)
    path = _write(tmp_path / "path.txt", [2] + [0, 1] * 20, list(range(40)), list(range(1, 41)),
                  np.full(40, 0.01), np.full(40, 0.05), np.zeros(40))
    assert "violations 0" in _run(checker, path, 32, 16, 1024, 64, 320)
