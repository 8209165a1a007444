"""The launch plan of HBM-resident templates, as ``pf_template_build`` makes it
(``tests/native/plan_check.cpp``, built with the sanitizers): which path a
network's factorisation takes, and a replay of its schedule."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from gen.grids import GridSpec, Network, SPECS, make_network

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_07099_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("plan") / "plan_check")
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "native", "plan_check.cpp"),
           os.path.join(CSRC, "hbm_plan.cpp"), os.path.join(CSRC, "symbolic.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    return out


def grid(n, seed=1, branches=1.4):
    return make_network(GridSpec("sized", 100, n, round(0.3 * n), round(branches * n), 1, 0.10, 1e-8,
                                 load_factor=0.05), seed)


def hubs(n, leaves, count=2):
    """A ring of n buses, ``leaves`` more at each of one or two of them: rows as
    long as that, whose task records have a step per leaf."""
    ring = np.arange(n)
    f = np.concatenate([ring, np.repeat([5, n // 2][:count], leaves)])
    t = np.concatenate([(ring + 1) % n, n + np.arange(count * leaves)])
    m = n + count * leaves
    bt = np.where(np.arange(m) % 7 == 3, 1, 0)
    bt[n:] = 0
    bt[0] = 2
    r = np.full(f.size, 0.01)
    return Network("hubs", m, bt.astype(np.int32), f.astype(np.int32), t.astype(np.int32), r, 5 * r,
                   np.zeros(f.size), np.ones(m), np.zeros(m), np.zeros(m))


def write(path, net):
    with open(path, "w") as fh:
        fh.write(f"{net.n_bus} {len(net.f)}\n" + " ".join(str(int(v)) for v in net.bus_type) + "\n")
        for k in range(len(net.f)):
            fh.write("%d %d %.17g %.17g %.17g\n" % (net.f[k], net.t[k], net.r[k], net.x[k], net.bc[k]))
    return str(path)


def plan(checker, path, precision="fp64", batch=256, threads=1024):
    r = subprocess.run([checker, path, precision, str(batch), str(threads)], capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0 and "violations 0" in r.stdout, r.stdout + r.stderr
    m = re.search(r"path (\w+) slice (\d+) y (\d+) lds (\d+) tail (\d+) longest (\d+) words (\d+) waves (\d+)", r.stdout)
    return dict(zip(("slice", "y", "lds", "tail", "longest", "words", "waves"), map(int, m.groups()[1:])), path=m.group(1))


@pytest.mark.parametrize("n", [300, 1354, 2600, 4200, 4600, 5000, 5600, 6000, 6600])
def test_single_scenario_fp64_slices_factor_as_tasks(checker, tmp_path, n):
    """y in LDS does not crowd out the wavefronts' row buffers."""
    assert plan(checker, write(tmp_path / "net.txt", grid(n)))["path"] == "tasks"


@pytest.mark.parametrize("leaves,words,waves", [(150, 650, 16), (200, 850, 8), (235, 1000, 8)])
def test_a_long_row_keeps_the_tasks(checker, tmp_path, leaves, words, waves):
    """A record beyond a wavefront's share of the metadata, and a row beyond its
    share of the buffers."""
    p = plan(checker, write(tmp_path / "net.txt", hubs(400, leaves)))
    assert p["path"] == "tasks" and p["longest"] > leaves and p["words"] > words and p["waves"] == waves
    # beyond one-byte targets: by levels
    assert plan(checker, write(tmp_path / "net.txt", hubs(400, 256)))["path"] == "levels"


def test_a_record_of_the_full_share_keeps_the_tasks(checker, tmp_path):
    """9000 buses whose longest record is a few words more than a sixteenth of
    the metadata area."""
    p = plan(checker, write(tmp_path / "net.txt", grid(9000, seed=2)))
    assert p["path"] == "tasks" and p["waves"] == 16


@pytest.mark.parametrize("n,precision,batch", [(300, "fp64", 1000), (300, "mixed", 2400), (118, "fp64", 400),
                                               (1354, "fp64", 2400), (1354, "fp64", 400)])
@pytest.mark.parametrize("threads", [64, 256, 512])
def test_narrow_workgroups_take_the_lds_they_use(checker, tmp_path, n, precision, batch, threads):
    p = plan(checker, write(tmp_path / "net.txt", grid(n)), precision, batch, threads)
    if threads == 64 and n <= 300 and p["slice"] <= 2:   # several of them fit a compute unit
        assert 3 * p["lds"] <= 160 * 1024


@pytest.mark.parametrize("name,precision,batch,path", [
    ("c1", "fp64", 37, "tasks"), ("c2", "fp64", 37, "tasks"), ("c4", "fp64", 256, "tasks"),
    ("c4", "mixed", 256, "tasks"), ("c3", "fp64", 2048, "rows"), ("c2", "fp64", 4096, "rows"),
    ("c2", "mixed", 4096, "rows"), ("c4", "fp64", 1100, "rows")])
def test_named_grids_replay_their_schedules(checker, tmp_path, name, precision, batch, path):
    assert plan(checker, write(tmp_path / "net.txt", make_network(SPECS[name])), precision, batch)["path"] == path


# either side of the lines between rows and levels
@pytest.mark.parametrize("n,precision,batch,threads,path", [
    (300, "fp64", 600, 1024, "levels"), (1354, "fp64", 600, 1024, "levels"), (2600, "fp64", 600, 1024, "rows"),
    (700, "fp64", 1100, 1024, "levels"), (1354, "fp64", 1100, 1024, "rows"), (300, "fp64", 2100, 1024, "rows"),
    (300, "mixed", 600, 1024, "levels"), (2600, "mixed", 600, 1024, "levels"), (1354, "mixed", 1100, 1024, "levels"),
    (2600, "mixed", 1100, 1024, "rows"), (300, "mixed", 2100, 1024, "levels"), (1100, "mixed", 2100, 1024, "rows"),
    (300, "mixed", 4200, 1024, "rows"), (300, "fp64", 250, 768, "tasks"), (2800, "mixed", 250, 1024, "levels"),
    (3400, "mixed", 250, 1024, "tasks"), (1354, "fp64", 400, 512, "levels"), (4000, "fp64", 400, 512, "tasks"),
    (4000, "mixed", 250, 512, "levels"), (300, "fp64", 400, 256, "levels"), (5000, "fp64", 250, 256, "tasks"),
    (30, "fp64", 4200, 256, "levels"), (30, "mixed", 600, 64, "levels"), (57, "fp64", 4200, 256, "rows"),
    (5000, "fp64", 400, 256, "levels"), (5000, "fp64", 250, 192, "levels")])
def test_rows_and_levels_where_each_is_the_faster(checker, tmp_path, n, precision, batch, threads, path):
    p = plan(checker, write(tmp_path / "net.txt", grid(n)), precision, batch, threads)
    assert p["path"] == path and p["slice"] == {2: 2, 4: 4, 8: 8, 16: 16}.get(batch // 256, 1)


def test_long_rows_of_wide_slices_go_row_by_row(checker, tmp_path):
    path = write(tmp_path / "net.txt", hubs(400, 150))
    assert plan(checker, path, "fp64", 600)["path"] == "rows"
    assert plan(checker, write(tmp_path / "net.txt", hubs(400, 20)), "fp64", 600)["path"] == "levels"


def test_meshed_networks_of_few_scenarios_go_by_levels(checker, tmp_path):
    """Three branches per bus: the chain of a row's steps outweighs the bytes."""
    path = write(tmp_path / "net.txt", grid(1200, branches=3.0))
    assert plan(checker, path, "fp64", 600)["path"] == "levels"
    assert plan(checker, path, "fp64", 1100)["path"] == "levels"
    assert plan(checker, path, "fp64", 2100)["path"] == "rows"


@pytest.mark.parametrize("precision,batch,slice_width",
                         [("mixed", 600, 2), *((p, *x) for p in ("fp64", "mixed")
                                               for x in ((1100, 4), (2100, 8), (4200, 16)))])
def test_rows_that_do_not_fit_leave_the_slice_its_width(checker, tmp_path, precision, batch, slice_width):
    p = plan(checker, write(tmp_path / "net.txt", hubs(20, 2000, 1)), precision, batch)
    assert p["path"] == "levels" and p["slice"] == slice_width


def test_rows_that_fit_half_the_slice_halve_it(checker, tmp_path):
    path = write(tmp_path / "net.txt", hubs(20, 400, 1))
    p = plan(checker, path, "fp64", 4200)
    assert p["path"] == "rows" and p["slice"] == 8
    # with y in device memory they fit the whole of a narrower one
    p = plan(checker, path, "fp64", 2100)
    assert p["path"] == "rows" and p["slice"] == 8 and p["y"] == 0
