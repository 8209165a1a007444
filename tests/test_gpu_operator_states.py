"""Operator values at unusual voltage states (zero, infinite, NaN and tiny
magnitudes at some buses) and at the edges of the launch rules.  The values are those of the documented entry
formulas (rectangular products, d/d|V| entries divided by the magnitude of the
column's bus), so where a formula has no value the result is NaN, and it does
not depend on whether the per-bus state is held in LDS (up to 4096 buses) or in
device memory."""
import numpy as np
import pytest

from gpu_helpers import to_dev
from gen.grids import GridSpec, make_network
from paper_2606_07099_amd.pf import ybus_from_branches

pytestmark = pytest.mark.gpu


def _network(n):
    return make_network(GridSpec("sized", 100, n, round(0.3 * n), round(1.4 * n), 1, 0.10, 1e-8, load_factor=0.05), 1)


def j1_values(net, indptr, indices, vm, va):
    """Values of J1 (rows dP of the PV and PQ buses, dQ of the PQ buses; columns
    |V| of the PQ buses, theta of the PV and PQ buses) at one state."""
    n = net.n_bus
    yp, yi, yg, yb = ybus_from_branches(n, net.f, net.t, net.r, net.x, net.bc)
    bt = np.asarray(net.bus_type)
    pvpq, pq = np.flatnonzero(bt != 2), np.flatnonzero(bt == 0)
    rows = np.repeat(np.arange(len(indptr) - 1), np.diff(indptr))
    is_p, is_vm = rows < pvpq.size, indices < pq.size
    i = np.concatenate([pvpq, pq])[rows]
    j = np.concatenate([pq, pvpq])[indices]
    yrow = np.repeat(np.arange(n), np.diff(yp))
    key, want = yrow.astype(np.int64) * n + yi, i.astype(np.int64) * n + j
    order = np.argsort(key)
    at = order[np.searchsorted(key[order], want)]
    assert (key[at] == want).all()
    G, B = np.asarray(yg)[at], np.asarray(yb)[at]
    e, f = vm * np.cos(va), vm * np.sin(va)
    ir, ii = np.zeros(n), np.zeros(n)
    np.add.at(ir, yrow, yg * e[yi] - yb * f[yi])
    np.add.at(ii, yrow, yg * f[yi] + yb * e[yi])
    P, Q = e * ir + f * ii, f * ir - e * ii
    c, s = e[i] * e[j] + f[i] * f[j], f[i] * e[j] - e[i] * f[j]
    gs, gc = G * s - B * c, G * c + B * s
    off = np.where(is_vm, np.where(is_p, gc, gs) / vm[j], np.where(is_p, gs, -gc))
    diag = np.where(is_vm, np.where(is_p, P[i] / vm[i] + G * vm[i], Q[i] / vm[i] - B * vm[i]),
                    np.where(is_p, -Q[i] - B * vm[i] ** 2, P[i] - G * vm[i] ** 2))
    return -np.where(i == j, diag, off)


def _compare(got, want):
    assert (np.isnan(got) == np.isnan(want)).all()
    inf = np.isinf(want)
    assert (got[inf] == want[inf]).all()
    ok = np.isfinite(want)
    # sums of a few products of values below the largest entry: 1e-12 of it
    assert np.abs(got[ok] - want[ok]).max() <= 1e-12 * np.abs(want[ok]).max()


@pytest.mark.parametrize("n", [118, 4200])
@pytest.mark.parametrize("bad", [0.0, float("inf"), float("nan"), 1e-30])
def test_special_magnitudes_follow_the_entry_formulas(n, bad, device):
    import torch
    from paper_2606_07099_amd import PFTemplate
    from paper_2606_07099_amd.pf import PF_OP_J1
    net = _network(n)
    tpl = PFTemplate.from_network(net, 1)
    pat = tpl.operator_pattern(PF_OP_J1)
    rng = np.random.default_rng(8)
    vm, va = 1 + 0.03 * rng.standard_normal((3, n)), 0.2 * rng.standard_normal((3, n))
    vm[1, np.flatnonzero(np.asarray(net.bus_type) == 0)[::40]] = bad
    got = tpl.operator(PF_OP_J1, to_dev(vm, device), to_dev(va, device)).values()
    torch.cuda.synchronize()
    got = got.cpu().numpy().reshape(3, -1)
    with np.errstate(all="ignore"):
        for b in range(3):
            _compare(got[b], j1_values(net, pat["indptr"], pat["indices"], vm[b], va[b]))


# two scenarios per workgroup up to 2048 buses, state in LDS up to 4096; the
# values of up to 64 scenarios in four or more splits, where each diagonal entry
# forms its own bus's injection
@pytest.mark.parametrize("n,count", [(300, 64), (300, 65), (2048, 513), (2049, 513), (4096, 1), (4096, 64),
                                     (4096, 65), (4097, 2)])
def test_values_at_the_edges_of_the_launch_rules(n, count, device):
    import torch
    from paper_2606_07099_amd import PFTemplate
    from paper_2606_07099_amd.pf import PF_OP_J1
    net = _network(n)
    tpl = PFTemplate.from_network(net, 1)
    pat = tpl.operator_pattern(PF_OP_J1)
    rng = np.random.default_rng(9)
    vm, va = 1 + 0.03 * rng.standard_normal((count, n)), 0.2 * rng.standard_normal((count, n))
    tvm, tva = to_dev(vm, device), to_dev(va, device)
    out = tpl.operator(PF_OP_J1, tvm, tva)
    out.values().fill_(float("nan"))
    got = tpl.operator(PF_OP_J1, tvm, tva, out=out).values()
    torch.cuda.synchronize()
    assert not bool(torch.isnan(got).any())
    for b in sorted({0, count // 2, count - 1}):
        _compare(got.view(count, -1)[b].cpu().numpy(), j1_values(net, pat["indptr"], pat["indices"], vm[b], va[b]))


# workgroups of 64, 128, 256, 512 and 1024 threads, one and two scenarios each
@pytest.mark.parametrize("count", [7, 515])
@pytest.mark.parametrize("n", [14, 42, 43, 85, 86, 170, 171, 511, 512])
def test_values_with_every_workgroup_size(n, count, device):
    test_values_at_the_edges_of_the_launch_rules(n, count, device)
