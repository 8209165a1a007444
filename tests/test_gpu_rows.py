"""The row-by-row factorisation of HBM-resident slices at its edges: every slice
width with a ragged last slice, and a network whose longest row does not fit its
buffers, which factors by levels; solutions and gradients against the dense
oracle."""
import numpy as np
import pytest

from gpu_helpers import to_dev
from gen.grids import Network, Scenarios, make_case
from oracle.adjoint import adjoint, loss_grad
from oracle.newton import newton
from oracle.ybus import ybus_of

pytestmark = pytest.mark.gpu


def _check(net, sc, tol, precision, device, picks, slice_width, **kw):
    import torch
    from paper_2606_07099_amd import PFTemplate
    tpl = PFTemplate.from_network(net, sc.batch, tol=tol, precision=precision, **kw)
    info = tpl.info()
    assert info["lds_resident"] == 0 and info["slice_width"] == slice_width
    vm, va, iters, status, _ = tpl.solve(*[to_dev(getattr(sc, k), device) for k in ("pd", "qd", "pg", "vset")])
    g = tpl.adjoint(*[to_dev(x, device) for x in loss_grad(vm.cpu().numpy(), va.cpu().numpy())])
    torch.cuda.synchronize()
    assert int((status != 0).sum()) == 0
    Y = ybus_of(net)
    for b in picks:
        r = newton(Y, net.bus_type, sc.pd[b], sc.qd[b], sc.pg[b], sc.vset[b], tol=tol)
        # FP64: the same iterate; mixed precision: at most one update more
        assert r.iters <= int(iters[b]) <= r.iters + (precision == "mixed")
        assert np.abs(vm[b].cpu().numpy() - r.vm).max() < 1e-8
        assert np.abs(va[b].cpu().numpy() - r.va).max() < 1e-8
        ref = adjoint(Y, net.bus_type, r.vm, r.va, *loss_grad(r.vm, r.va))
        ours = np.concatenate([x[b].cpu().numpy() for x in g])
        want = np.concatenate([ref.pd, ref.qd, ref.pg, ref.vset])
        assert np.linalg.norm(ours - want) <= 1e-6 * np.linalg.norm(want)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("batch,slice_width", [(513, 2), (1027, 4), (2049, 8), (4099, 16)])
def test_every_slice_width_matches_the_oracle(batch, slice_width, precision, device):
    spec, net, sc = make_case("c3", batch=batch)
    _check(net, sc, 1e-8, precision, device, (0, 300, batch - 1), slice_width)


def test_narrow_workgroups_match_the_oracle(device):
    spec, net, sc = make_case("c1", batch=515)
    _check(net, sc, 1e-8, "fp64", device, (0, 514), 2, block_threads=192)


def test_a_row_beyond_the_buffers_factors_by_levels(device):
    """A star of 2000 leaves: the hub's row is refused at two scenarios per
    slice, and the template falls back to one, by levels."""
    n, batch = 2002, 520
    rng = np.random.default_rng(5)
    leaves = np.arange(2, n)
    f = np.concatenate([np.full(n - 2, 1), [0]]).astype(np.int32)
    t = np.concatenate([leaves, [1]]).astype(np.int32)
    r = np.concatenate([rng.uniform(0.01, 0.05, n - 2), [1e-4]])
    bt = np.zeros(n, np.int32)
    bt[0] = 2
    net = Network("star", n, bt, f, t, r, 5 * r, np.zeros(n - 1), np.ones(n), np.zeros(n), np.zeros(n))
    pd = np.zeros((batch, n))
    pd[:, 2:] = rng.uniform(1e-3, 3e-3, (batch, n - 2))
    sc = Scenarios(pd, 0.3 * pd, np.zeros_like(pd), np.ones_like(pd))
    _check(net, sc, 1e-8, "fp64", device, (519,), 1)
