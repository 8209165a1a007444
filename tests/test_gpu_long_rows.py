"""The HBM-resident paths against the dense oracle where other tests do not take
them: long rows (a task record and a buffer beyond a wavefront's share, a row
that fits no row chunk), narrow slices row by row, tasks of narrow workgroups."""
from dataclasses import replace

import numpy as np
import pytest

from test_gpu_rows import _check
from test_host_plan import hubs
from gen.grids import GridSpec, Scenarios, make_network, make_scenarios

pytestmark = pytest.mark.gpu


def _scenarios(net, batch, seed=3):
    rng = np.random.default_rng(seed)
    pq = np.asarray(net.bus_type) == 0
    pd = np.where(pq, rng.uniform(1e-5, 2e-5, (batch, net.n_bus)), 0.0)
    return Scenarios(pd, 0.3 * pd, np.zeros_like(pd), np.ones_like(pd))


def _path(net, batch, precision, **kw):
    from paper_2606_07099_amd import PFTemplate
    tpl = PFTemplate.from_network(net, batch, precision=precision, **kw)
    path = tpl.info()["factor_path"]
    tpl.close()
    return path


@pytest.mark.parametrize("leaves", [150, 200, 235])
def test_long_rows_as_tasks_match_the_oracle(leaves, device):
    net = hubs(300, leaves)
    sc = _scenarios(net, 20)
    _check(net, sc, 1e-9, "fp64", device, (0, 19), 1)


def test_the_template_tells_its_path(device):
    from paper_2606_07099_amd import PFTemplate
    from gen.grids import SPECS, make_network
    c0 = make_network(SPECS["c0"])
    for net, batch, precision, path in ((c0, 4, "fp64", "lds"), (hubs(300, 235), 20, "fp64", "tasks"),
                                        (hubs(300, 256), 20, "fp64", "levels"),
                                        (hubs(900, 20), 20, "mixed", "levels"), (hubs(900, 20), 4200, "fp64", "rows")):
        tpl = PFTemplate.from_network(net, batch, precision=precision)
        assert tpl.info()["factor_path"] == path
        tpl.close()


@pytest.mark.parametrize("batch,slice_width", [(1030, 4), (2050, 8), (4100, 16)])
def test_wide_slices_by_levels_match_the_oracle(batch, slice_width, device):
    """A hub's row of 2000 blocks fits no row chunk: the slice keeps its width
    and factors by levels in place.  (FP64 only: with FP32 factors the gradient of
    such a network is good to 3e-4, on every path.)"""
    net = hubs(20, 2000, 1)
    sc = _scenarios(net, batch)
    _check(net, sc, 1e-9, "fp64", device, (batch - 1,), slice_width)


def _grid(n, batch):
    """A grid of n buses at a load that the flat start converges from."""
    spec = GridSpec("sized", 100, n, round(0.3 * n), round(1.4 * n), 1, 0.10, 1e-8, load_factor=0.05,
                    z_scale=min(1.0, (118 / n) ** 0.5))
    net = make_network(spec, 1)
    net = replace(net, vset=1.0 + 0.3 * (net.vset - 1.0))
    return net, make_scenarios(net, spec, batch, 1)


@pytest.mark.parametrize("n,batch,precision,slice_width", [(1200, 1030, "fp64", 4), (2300, 520, "fp64", 2),
                                                           (2300, 1030, "mixed", 4)])
def test_narrow_slices_row_by_row_match_the_oracle(n, batch, precision, slice_width, device):
    net, sc = _grid(n, batch)
    assert _path(net, batch, precision) == "rows"
    _check(net, sc, 1e-8, precision, device, (batch - 1,), slice_width)


def test_mixed_rows_of_two_match_fp64(device):
    """Only the largest grid takes them: too large for the dense oracle."""
    import torch
    from oracle.adjoint import loss_grad
    from gpu_helpers import make_gpu_case
    out = {}
    for precision in ("fp64", "mixed"):
        spec, net, sc, tpl, d, tol = make_gpu_case("c4", device, batch=513, precision=precision)
        info = tpl.info()
        assert info["factor_path"] == "rows" and info["slice_width"] == 2
        vm, va, _, status, _ = tpl.solve(*(d[k] for k in ("pd", "qd", "pg", "vset")))
        if precision == "fp64":
            upstream = [torch.as_tensor(x, device=device) for x in loss_grad(vm.cpu().numpy(), va.cpu().numpy())]
        g = tpl.adjoint(*upstream)
        torch.cuda.synchronize()
        assert int((status != 0).sum()) == 0
        out[precision] = [vm, va, *g]
        tpl.close()
    for i, (a, b) in enumerate(zip(out["fp64"], out["mixed"])):
        assert float((a - b).abs().max()) <= (1e-8 if i < 2 else 1e-6 * float(a.abs().max()))


# few wavefronts, all of which wait for each other's rows
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_tasks_of_a_narrow_workgroup_match_the_oracle(precision, device):
    net, sc = _grid(4200, 3)
    assert _path(net, 3, precision, block_threads=256) == "tasks"
    _check(net, sc, 1e-8, precision, device, (2,), 1, block_threads=256)
