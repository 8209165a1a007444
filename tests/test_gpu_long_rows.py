"""Networks with long rows on the HBM-resident paths, against the dense oracle:
a row whose task record and buffer take the share of several wavefronts, so that
only some of them take tasks, with wide and narrow workgroups."""
import numpy as np
import pytest

from test_gpu_rows import _check
from test_host_plan import hubs
from gen.grids import Scenarios

pytestmark = pytest.mark.gpu


def _scenarios(net, batch, seed=3):
    rng = np.random.default_rng(seed)
    pq = np.asarray(net.bus_type) == 0
    pd = np.where(pq, rng.uniform(1e-5, 2e-5, (batch, net.n_bus)), 0.0)
    return Scenarios(pd, 0.3 * pd, np.zeros_like(pd), np.ones_like(pd))


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
