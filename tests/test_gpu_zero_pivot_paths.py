"""The zero-pivot status on every HBM-resident factorisation: a bus that hangs on
a branch of zero admittance (its entries are in the pattern) has an all-zero
pivot block, which each path must report for every scenario, in the last, ragged
slice too, while the same network without that bus converges."""
import numpy as np
import pytest

from gpu_helpers import to_dev
from test_gpu_long_rows import _grid
from paper_2606_07099_amd.pf import ybus_from_branches

pytestmark = pytest.mark.gpu


def _with_dead_bus(net):
    """CSR Y_bus of the network and one more bus on a zero branch at its last one."""
    n = net.n_bus
    ip, ix, g, b = (np.asarray(a) for a in ybus_from_branches(n, net.f, net.t, net.r, net.x, net.bc))
    indptr = np.concatenate([ip, [ip[-1] + 3]]).astype(np.int32)
    indptr[n] += 1
    zero = np.zeros(3)
    return (n + 1, np.concatenate([net.bus_type, [0]]).astype(np.int32), indptr,
            np.concatenate([ix, [n], [n - 1, n]]).astype(np.int32), np.concatenate([g, zero]),
            np.concatenate([b, zero]))


@pytest.mark.parametrize("n,batch,precision,path,slice_width", [
    (300, 5, "fp64", "tasks", 1), (3200, 5, "mixed", "tasks", 1), (300, 5, "mixed", "levels", 1),
    (300, 513, "fp64", "levels", 2), (300, 1027, "mixed", "levels", 4), (300, 2049, "mixed", "levels", 8),
    (2300, 513, "fp64", "rows", 2), (1000, 1027, "fp64", "rows", 4), (300, 2049, "fp64", "rows", 8),
    (300, 4099, "mixed", "rows", 16)])
def test_a_zero_pivot_is_reported(n, batch, precision, path, slice_width, device):
    import torch
    from paper_2606_07099_amd import PFTemplate
    net, sc = _grid(n, batch)
    more = np.zeros((batch, 1))
    for dead in (False, True):
        if dead:
            tpl = PFTemplate(*_with_dead_bus(net), batch, precision=precision)
        else:
            tpl = PFTemplate.from_network(net, batch, precision=precision)
        info = tpl.info()
        assert info["factor_path"] == path and info["slice_width"] == slice_width
        x = [getattr(sc, k) for k in ("pd", "qd", "pg", "vset")]
        if dead:
            x = [np.concatenate([a, more + (i == 3)], axis=1) for i, a in enumerate(x)]
        status = tpl.solve(*[to_dev(a, device) for a in x])[3]
        torch.cuda.synchronize()
        assert bool((status == (3 if dead else 0)).all())
        tpl.close()
