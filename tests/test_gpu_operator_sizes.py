"""Operator value refresh at the edges of its launch rules: one and two
scenarios per workgroup (a last workgroup with one of two), values split over
several workgroups, both workgroup sizes, against the oracle's dense operators
at random states."""
import numpy as np
import pytest

from gpu_helpers import random_states, to_dev
from gen.grids import make_case
from oracle.operators import operators
from oracle.ybus import ybus_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,count", [("c0", 1), ("c1", 511), ("c1", 513), ("c2", 3), ("c2", 513)])
def test_operator_values_at_the_edges_of_the_launch_rules(name, count, device):
    import torch
    from paper_2606_07099_amd import PFTemplate
    spec, net, sc = make_case(name, batch=1)
    tpl = PFTemplate.from_network(net, 1)
    vm, va = random_states(net, count, seed=33)
    vm_d, va_d = to_dev(vm, device), to_dev(va, device)
    Y = ybus_of(net)
    for which, key in {0: "J", 1: "J1", 2: "J1T", 3: "J2T", 4: "J3T"}.items():
        pat = tpl.operator_pattern(which)
        rows = np.repeat(np.arange(pat["n_rows"]), np.diff(pat["indptr"]))
        out = tpl.operator(which, vm_d, va_d)
        out.values().fill_(float("nan"))
        tpl.operator(which, vm_d, va_d, out=out)
        torch.cuda.synchronize()
        vals = out.values().cpu().numpy().reshape(count, -1)
        assert not np.isnan(vals).any(), key
        for b in sorted({0, count - 1}):
            ref = operators(Y, net.bus_type, vm[b], va[b])[key]
            # sums of a few products of values below the largest entry: 1e-12 of it
            assert np.abs(vals[b] - ref[rows, pat["indices"]]).max() <= 1e-12 * np.abs(ref).max(), (key, b)
