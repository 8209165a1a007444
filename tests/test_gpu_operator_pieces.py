"""The operator refresh of networks beyond 4096 buses, whose per-bus state goes
through device memory: pf_operator_values grows its buffer from one call to the
next, pf_operator_values_static works in pieces of its fixed array (249 scenarios
of 4200 buses); both give the same values, those of the entry formulas."""
import numpy as np
import pytest

from gpu_helpers import to_dev
from test_gpu_operator_states import _compare, _network, j1_values
from test_zz_no_alloc import _values

pytestmark = pytest.mark.gpu


def test_growing_buffer_and_pieces(device):
    import torch
    from paper_2606_07099_amd import PFTemplate
    from paper_2606_07099_amd.pf import PF_OP_J1, PF_OP_J3T
    n = 4200
    net = _network(n)
    tpl = PFTemplate.from_network(net, 1)
    pat = tpl.operator_pattern(PF_OP_J1)
    for call, count in enumerate((2, 600, 300)):
        rng = np.random.default_rng(40 + call)
        vm, va = 1 + 0.03 * rng.standard_normal((count, n)), 0.2 * rng.standard_normal((count, n))
        tvm, tva = to_dev(vm, device), to_dev(va, device)
        for which in (PF_OP_J1, PF_OP_J3T):
            ref = _values(tpl, "pf_operator_values", which, tvm, tva)
            got = _values(tpl, "pf_operator_values_static", which, tvm, tva)
            torch.cuda.synchronize()
            assert not bool(torch.isnan(ref).any()) and torch.equal(got, ref), (which, count)
            if which == PF_OP_J1:
                for b in sorted({0, count // 2, min(count - 1, 248), min(count - 1, 249), count - 1}):
                    _compare(got.view(count, -1)[b].cpu().numpy(),
                             j1_values(net, pat["indptr"], pat["indices"], vm[b], va[b]))
