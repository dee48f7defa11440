"""The split channel products on the GPU, against the float64 oracle."""

import numpy as np
import pytest

from oracle import conv as oc
from tests import split_cases as sc
from tests.cases import max_rel

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _n(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("policy", ["all", "groups"])
@pytest.mark.parametrize("i", range(len(sc.CASES)), ids=sc.IDS)
def test_split_products(gpu, i, policy):
    from paper_2607_18074_amd import api
    case = sc.case(i)
    irr_in, lmax, irr_out, K = case["sig"]
    plan, g = api.Plan(irr_in, lmax, irr_out, K, policy=policy), case["graph"]
    graph = api.Graph(_t(g.rowptr), _t(g.sender))
    args = [_t(v) for v in (case["x"], g.evec, g.phi, case["W"])]
    oa = (oc.Problem(irr_in, lmax, irr_out, K), case["x"], g.evec, g.phi, case["W"], g.rowptr, g.sender)
    ref = oc.bwd(*oa, case["gout"])
    for budget in (0, 200_000):
        assert max_rel(_n(api.conv_fwd(plan, graph, *args, budget=budget)), oc.fwd(*oa)) <= sc.TOL
        for name, o in zip(("gx", "gevec", "gphi", "gW"), api.conv_bwd(plan, graph, *args, _t(case["gout"]), budget=budget)):
            assert max_rel(_n(o), ref[name]) <= sc.TOL, (budget, name)
