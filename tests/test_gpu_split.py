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


@pytest.mark.parametrize("sig,partials", [(("12x0e", 0, "16x0e", 3), False), (("8x0e+8x1o", 1, "8x0e+8x1o", 8), False),
                                          (("20x0e+12x1o", 1, "36x0e+72x1o", 5), True)])
def test_partials_only_where_shared(gpu, sig, partials):
    """Few receivers: reductions of at most 128 go straight into the output, longer ones are shared out and summed."""
    from paper_2607_18074_amd import _lib, api
    from tests.cases import make_case
    case = make_case(sig, 40, 200, 31)
    plan, g = api.Plan(*sig), case["graph"]
    graph = api.Graph(_t(g.rowptr), _t(g.sender))
    _lib.profile_reset()
    _lib.profile_enable(True)
    out = api.conv_fwd(plan, graph, *[_t(v) for v in (case["x"], g.evec, g.phi, case["W"])])
    ran = set(_lib.profile_read())
    _lib.profile_enable(False)
    assert "sobek_sp3_sa" in ran and ("sobek_sp3_red" in ran) == partials
    ref = oc.fwd(oc.Problem(*sig), case["x"], g.evec, g.phi, case["W"], g.rowptr, g.sender)
    assert max_rel(_n(out), ref) <= sc.TOL
