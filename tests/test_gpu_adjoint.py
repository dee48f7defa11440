"""The moment-form adjoint kernels on the GPU, against the float64 oracle."""

import numpy as np
import pytest

from oracle import conv as oc
from tests import adjoint_cases as ac
from tests.cases import max_rel

pytestmark = pytest.mark.gpu


def _t(a):
    import torch
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _check(outs, ref, names, what):
    for name, o in zip(names, outs):
        got = o.detach().cpu().numpy()
        if np.abs(ref[name]).max() == 0:
            assert np.abs(got).max() == 0, (what, name)
        else:
            assert max_rel(got, ref[name]) <= ac.TOL, (what, name)


@pytest.mark.parametrize("i", range(len(ac.SIGS)), ids=ac.IDS)
def test_adjoint(gpu, i):
    from paper_2607_18074_amd import api
    case = ac.case(i)
    irr_in, lmax, irr_out, K = case["sig"]
    plan, g = api.Plan(irr_in, lmax, irr_out, K), case["graph"]
    graph = api.Graph(_t(g.rowptr), _t(g.sender))
    args, gout = [_t(v) for v in (case["x"], g.evec, g.phi, case["W"])], _t(case["gout"])
    oa = (oc.Problem(irr_in, lmax, irr_out, K), case["x"], g.evec, g.phi, case["W"], g.rowptr, g.sender)
    ref = oc.bwd(*oa, case["gout"])
    adj = api.new_state(plan, graph)
    adj.fill_(float("nan"))
    for budget in (0, 1 << 21):   # one chunk of receivers; several
        _check(api.conv_bwd(plan, graph, *args, gout, budget=budget), ref, ("gx", "gevec", "gphi", "gW"), budget)
    _check(api.conv_bwd(plan, graph, *args, gout, adj_state=adj), ref, ("gx", "gevec", "gphi", "gW"), "kept")
    for which in ac.COTANGENTS:
        t = ac.cotangents(case, which)
        ref = oc.dbwd(*oa, case["gout"], t_gx=t["x"], t_gevec=t["evec"], t_gphi=t["phi"], t_gW=t["W"])
        for kw in (dict(), dict(adj_state=adj), dict(budget=1 << 21)):
            outs = api.conv_dbwd(plan, graph, *args, gout, *[_t(t[k]) for k in ("x", "evec", "phi", "W")], **kw)
            _check(outs, ref, ("g_gout", "g_x", "g_evec", "g_phi", "g_W"), (which, list(kw)))
