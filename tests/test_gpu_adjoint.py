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
    import torch
    from paper_2607_18074_amd import _lib, api
    case = ac.case(i)
    irr_in, lmax, irr_out, K = case["sig"]
    plan, g = api.Plan(irr_in, lmax, irr_out, K), case["graph"]
    graph = api.Graph(_t(g.rowptr), _t(g.sender))
    args, gout = [_t(v) for v in (case["x"], g.evec, g.phi, case["W"])], _t(case["gout"])
    oa = (oc.Problem(irr_in, lmax, irr_out, K), case["x"], g.evec, g.phi, case["W"], g.rowptr, g.sender)
    ref = oc.bwd(*oa, case["gout"])
    adj = api.new_state(plan, graph)
    adj.fill_(float("nan"))
    _lib.profile_reset()
    _lib.profile_enable(True)
    api.conv_bwd(plan, graph, *args, gout, budget=0)
    api.conv_dbwd(plan, graph, *args, gout, t_gevec=_t(case["cot"]["evec"]))
    ran = set(_lib.profile_read())
    _lib.profile_enable(False)
    assert {"sobek_adj_E", "sobek_adj_dE"} <= ran and not ran & {"sobek_bwd_E", "sobek_dbwd_E_r", "sobek_dbwd_E"}
    for budget in (0, 1 << 21):   # one chunk of receivers; several
        _check(api.conv_bwd(plan, graph, *args, gout, budget=budget), ref, ("gx", "gevec", "gphi", "gW"), budget)
    _check(api.conv_bwd(plan, graph, *args, gout, adj_state=adj), ref, ("gx", "gevec", "gphi", "gW"), "kept")
    for which in ac.COTANGENTS:
        t = ac.cotangents(case, which)
        ref = oc.dbwd(*oa, case["gout"], t_gx=t["x"], t_gevec=t["evec"], t_gphi=t["phi"], t_gW=t["W"])
        for kw in (dict(), dict(adj_state=adj), dict(budget=1 << 21)):
            # memory that the outputs may be given: not zero by chance
            poison = [torch.full(s, float("nan"), device="cuda") for s in
                      ((g.N, plan.dim_out), (g.N, plan.dim_in), (g.E, 3), (g.E, K), (K, plan.n_weights))]
            del poison
            outs = api.conv_dbwd(plan, graph, *args, gout, *[_t(t[k]) for k in ("x", "evec", "phi", "W")], **kw)
            _check(outs, ref, ("g_gout", "g_x", "g_evec", "g_phi", "g_W"), (which, list(kw)))


def _run(degrees, i=0):
    from paper_2607_18074_amd import api
    case = ac.case(i, degrees)
    irr_in, lmax, irr_out, K = case["sig"]
    plan, g = api.Plan(irr_in, lmax, irr_out, K), case["graph"]
    graph = api.Graph(_t(g.rowptr), _t(g.sender))
    args, gout = [_t(v) for v in (case["x"], g.evec, g.phi, case["W"])], _t(case["gout"])
    oa = (oc.Problem(irr_in, lmax, irr_out, K), case["x"], g.evec, g.phi, case["W"], g.rowptr, g.sender)
    return api, plan, graph, case, args, gout, oa


def test_shares_of_a_receiver(gpu):
    """Two blocks a receiver, of which the first takes a second turn for edges 128 and on, the second has none of
    most receivers."""
    api, plan, graph, case, args, gout, oa = _run((129, 1) + (2,) * 300 + (64, 192, 65))
    _check(api.conv_bwd(plan, graph, *args, gout, need=(True, True, True, False)), oc.bwd(*oa, case["gout"]),
           ("gx", "gevec", "gphi"), "bwd")
    t = ac.cotangents(case, ("x", "evec"))
    ref = oc.dbwd(*oa, case["gout"], t_gx=t["x"], t_gevec=t["evec"])
    outs = api.conv_dbwd(plan, graph, *args, gout, _t(t["x"]), _t(t["evec"]), need=(False, True, True, True, False))
    _check(outs[1:4], ref, ("g_x", "g_evec", "g_phi"), "dbwd")


def _autograd_case():
    import torch
    api, plan, graph, case, args, _, oa = _run((3, 0, 20, 65))
    return torch, api, plan, graph, case, args, oa


@pytest.mark.parametrize("retain", [False, True])
def test_autograd_of_some_inputs(gpu, retain):
    """Inputs without gradients (phi, W), and a loss on one of the first gradients."""
    torch, api, plan, graph, case, args, oa = _autograd_case()
    x, ev = args[0].requires_grad_(), args[1].requires_grad_()
    gout = _t(case["gout"])
    m = api.tp_conv(plan, graph, *args, retain_state=retain)
    gx, gev = torch.autograd.grad(m, (x, ev), gout, create_graph=True)
    ref = oc.bwd(*oa, case["gout"])
    _check((gx, gev), ref, ("gx", "gevec"), "first")
    d = torch.autograd.grad((gev ** 2).sum(), (x, ev))
    ref = oc.dbwd(*oa, case["gout"], t_gevec=2 * gev.detach().cpu().numpy().astype(np.float64))
    _check(d, ref, ("g_x", "g_evec"), "second")


def test_autograd_without_cotangents(gpu):
    """A node downstream that returns no gradient: the double backward is called with none and gives zeros."""
    torch, api, plan, graph, case, args, oa = _autograd_case()

    class Drop(torch.autograd.Function):
        @staticmethod
        def forward(ctx, a):
            return a.clone()

        @staticmethod
        def backward(ctx, g):
            return None

    for a in args:
        a.requires_grad_()
    m = api.tp_conv(plan, graph, *args)
    g1 = torch.autograd.grad(m, args, _t(case["gout"]), create_graph=True)
    loss = sum(Drop.apply(v).sum() for v in g1)
    poison = [torch.full_like(a, float("nan")) for a in args]
    del poison
    for a, d in zip(args, torch.autograd.grad(loss, args, allow_unused=True)):
        assert d is None or float(d.abs().max()) == 0
