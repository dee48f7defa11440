"""The moment-form adjoint kernels on the CPU emulation build, against the float64 oracle."""

import numpy as np
import pytest

from oracle import conv as oc
from tests import adjoint_cases as ac
from tests.cases import max_rel
from tests.emu import build as emu_build


@pytest.mark.skipif(not emu_build.available(), reason="ROCm clang++ not found")
def test_adjoint():
    from tests.emu import harness as H
    case = ac.case(0, (0, 65))
    irr_in, lmax, irr_out, K = case["sig"]
    plan, g = H.Plan(irr_in, lmax, irr_out, K), case["graph"]
    graph = H.Graph(g.rowptr, g.sender)
    args, gout = [H.dev(v) for v in (case["x"], g.evec, g.phi, case["W"])], H.dev(case["gout"])
    oa = (oc.Problem(irr_in, lmax, irr_out, K), case["x"], g.evec, g.phi, case["W"], g.rowptr, g.sender)
    ref = oc.bwd(*oa, case["gout"])
    outs = H.conv_bwd(plan, graph, *args, gout, need=(True, True, True, False))
    for name, o in zip(("gx", "gevec", "gphi"), outs):
        assert max_rel(o.np(), ref[name]) <= ac.TOL, name
    t = case["cot"]
    ref = oc.dbwd(*oa, case["gout"], t_gx=t["x"], t_gevec=t["evec"], t_gphi=t["phi"], t_gW=t["W"])
    outs = H.conv_dbwd(plan, graph, *args, gout, *[H.dev(t[k]) for k in ("x", "evec", "phi", "W")],
                        need=(False, True, True, True, False))
    for name, o in zip(("g_x", "g_evec", "g_phi"), outs[1:4]):
        assert max_rel(o.np(), ref[name]) <= ac.TOL, name
        assert np.isfinite(o.np()).all()


@pytest.mark.skipif(not emu_build.available(), reason="ROCm clang++ not found")
def test_no_cotangent():
    """A double backward without cotangents writes zeros to every output asked for (the emulation fills new
    buffers with 0xff), in both layouts, with and without a kept adjoint state."""
    from tests.emu import harness as H
    case = ac.case(0, (0, 3))
    irr_in, lmax, irr_out, K = case["sig"]
    g = case["graph"]
    graph = H.Graph(g.rowptr, g.sender)
    args, gout = [H.dev(v) for v in (case["x"], g.evec, g.phi, case["W"])], H.dev(case["gout"])
    for layout in ("ir_mul", "mul_ir"):
        plan = H.Plan(irr_in, lmax, irr_out, K, layout=layout)
        adj = H.new_state(plan, graph)
        H.conv_bwd(plan, graph, *args, gout, need=(True, True, True, False), adj_state=adj)
        for kw in (dict(), dict(adj_state=adj)):
            outs = H.conv_dbwd(plan, graph, *args, gout, **kw)
            for name, o in zip(("g_gout", "g_x", "g_evec", "g_phi", "g_W"), outs):
                assert np.abs(o.np()).max() == 0, (layout, list(kw), name)
