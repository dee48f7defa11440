"""The split channel products on the CPU emulation build, against the float64 oracle."""

import re

import pytest

from oracle import conv as oc
from tests import split_cases as sc
from tests.cases import max_rel
from tests.emu import build as emu_build


@pytest.mark.skipif(not emu_build.available(), reason="ROCm clang++ not found")
@pytest.mark.parametrize("policy", ["all", "groups"])
@pytest.mark.parametrize("i", range(len(sc.CASES)), ids=sc.IDS)
def test_split_products(i, policy):
    from tests.emu import harness as H
    case = sc.case(i)
    irr_in, lmax, irr_out, K = case["sig"]
    plan, g = H.Plan(irr_in, lmax, irr_out, K, policy=policy), case["graph"]
    graph = H.Graph(g.rowptr, g.sender)
    args = [H.dev(v) for v in (case["x"], g.evec, g.phi, case["W"])]
    oa = (oc.Problem(irr_in, lmax, irr_out, K), case["x"], g.evec, g.phi, case["W"], g.rowptr, g.sender)
    ref = oc.bwd(*oa, case["gout"])
    for budget in (0, 200_000):   # one chunk; many, the partials added up over them
        assert max_rel(H.conv_fwd(plan, graph, *args, budget=budget).np(), oc.fwd(*oa)) <= sc.TOL
        for name, o in zip(("gx", "gevec", "gphi", "gW"), H.conv_bwd(plan, graph, *args, H.dev(case["gout"]), budget=budget)):
            assert max_rel(o.np(), ref[name]) <= sc.TOL, (budget, name)


def test_only_what_runs_is_generated():
    """The streaming adjoint-state kernel: not where the split products (fp32, up to 128 wide) or the bf16 form run."""
    from paper_2607_18074_amd import _lib
    sig = ("8x0e+8x1o", 1, "132x0e+4x1o+32x1e", 8)
    for dtype, widths in (("f32", {"132"}), ("bf16_gemm", {"132", "4"})):
        src = _lib.plan_source(*sig, "ir_mul", "none", "uvw", dtype)
        assert set(re.findall(r"void sobek_gemm_sbar_c(\d+)\(", src)) == widths
