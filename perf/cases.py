"""The measured cases: what a program that trains or runs an equivariant interatomic model has the
convolution do, through `paper_2607_18074_amd.api`.

A case is one layer's call (or the calls of one step) on one graph: an operator signature, a kind of
graph, its size and mean degree, and the operation:

  fwd     the forward alone (energies)
  forces  forward, then the gradients for forces (x, edge vectors, radial features; no weights)
  fwdbwd  forward keeping its state and the whole backward that reads it (training without forces)
  bwd     the whole backward with nothing kept
  dbwd    the double backward for the cotangent of a loss on the edge-vector gradients
  step    the three passes of a force-matching step with the receiver and adjoint states kept
  train   the same step through autograd (`tp_conv`), the loss on all the gradients that a
          multi-layer model passes on (x, edge vectors, radial features)

Graphs are batches of ragged molecules (every pair of one molecule within the cutoff) or one box of
points (every pair within the cutoff, node ids in no spatial order); the cutoff gives the mean degree.  `exact` evaluates the same
operator in float64 with plain torch: real spherical harmonics in closed form, coupling tensors as the
invariant of three rotations, per-edge weights and messages materialised, derivatives by autograd.
"""
import functools
import math

import torch

from paper_2607_18074_amd import api

GIB = 1 << 30

# (input irreps = output irreps unless given, lmax, K) of the workloads and profiles of the benchmark
SIGNATURES = {
    "small": ("32x0e+32x1o+32x2e", 2, None, 8),
    "medium": ("64x0e+64x1o+64x1e+64x2e", 3, None, 16),
    "wide": ("128x0e+128x1o+128x2e+64x3o", 3, None, 16),
    "tiny": ("8x0e+8x1o", 1, None, 8),
    "odd": ("3x0e+5x1o+2x2e+1x0o", 1, "4x0e+3x1o+2x2e+1x3e", 4),
    "128/64": ("128x0e+64x1o", 1, None, 16),
    "128/64/64": ("128x0e+64x1o+64x2e", 2, None, 16),
    "64/64/64": ("64x0e+64x1o+64x2e", 2, None, 16),
    "64/32/32/32": ("64x0e+32x1o+32x2e+32x3o", 3, None, 16),
    "128/128/128": ("128x0e+128x1o+128x2e", 2, None, 16),
    "64/64/64/64": ("64x0e+64x1o+64x2e+64x3o", 3, None, 16),
    "256/256": ("256x0e+256x1o", 1, None, 16),
}

BASE = dict(mode="uvw", layout="ir_mul", norm="none", dtype="f32", budget=0)


def _case(name, sig, op, graph, nodes, degree, **kw):
    c = dict(BASE, sig=sig, op=op, graph=graph, nodes=nodes, degree=degree, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small molecule's energy: launches and latency
        _case("molecule_fwd", "tiny", "fwd", "batch", 64, 16),
        # one molecule's energy and forces, a molecular-dynamics step: latency, few receivers
        _case("molecule_forces", "small", "forces", "batch", 57, 20),
        # odd multiplicities, mul_ir layout and path normalisation, a ragged batch, trained on forces
        _case("odd_train", "odd", "train", "batch", 1171, 13, layout="mul_ir", norm="fan_in"),
        # a box of 2,000 atoms, energy and forces
        _case("small_forces", "small", "forces", "radius", 2000, 32),
        # a batch of molecules through one of the paper's profiles, forward
        _case("batch_fwd", "128/64", "fwd", "batch", 27776, 29),
        # a batch of molecules, a force-matching step through autograd, nothing kept
        _case("batch_train", "64/64/64", "train", "batch", 5171, 29),
        # a box of 20,000 atoms: each pass alone within the default workspace
        _case("medium_fwd", "medium", "fwd", "radius", 20000, 50),
        _case("medium_bwd", "medium", "bwd", "radius", 20000, 50),
        _case("medium_dbwd", "medium", "dbwd", "radius", 20000, 50),
        # wide features, reduced-precision channel products, training without forces
        _case("wide_bf16_fwdbwd", "wide", "fwdbwd", "radius", 12000, 40, dtype="bf16_gemm", budget=8 * GIB),
        # channelwise mixing, training without forces
        _case("uvu_fwdbwd", "128/128/128", "fwdbwd", "batch", 11008, 29, mode="uvu"),
        # the largest: a force-matching step on a box of 200,000 atoms with both states kept
        _case("stress_step", "small", "step", "radius", 200000, 80, budget=8 * GIB),
    ]


# what a drawn case is drawn from: signature, options, operations, most nodes
_FAMILIES = [
    ("tiny", {}, ("fwd", "forces", "bwd", "train"), 4000),
    ("small", {}, ("fwd", "forces", "bwd", "dbwd", "step", "train"), 60000),
    ("small", dict(dtype="bf16_gemm"), ("fwd", "fwdbwd"), 60000),
    ("odd", dict(layout="mul_ir", norm="fan_in"), ("fwd", "bwd", "dbwd", "train"), 4000),
    ("odd", {}, ("fwd", "forces", "bwd"), 4000),
    ("128/64", {}, ("fwd", "bwd", "dbwd", "step"), 30000),
    ("128/64/64", {}, ("fwd", "bwd", "dbwd"), 5000),
    ("64/64/64", {}, ("fwd", "forces", "bwd", "step", "train"), 6000),
    ("64/32/32/32", {}, ("fwd", "bwd", "dbwd"), 6000),
    ("medium", {}, ("fwd", "bwd", "dbwd", "step", "train"), 5000),
    ("wide", {}, ("fwd", "fwdbwd"), 1200),
    ("wide", dict(dtype="bf16_gemm"), ("fwd", "fwdbwd"), 2000),
    ("128/128/128", dict(mode="uvu"), ("fwd", "bwd", "dbwd", "fwdbwd"), 8000),
    ("64/64/64/64", dict(mode="uvu"), ("fwd", "bwd", "dbwd"), 8000),
    ("256/256", dict(mode="uvu"), ("fwd", "bwd", "dbwd"), 8000),
]


def draw(rng):
    sig, opts, ops, most = rng.choice(_FAMILIES)
    nodes = int(round(math.exp(rng.uniform(math.log(20), math.log(most)))))
    degree = int(round(math.exp(rng.uniform(math.log(4), math.log(100)))))
    graph = rng.choice(("batch", "radius"))
    if graph == "batch":
        degree = min(degree, 40)
    degree = max(1, min(degree, nodes // 3))
    budget = rng.choice((0, 0, 128 << 20, 4 * GIB))
    return _case(None, sig, rng.choice(ops), graph, nodes, degree, **dict(opts, budget=budget))


# ---------------------------------------------------------------------------
# the operator's static description
# ---------------------------------------------------------------------------

def _irreps(spec):
    out = []
    for part in spec.split("+"):
        mul, rest = part.split("x")
        out.append((int(mul), int(rest[:-1]), 1 if rest[-1] == "e" else -1))
    return out


class _Op:
    """Paths (input, SH order, output, weight offset) and sizes of a case's operator."""

    def __init__(self, case):
        spec_in, self.lmax, spec_out, self.K = SIGNATURES[case["sig"]]
        self.spec_in, self.spec_out = spec_in, spec_out or spec_in
        self.ins, self.outs = _irreps(self.spec_in), _irreps(self.spec_out)
        self.uvu = case["mode"] == "uvu"
        self.paths, self.n_w, self.fan = [], 0, {}
        for a, (ca, la, pa) in enumerate(self.ins):
            for ls in range(self.lmax + 1):
                for c, (cc, lc, pc) in enumerate(self.outs):
                    if abs(la - ls) <= lc <= la + ls and pc == pa * (-1) ** ls:
                        self.paths.append((a, ls, c, self.n_w))
                        self.n_w += ca if self.uvu else ca * cc
                        self.fan[c] = self.fan.get(c, 0) + (1 if self.uvu else ca)
        self.dim_in = sum(c * (2 * l + 1) for c, l, _ in self.ins)
        self.dim_out = sum(c * (2 * l + 1) for c, l, _ in self.outs)

    def weight_std(self, device):
        s = torch.empty(self.n_w, device=device)
        for a, _, c, off in self.paths:
            s[off:off + self.ins[a][0] * (1 if self.uvu else self.outs[c][0])] = (self.K * self.fan[c]) ** -0.5
        return s


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

R_CUT = 5.0


def _pairs(pos, group, lo, hi, most):
    """(receiver, sender, squared distance) of the ordered pairs closer than `most`; the 2,048 rows of
    block b meet the columns [lo[b], hi[b]), pairs of two groups aside."""
    rs, ss, ds = [], [], []
    n = 2048
    for b in range(0, pos.shape[0], n):
        p, q = pos[b:b + n], pos[lo[b // n]:hi[b // n]]
        d2 = ((p[:, None, :] - q[None, :, :]) ** 2).sum(-1)
        m = (d2 < most ** 2) & (d2 > 0)
        if group is not None:
            m &= group[b:b + n, None] == group[None, lo[b // n]:hi[b // n]]
        r, s = m.nonzero(as_tuple=True)
        rs.append(r + b)
        ss.append(s + lo[b // n])
        ds.append(d2[r, s])
    return torch.cat(rs), torch.cat(ss), torch.cat(ds)


def _points(index, side, gen):
    """One point per site of a cubic lattice of `side` sites a side, moved within its cell (atoms keep apart)."""
    site = torch.stack((index % side, index // side % side, index // (side * side)), 1).double()
    return site + 0.8 * torch.rand(len(index), 3, generator=gen, device=index.device, dtype=torch.float64)


def _graph(case, gen, dev):
    """Receiver-sorted CSR and float64 edge vectors of the case's graph: the closest pairs, as many as
    the mean degree asks for, in units in which the furthest of them is at the cutoff."""
    N, degree = case["nodes"], case["degree"]
    E = 2 * ((N * degree + 1) // 2)
    blocks = range(0, N, 2048)
    if case["graph"] == "batch":
        # molecules of 64 to 192 nodes (a smaller batch is one molecule), each in a cube of its own
        sizes, left = [], N
        while left > 0:
            m = int(torch.randint(64, 193, (1,), generator=gen, device=dev))
            m = left if left - m < 64 else m
            sizes.append(m)
            left -= m
        sz = torch.tensor(sizes, device=dev)
        group = torch.repeat_interleave(torch.arange(len(sizes), device=dev), sz)
        last = torch.cumsum(sz, 0)
        within = torch.arange(N, device=dev) - (last - sz)[group]
        pos = _points(within, torch.ceil(sz.double().pow(1 / 3)).long()[group], gen)
        ends = last.tolist()
        lo, hi, g0, g1 = [], [], 0, 0
        for b in blocks:
            while ends[g0] <= b:
                g0 += 1
            while ends[g1] < min(N, b + 2048):
                g1 += 1
            lo.append(ends[g0 - 1] if g0 else 0)
            hi.append(ends[g1])
        r, s, d2 = _pairs(pos, group, lo, hi, math.inf)
    else:
        shuffled = torch.randperm(N, generator=gen, device=dev)
        pos = _points(shuffled, torch.tensor(math.ceil(N ** (1 / 3) - 1e-9), device=dev), gen)
        order = torch.argsort(pos[:, 2])
        p = pos[order]
        lo, hi, most = [0] * len(blocks), [N] * len(blocks), math.inf
        if N > 4096:  # a box this large: twice the volume that holds `degree` points, slab by slab
            most = (degree / (4 / 3 * math.pi)) ** (1 / 3) * 1.3
            z = p[:, 2].contiguous()
            first = torch.tensor(list(blocks), device=dev)
            last = torch.clamp(first + 2047, max=N - 1)
            lo = torch.searchsorted(z, z[first] - most).tolist()
            hi = torch.searchsorted(z, z[last] + most).tolist()
        r, s, d2 = _pairs(p, None, lo, hi, most)
        r, s = order[r], order[s]
    cut2 = torch.sort(d2).values[E - 1]
    keep = d2 <= cut2
    key = torch.sort(r[keep] * N + s[keep]).values
    r, s = key // N, key % N
    evec = (pos[s] - pos[r]) * (R_CUT / cut2.sqrt())
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device=dev)
    rowptr[1:] = torch.cumsum(torch.bincount(r, minlength=N), 0).int()
    return rowptr, s.int(), evec


def _radial(evec, K, p=6):
    """K Bessel functions of the edge length under the polynomial cutoff envelope."""
    d = evec.norm(dim=1)
    t = d / R_CUT
    u = 1 - (p + 1) * (p + 2) / 2 * t ** p + p * (p + 2) * t ** (p + 1) - p * (p + 1) / 2 * t ** (p + 2)
    n = torch.arange(1, K + 1, device=d.device, dtype=d.dtype)
    return math.sqrt(2 / R_CUT) * torch.sin(n * math.pi * t[:, None]) / d[:, None] * u[:, None]


def _inputs(case, seed, dev):
    op = _Op(case)
    gen = torch.Generator(device=dev).manual_seed(seed)
    rowptr, sender, evec = _graph(case, gen, dev)
    E = sender.shape[0]

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev)

    t = dict(rowptr=rowptr, sender=sender, evec=evec.float(), phi=_radial(evec, op.K).float(),
             x=normal(case["nodes"], op.dim_in), W=normal(op.K, op.n_w) * op.weight_std(dev),
             gout=normal(case["nodes"], op.dim_out))
    if case["op"] == "dbwd":
        t["t_gevec"] = normal(E, 3)
    return op, t


# ---------------------------------------------------------------------------
# the framework's calls
# ---------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _plan(sig, mode, layout, norm, dtype):
    spec_in, lmax, spec_out, K = SIGNATURES[sig]
    return api.Plan(spec_in, lmax, spec_out or spec_in, K, layout=layout, normalization=norm, mode=mode, dtype=dtype)


def prepare(case, seed):
    dev = torch.device("cuda")
    op, t = _inputs(case, seed, dev)
    plan = _plan(case["sig"], case["mode"], case["layout"], case["norm"], case["dtype"])
    graph = api.Graph(t.pop("rowptr"), t.pop("sender"))
    state = dict(t, op=case["op"], plan=plan, graph=graph, budget=case["budget"])
    passes = {"fwd": ("fwd",), "forces": ("fwd", "bwd"), "fwdbwd": ("fwd", "bwd"), "bwd": ("bwd",),
              "dbwd": ("dbwd",), "step": ("fwd", "bwd", "dbwd"), "train": ("fwd", "bwd", "dbwd")}[case["op"]]
    for p in passes:
        graph.workspace(plan, p, 0 if case["op"] == "train" else case["budget"])
    state["S"] = None       # the channelwise backward reads no receiver state: nothing is kept for it
    if case["op"] in ("fwdbwd", "step") and case["mode"] == "uvw":
        state["S"] = api.new_state(plan, graph)
    if case["op"] == "step":
        state["Sbar"] = api.new_state(plan, graph)
    if case["op"] == "train":
        for k in ("x", "evec", "phi", "W"):
            state[k].requires_grad_()
    return state


def run(s):
    op, plan, graph, b = s["op"], s["plan"], s["graph"], s["budget"]
    ins = (s["x"], s["evec"], s["phi"], s["W"])
    if op == "fwd":
        return api.conv_fwd(plan, graph, *ins, budget=b)
    if op == "forces":
        out = api.conv_fwd(plan, graph, *ins, budget=b)
        return out, api.conv_bwd(plan, graph, *ins, s["gout"], need=(True, True, True, False), budget=b)[:3]
    if op == "fwdbwd":
        out = api.conv_fwd(plan, graph, *ins, budget=b, state=s["S"])
        return out, api.conv_bwd(plan, graph, *ins, s["gout"], budget=b, state=s["S"])
    if op == "bwd":
        return api.conv_bwd(plan, graph, *ins, s["gout"], budget=b)
    if op == "dbwd":
        return api.conv_dbwd(plan, graph, *ins, s["gout"], t_gevec=s["t_gevec"], budget=b)
    if op == "step":
        out = api.conv_fwd(plan, graph, *ins, budget=b, state=s["S"])
        g = api.conv_bwd(plan, graph, *ins, s["gout"], budget=b, state=s["S"], adj_state=s["Sbar"])
        return out, g, api.conv_dbwd(plan, graph, *ins, s["gout"], t_gevec=g[1] * 2, budget=b, adj_state=s["Sbar"])
    out = api.tp_conv(plan, graph, *ins)
    energy = (out * s["gout"]).sum()
    g = torch.autograd.grad(energy, ins[:3], create_graph=True)
    loss = sum((v * v).sum() for v in g)
    return out.detach(), [v.detach() for v in g], torch.autograd.grad(loss, ins)


# ---------------------------------------------------------------------------
# the work of a pass
# ---------------------------------------------------------------------------

def work(case):
    """Operands once, results once; operations of the reassociated evaluation: per edge the state update
    (2 K per state element) and the coupling (2 per non-zero coefficient and channel), per receiver the
    channel products.  A uvu edge forms its path weights (2 K per weight) and scales the coupled values."""
    op = _Op(case)
    N, K = case["nodes"], op.K
    E = 2 * ((N * case["degree"] + 1) // 2)
    SD = NZ = G = 0
    for a, ls, c, _ in op.paths:
        ca, la, _p = op.ins[a]
        cc, lc, _p = op.outs[c]
        SD += ca * (2 * lc + 1)
        NZ += ca * int((_coupling(la, ls, lc).abs() > 1e-12).sum())
        G += ca * (2 * lc + 1) * cc
    if op.uvu:
        fwd = E * (2 * K * op.n_w + 2 * NZ + 2 * SD)
        bwd = E * (4 * K * op.n_w + 6 * NZ + 4 * SD)
        dbwd = E * (6 * K * op.n_w + 6 * NZ + 6 * SD)
    else:
        fwd = E * (2 * K * SD + 2 * NZ) + 2 * N * K * G
        bwd = E * (4 * K * SD + 6 * NZ) + 4 * N * K * G
        dbwd = E * (6 * K * SD + 6 * NZ) + 6 * N * K * G
    w, edge, nx, no = 4 * K * op.n_w, 4 * E * (3 + K), 4 * N * op.dim_in, 4 * N * op.dim_out
    read = 4 * (E + N) + edge + nx + w          # graph, edges, features, weights
    b = {"fwd": read + no, "bwd": read + no + edge + nx + w}
    b["dbwd"] = b["bwd"] + 4 * 3 * E + no
    forces = b["bwd"] - w
    flops = {"fwd": fwd, "forces": fwd + bwd - (0 if op.uvu else 2 * N * K * G), "fwdbwd": fwd + bwd, "bwd": bwd,
             "dbwd": dbwd, "step": fwd + bwd + dbwd, "train": fwd + bwd + dbwd}
    nbytes = {"fwd": b["fwd"], "forces": b["fwd"] + forces, "fwdbwd": b["fwd"] + b["bwd"], "bwd": b["bwd"],
              "dbwd": b["dbwd"], "step": sum(b.values()), "train": sum(b.values()) + 4 * E * K + nx}
    return {"bytes": nbytes[case["op"]], "flops": flops[case["op"]]}


def tolerance(case):
    # bf16 rounding of the channel products' operands (2.3e-3 measured); fp32 sums elsewhere (up to 9e-7)
    return {"rel": 1e-2, "max": 0.2} if case["dtype"] == "bf16_gemm" else {"rel": 5e-6, "max": 5e-4}


# ---------------------------------------------------------------------------
# the operator in float64
# ---------------------------------------------------------------------------

def _harmonics(u, l):
    """Real spherical harmonics of unit vectors, sum of squares 2l + 1, m = -l .. l."""
    x, y, z = u.unbind(-1)
    r = math.sqrt
    if l == 0:
        v = [torch.ones_like(x)]
    elif l == 1:
        v = [r(3) * y, r(3) * z, r(3) * x]
    elif l == 2:
        v = [r(15) * x * y, r(15) * y * z, r(5) / 2 * (3 * z * z - 1), r(15) * x * z, r(15) / 2 * (x * x - y * y)]
    else:
        v = [r(35 / 8) * y * (3 * x * x - y * y), r(105) * x * y * z, r(21 / 8) * y * (5 * z * z - 1),
             r(7) / 2 * z * (5 * z * z - 3), r(21 / 8) * x * (5 * z * z - 1), r(105) / 2 * z * (x * x - y * y),
             r(35 / 8) * x * (x * x - 3 * y * y)]
    return torch.stack(v, -1)


@functools.lru_cache(maxsize=None)
def _coupling(l1, l2, l3):
    """Real coupling tensor: the one invariant of three rotations, norm sqrt(2 l3 + 1), first entry positive."""
    gen = torch.Generator().manual_seed(1)
    u = torch.nn.functional.normalize(torch.randn(64, 3, generator=gen, dtype=torch.float64), dim=1)
    rows = []
    for _ in range(3):
        q, _r = torch.linalg.qr(torch.randn(3, 3, generator=gen, dtype=torch.float64))
        q = q * torch.linalg.det(q)
        d = [torch.linalg.lstsq(_harmonics(u, l), _harmonics(u @ q.T, l)).solution.T for l in (l1, l2, l3)]
        rows.append(torch.kron(torch.kron(d[0].contiguous(), d[1].contiguous()), d[2].contiguous()))
    eye = torch.eye(rows[0].shape[0], dtype=torch.float64)
    v = torch.linalg.svd(torch.cat([m - eye for m in rows]))[2][-1]
    v = torch.where(v.abs() < 1e-10, torch.zeros_like(v), v)
    v = v * math.sqrt(2 * l3 + 1) / v.norm() * torch.sign(v[v != 0][0])
    return v.reshape(2 * l1 + 1, 2 * l2 + 1, 2 * l3 + 1)


def _blocks(v, irreps, mul_ir):
    """Irrep blocks of node rows as [n][multiplicity][m]."""
    out, off = [], 0
    for c, l, _ in irreps:
        b = v[:, off:off + c * (2 * l + 1)]
        out.append(b.reshape(-1, c, 2 * l + 1) if mul_ir else b.reshape(-1, 2 * l + 1, c).transpose(1, 2))
        off += c * (2 * l + 1)
    return out


def _conv64(case, op, x, evec, phi, W, recv, send, n):
    """Rows [0, n) of the convolution: edges (recv, send) with per-edge weights and messages materialised."""
    mul_ir = case["layout"] == "mul_ir"
    u = evec / evec.norm(dim=1, keepdim=True)
    Y = [_harmonics(u, l) for l in range(op.lmax + 1)]
    xs = [b[send] for b in _blocks(x, op.ins, mul_ir)]
    outs = [None] * len(op.outs)
    for a, ls, c, off in op.paths:
        ca, la, _ = op.ins[a]
        cc, lc, _ = op.outs[c]
        Q = _coupling(la, ls, lc).to(x.device)
        if case["norm"] == "fan_in":
            Q = Q * op.fan[c] ** -0.5
        M = (Y[ls] @ Q.permute(1, 0, 2).reshape(2 * ls + 1, -1)).reshape(-1, 2 * la + 1, 2 * lc + 1)
        C = torch.bmm(xs[a], M)
        w = phi @ W[:, off:off + ca * (1 if op.uvu else cc)]
        msg = w[:, :, None] * C if op.uvu else torch.bmm(w.reshape(-1, ca, cc).transpose(1, 2), C)
        part = torch.zeros(n, cc, 2 * lc + 1, dtype=x.dtype, device=x.device).index_add(0, recv, msg)
        outs[c] = part if outs[c] is None else outs[c] + part
    rows = []
    for c, (cc, lc, _) in enumerate(op.outs):
        o = outs[c] if outs[c] is not None else torch.zeros(n, cc, 2 * lc + 1, dtype=x.dtype, device=x.device)
        rows.append((o if mul_ir else o.transpose(1, 2)).reshape(n, -1))
    return torch.cat(rows, 1)


def exact(case, seed):
    op = _Op(case)
    kind = case["op"]
    heavy = {"fwd": 1, "forces": 3, "fwdbwd": 3, "bwd": 3, "dbwd": 8, "step": 10, "train": 10}[kind]
    if case["nodes"] * case["degree"] * float(op.n_w) * heavy > 1.2e12:
        return None
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    _, t = _inputs(case, seed, dev)
    rowptr, send = t["rowptr"].long(), t["sender"].long()
    N = case["nodes"]
    x, evec, phi, W, gout = (t[k].double() for k in ("x", "evec", "phi", "W", "gout"))
    deg = rowptr[1:] - rowptr[:-1]
    recv = torch.repeat_interleave(torch.arange(N, device=dev), deg)
    first = kind in ("forces", "fwdbwd", "bwd", "step", "train")
    second = kind in ("dbwd", "step", "train")
    out = torch.zeros(N, op.dim_out, dtype=torch.float64, device=dev)
    g1 = [torch.zeros_like(v) for v in (x, evec, phi, W)]
    g2 = [torch.zeros_like(v) for v in (x, evec, phi, W)]
    g_gout = torch.zeros_like(gout)
    # the loss of a training step is on the whole x-gradient: its cotangent is known only after every chunk
    passes = [0, 1] if second and kind != "dbwd" else ([1] if kind == "dbwd" else [0])
    chunk = max(1, int(6e7 / op.n_w))           # edges of a chunk of receivers
    ptr = rowptr.tolist()
    for p in passes:
        b = 0
        while b < N:
            e = b + 1
            while e < N and ptr[e + 1] - ptr[b] <= chunk:
                e += 1
            es = slice(ptr[b], ptr[e])
            leaf = [v.detach().requires_grad_(first or second) for v in (x, evec[es], phi[es], W)]
            go = gout[b:e].detach().requires_grad_(second)
            o = _conv64(case, op, *leaf, recv[es] - b, send[es], e - b)
            if p == 0:
                out[b:e] = o.detach()
            if first and p == 0:
                d = torch.autograd.grad((o * go).sum(), leaf)
                g1[0] += d[0]
                g1[1][es], g1[2][es] = d[1], d[2]
                g1[3] += d[3]
            if second and p == 1:
                d = torch.autograd.grad((o * go).sum(), leaf[:3], create_graph=True)
                if kind == "dbwd":
                    loss = (d[1] * t["t_gevec"][es].double()).sum()
                elif kind == "step":
                    loss = (d[1] * 2 * g1[1][es]).sum()
                else:
                    loss = sum((v * 2 * c).sum() for v, c in zip(d, (g1[0], g1[1][es], g1[2][es])))
                d = torch.autograd.grad(loss, [go] + leaf, allow_unused=True)
                d = [torch.zeros_like(v) if g is None else g for g, v in zip(d, [go] + leaf)]
                g_gout[b:e] = d[0]
                g2[0] += d[1]
                g2[1][es], g2[2][es] = d[2], d[3]
                g2[3] += d[4]
            b = e
    if kind == "fwd":
        return out
    if kind == "forces":
        return out, tuple(g1[:3])
    if kind == "fwdbwd":
        return out, tuple(g1)
    if kind == "bwd":
        return tuple(g1)
    if kind == "dbwd":
        return (g_gout, *g2)
    if kind == "step":
        return out, tuple(g1), (g_gout, *g2)
    return out, g1[:3], tuple(g2)
