"""The measured work of the framework: what a Newton-Krylov program has it do.

Every case goes through the public Python entry points on the synthetic
Newton systems of `synth` (element blocks and trace right-hand sides drawn
on the device from the seed), for structured meshes of nx x ny x nz elements
of degree p (n = 20 (p+1)^3 local dofs, b = 5 (p+1)^2 dofs a face).  A case
names the kind of work, the mesh, the degree and the precision:

  condense   static condensation of every element (the bulk of a Newton step)
  factor     assembly of K and R, BILU(0) of K (after every condensation)
  iedg       the trace system on shared trace nodes (5 x 5 node blocks):
             assembly, BILU(0), GMRES
  rhs        a further right-hand side with the retained factors: FP64, or
             low-precision factors with FP64 refinement (a serving hit)
  residual   the FP64 residual of the uncondensed system (each refinement step)
  newton     the whole Newton-step solve, FP64 or mixed FP32
  batch      several meshes of uneven size and degree in one captured graph
"""
import functools
import math

import numpy as np
import torch

from paper_1605_01020_amd import api, F64, F32, BF16
from paper_1605_01020_amd.autotune import apply_tuning
from paper_1605_01020_amd.batch import BatchGroup, Simulation
from paper_1605_01020_amd.solver import NewtonStepSolver
from synth import ElementSpec, StructuredHexMesh
from synth import device as sdev
from synth.matrices import MeshCase

PREC = {"f64": F64, "f32": F32, "bf16": BF16}


def _case(name, kind, dims, p, prec, **more):
    c = {"kind": kind, "nx": dims[0], "ny": dims[1], "nz": dims[2], "p": p, "prec": prec}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a handful of small elements, latency and launches
        _case("condense_f64_2x2x2_p1", "condense", (2, 2, 2), 1, "f64"),
        # the small FP64 simulation: fewer elements than the GPU has CUs
        _case("condense_f64_4x4x4_p2", "condense", (4, 4, 4), 2, "f64"),
        # an ordinary simulation of the serving mix, FP32 factors
        _case("condense_f32_12x12x6_p3", "condense", (12, 12, 6), 3, "f32"),
        # the largest elements, BF16 operands
        _case("condense_bf16_6x6x6_p4", "condense", (6, 6, 6), 4, "bf16"),
        # trace set-up after a condensation, FP32 blocks of 80 (odd mesh)
        _case("factor_f32_9x7x5_p3", "factor", (9, 7, 5), 3, "f32"),
        # the IEDG numbering of the same element matrices, 5 x 5 blocks
        _case("iedg_f64_4x4x4_p2", "iedg", (4, 4, 4), 2, "f64"),
        # a further right-hand side of the small FP64 simulation
        _case("rhs_f64_4x4x4_p2", "rhs", (4, 4, 4), 2, "f64"),
        # a serving hit: low-precision factors, FP64 refinement
        _case("rhs_f32_8x8x4_p3", "rhs", (8, 8, 4), 3, "f32"),
        # the refinement's pass over the FP64 blocks, largest elements
        _case("residual_f64_6x6x6_p4", "residual", (6, 6, 6), 4, "f64"),
        # the small simulation's whole FP64 Newton step
        _case("newton_f64_4x4x4_p2", "newton", (4, 4, 4), 2, "f64"),
        # the headline: one paper-sized subdomain, mixed precision
        _case("newton_f32_16x16x8_p3", "newton", (16, 16, 8), 3, "f32"),
        # meshes of uneven size and degree, one captured graph
        {"name": "batch_f32_3_meshes", "kind": "batch", "meshes": "4x4x4:2,6x6x6:3,8x8x4:2", "prec": "f32"},
    ]


def _group(case):
    """(dims, p) of every mesh of a batched group."""
    each = [m.split(":") for m in case["meshes"].split(",")]
    return [(tuple(int(x) for x in dims.split("x")), int(p)) for dims, p in each]


def _dims(rng, most):
    """Mesh dimensions with at most `most` elements, spread over the logarithm
    of their number, odd ones among them."""
    while True:
        target = math.exp(rng.uniform(0.0, math.log(most)))
        r = max(1.0, target ** (1.0 / 3.0))
        d = [max(1, round(r * rng.uniform(0.6, 1.6))) for _ in range(3)]
        if d[0] * d[1] * d[2] <= most:
            return sorted(d, reverse=True)


def _drawn(rng):
    kind = rng.choice(["condense", "condense", "condense", "factor", "iedg", "rhs", "residual", "newton", "batch"])
    p = rng.choice([1, 2, 3, 4])
    most = {1: 2048, 2: 2048, 3: 864, 4: 216}[p]
    if kind == "condense":
        return _case(None, kind, _dims(rng, most), p, rng.choice(["f64", "f32", "bf16"]))
    if kind == "factor":
        return _case(None, kind, _dims(rng, min(most, 512)), p, rng.choice(["f64", "f32"]))
    if kind == "iedg":
        p = rng.choice([1, 2, 3])
        return _case(None, kind, _dims(rng, {1: 512, 2: 128, 3: 32}[p]), p, rng.choice(["f64", "f32"]))
    if kind == "residual":
        return _case(None, kind, _dims(rng, most), p, "f64")
    if kind == "batch":
        each = []
        for _ in range(rng.randint(2, 3)):
            q = rng.choice([2, 3, 4])
            each.append("%dx%dx%d:%d" % (*_dims(rng, {2: 256, 3: 216, 4: 32}[q]), q))
        return {"kind": kind, "meshes": ",".join(each), "prec": rng.choice(["f64", "f32"])}
    return _case(None, kind, _dims(rng, most), p, rng.choice(["f64", "f32"]))


def draw(rng):
    taken = [{k: v for k, v in c.items() if k != "name"} for c in listed()]
    while True:
        c = _drawn(rng)
        if c not in taken:
            return c


# ---- inputs ---------------------------------------------------------------
@functools.lru_cache(maxsize=1)
def _context():
    """The program's context, tuned as the benchmark program tunes its own."""
    ctx = api.Context()
    apply_tuning(ctx)
    return ctx


def _mesh(case):
    return StructuredHexMesh(case["nx"], case["ny"], case["nz"])


def _units(case):
    """Trace units of every element's slots, their number and dofs a unit."""
    hm, spec = _mesh(case), ElementSpec(case["p"])
    if case["kind"] == "iedg":
        nodes, count = hm.iedg_trace_nodes(case["p"])
        return nodes, count, 5
    return hm.elem_faces(), hm.n_face, spec.b


def _blocks(case, seed, which, mesh_id=0):
    return sdev.gen_blocks(ElementSpec(case["p"]), seed, mesh_id, _mesh(case).n_elem, which=which)


def _trace_inputs(case, seed):
    """Element trace matrices with the values a condensation leaves (D and a
    small C A^-1 B), r and G."""
    spec, E = ElementSpec(case["p"]), _mesh(case).n_elem
    units, count, b = _units(case)
    Ke = _blocks(case, seed, "D")["D"].to(api.PREC_DTYPE[PREC[case["prec"]]])
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = 0.3 * torch.randn((E, spec.t), dtype=torch.float64, device="cuda", generator=g)
    G = torch.randn(count * b, dtype=torch.float64, device="cuda", generator=g)
    return Ke, r, G


def _dev_mesh(case):
    units, count, b = _units(case)
    return api.Mesh(_context(), units, count, b, slots=case["kind"] == "iedg")


def _system(case, seed):
    d = _blocks(case, seed, "ABCDF")
    G = sdev.gen_trace_rhs(ElementSpec(case["p"]), seed, 0, _mesh(case).n_face)
    return d, G


def prepare(case, seed):
    ctx, kind, prec = _context(), case["kind"], PREC[case["prec"]]
    spec = ElementSpec(case.get("p", 0))
    s = {"case": case, "ctx": ctx, "prec": prec}
    if kind == "condense":
        E = _mesh(case).n_elem
        s["d"] = _blocks(case, seed, "ABCDF")
        s["out"] = api.alloc_condense_out(E, spec.n, spec.t, prec, "cuda")
    elif kind in ("factor", "iedg"):
        s["mesh"] = _dev_mesh(case)
        s["Ke"], s["r"], s["G"] = _trace_inputs(case, seed)
        nnzb, b = s["mesh"].nnzb, s["mesh"].b
        s["K"] = torch.empty((nnzb, b, b), dtype=api.PREC_DTYPE[prec], device="cuda")
        s["M"] = torch.empty_like(s["K"])
        if kind == "iedg":
            s["gm"] = api.GmresState(ctx, s["mesh"], 50)
    elif kind == "residual":
        s["mesh"] = _dev_mesh(case)
        s["d"], s["G"] = _system(case, seed)
        g = torch.Generator(device="cuda").manual_seed(seed)
        s["z"] = torch.randn((s["mesh"].n_elem, spec.n), dtype=torch.float64, device="cuda", generator=g)
        s["u"] = torch.randn(s["mesh"].n_trace, dtype=torch.float64, device="cuda", generator=g)
    elif kind in ("rhs", "newton"):
        s["d"], s["G"] = _system(case, seed)
        s["solver"] = NewtonStepSolver(ctx, _dev_mesh(case), spec.n)
        if kind == "rhs":
            d = s["d"]
            s["solver"].factor(d["A"], d["B"], d["C"], d["D"], None, prec=prec)
    else:
        sims = [Simulation(ctx, MeshCase(i, dims, p), seed, prec=prec) for i, (dims, p) in enumerate(_group(case))]
        for sim in sims:
            sim.generate()
        s["group"] = BatchGroup(ctx, sims)
        s["group"].enqueue()
        torch.cuda.synchronize()
        ctx.sync_status()
        s["group"].capture()
    return s


# ---- one pass -------------------------------------------------------------
def run(s):
    case, ctx, prec = s["case"], s["ctx"], s["prec"]
    kind = case["kind"]
    if kind == "condense":
        d = s["d"]
        return api.condense(ctx, d["A"], d["B"], d["C"], d["D"], d["F"], prec=prec, out=s["out"])
    if kind in ("factor", "iedg"):
        K, R = api.assemble(ctx, s["mesh"], Ke=s["Ke"], r=s["r"], G=s["G"], prec=prec, Kbsr=s["K"])
        M = api.factor_ilu0(ctx, s["mesh"], K, prec=prec, Mbsr=s["M"])
        if kind == "factor":
            return {"K": K, "R": R, "M": M}
        x, _ = api.gmres_solve(ctx, s["mesh"], K, M, R, 50, 1e-10, kprec=prec, mprec=prec, state=s["gm"])
        return {"M": M, "x": x}
    if kind == "residual":
        d = s["d"]
        rF, rG, sums = api.residual_full(ctx, s["mesh"], d["A"], d["B"], d["C"], d["D"], d["F"], s["G"], s["z"], s["u"])
        return {"rF": rF, "rG": rG, "sums": sums}
    if kind == "batch":
        s["group"].run()
        return [{"z": sim.z, "uhat": sim.uhat} for sim in s["group"].sims]
    d, G, solver = s["d"], s["G"], s["solver"]
    blocks = (d["A"], d["B"], d["C"], d["D"])
    if kind == "rhs":
        if prec == F64:
            z, uhat, _ = solver.solve_rhs_fp64(d["F"], G, 1e-10)
        else:
            z, uhat, _ = solver.solve_rhs_mixed(*blocks, d["F"], G, tol=1e-8)
    elif prec == F64:
        z, uhat, _ = solver.solve_fp64(*blocks, d["F"], G, 1e-10)
    else:
        z, uhat, _ = solver.solve_mixed(*blocks, d["F"], G, tol=1e-8, prec=prec)
    return {"z": z, "uhat": uhat}


# ---- what a pass cannot do without ------------------------------------------
def _newton_work(hm, spec):
    E, n, t = hm.n_elem, spec.n, spec.t
    bytes_ = 8.0 * E * (n * n + 2 * n * t + t * t + 2 * n) + 16.0 * hm.n_face * spec.b
    flops = E * (2.0 / 3.0 * n ** 3 + 2.0 * n * n * t + 2.0 * n * t * t)
    return bytes_, flops


def work(case):
    if case["kind"] == "batch":
        each = [_newton_work(StructuredHexMesh(*dims), ElementSpec(p)) for dims, p in _group(case)]
        return {"bytes": sum(w[0] for w in each), "flops": sum(w[1] for w in each)}
    hm, spec = _mesh(case), ElementSpec(case["p"])
    E, n, t, b = hm.n_elem, spec.n, spec.t, spec.b
    es = 8 if case["prec"] == "f64" else 4
    blocks = float(E) * (n * n + 2 * n * t + t * t)
    nnzb = hm.n_face + 30 * E
    kind = case["kind"]
    if kind == "condense":
        return {"bytes": (8 + es) * blocks + E * (16.0 * n + 8.0 * t + 4.0 * n), "flops": _newton_work(hm, spec)[1]}
    if kind == "factor":
        return {"bytes": es * (float(E) * t * t + 2.0 * nnzb * b * b) + 8.0 * E * t + 16.0 * hm.n_face * b,
                "flops": 2.0 * b ** 3 * (70.0 * E + hm.n_face)}
    if kind == "iedg":
        return {"bytes": (es + 8.0) * E * t * t, "flops": 2.0 * 10 * E * t * t}
    if kind == "residual":
        return {"bytes": 8.0 * blocks + 24.0 * E * n + 24.0 * hm.n_face * b, "flops": 2.0 * blocks}
    if kind == "rhs":
        passes = es * float(E) * (n * n + 2 * n * t) + 2.0 * es * nnzb * b * b
        return {"bytes": passes + (0.0 if es == 8 else 8.0 * blocks) + 16.0 * E * n + 16.0 * hm.n_face * b,
                "flops": 2.0 * blocks}
    bytes_, flops = _newton_work(hm, spec)
    return {"bytes": bytes_, "flops": flops}


# ---- the same in 64 bits, plain torch ---------------------------------------
def _chunks(E, n):
    step = max(1, int(2e9 / (8.0 * n * n)))
    return [(e, min(E, e + step)) for e in range(0, E, step)]


def _exact_condense(case, seed):
    spec, E = ElementSpec(case["p"]), _mesh(case).n_elem
    n, t = spec.n, spec.t
    d = _blocks(case, seed, "ABCDF")
    o = {"LU": torch.empty_like(d["A"]), "U12": torch.empty_like(d["B"]), "L21": torch.empty_like(d["C"]),
         "Ke": torch.empty_like(d["D"]), "w": torch.empty_like(d["F"]),
         "r": torch.empty((E, t), dtype=torch.float64, device="cuda"), "perm": None}
    for e0, e1 in _chunks(E, n):
        lu, piv = torch.linalg.lu_factor(d["A"][e0:e1])
        P, L, U = torch.lu_unpack(lu, piv)
        at = P.argmax(dim=1)                       # row i of P^T A: the row of A at position i
        rhs = torch.cat([d["B"][e0:e1], d["F"][e0:e1, :, None]], dim=2)
        rhs = torch.gather(rhs, 1, at[:, :, None].expand(-1, -1, t + 1))
        y = torch.linalg.solve_triangular(L, rhs, upper=False, unitriangular=True)
        x = torch.linalg.solve_triangular(U, d["C"][e0:e1], upper=True, left=False)
        S = torch.matmul(x.contiguous(), y.contiguous())
        back = torch.argsort(at, dim=1)            # stored row at[i] holds position i
        o["LU"][e0:e1] = torch.gather(lu, 1, back[:, :, None].expand(-1, -1, n))
        y = torch.gather(y, 1, back[:, :, None].expand(-1, -1, t + 1))
        o["U12"][e0:e1], o["w"][e0:e1] = y[:, :, :t], y[:, :, t]
        o["L21"][e0:e1] = x
        o["Ke"][e0:e1] = d["D"][e0:e1] - S[:, :, :t]
        o["r"][e0:e1] = -S[:, :, t]
    return o


def _gather(units, b):
    u = torch.as_tensor(units, dtype=torch.int64, device="cuda")
    return (u[:, :, None] * b + torch.arange(b, device="cuda")).reshape(u.shape[0], -1)


def _solve_trace(Ke, idx, R):
    """K x = R by GMRES with a diagonal preconditioner to rounding level."""
    N = R.numel()
    flat = idx.reshape(-1)

    def mv(x):
        y = torch.matmul(Ke, x[idx][:, :, None])
        return torch.zeros(N, dtype=torch.float64, device="cuda").index_add_(0, flat, y.reshape(-1))

    dg = torch.zeros(N, dtype=torch.float64, device="cuda")
    dg.index_add_(0, flat, torch.diagonal(Ke, dim1=1, dim2=2).reshape(-1))
    x = torch.zeros_like(R)
    for _ in range(4):
        r = (R - mv(x)) / dg
        beta = r.norm()
        if float(beta) <= 1e-15 * float((R / dg).norm()):
            break
        V, H = [r / beta], torch.zeros((61, 60), dtype=torch.float64)
        for j in range(60):
            w = mv(V[j]) / dg
            W = torch.stack(V)
            h = W @ w
            w = w - W.T @ h
            h2 = W @ w
            w = w - W.T @ h2
            H[: j + 1, j] = (h + h2).cpu()
            H[j + 1, j] = float(w.norm())
            if float(H[j + 1, j]) < 1e-14:
                break
            V.append(w / w.norm())
        m = j + 1
        e1 = torch.zeros(m + 1, dtype=torch.float64)
        e1[0] = float(beta)
        y = torch.linalg.lstsq(H[: m + 1, :m], e1[:, None]).solution[:, 0]
        x = x + torch.stack(V[:m]).T @ y.cuda()
    return x


def _exact_newton(d, G, idx):
    E, n = d["F"].shape
    t = idx.shape[1]
    Ke = torch.empty_like(d["D"])
    xb, xf = torch.empty_like(d["B"]), torch.empty_like(d["F"])
    r = torch.empty((E, t), dtype=torch.float64, device="cuda")
    for e0, e1 in _chunks(E, n):
        X = torch.linalg.solve(d["A"][e0:e1], torch.cat([d["B"][e0:e1], d["F"][e0:e1, :, None]], dim=2)).contiguous()
        S = torch.matmul(d["C"][e0:e1], X)
        Ke[e0:e1], r[e0:e1] = d["D"][e0:e1] - S[:, :, :t], -S[:, :, t]
        xb[e0:e1], xf[e0:e1] = X[:, :, :t], X[:, :, t]
    R = G.clone().index_add_(0, idx.reshape(-1), r.reshape(-1))
    u = _solve_trace(Ke, idx, R)
    z = xf - torch.matmul(xb, u[idx][:, :, None])[:, :, 0]
    return {"z": z, "uhat": u}


def _exact_factor(case, seed):
    """K in block rows ordered by a greedy colouring of the faces and its
    zero-fill block ILU, one block product at a time."""
    Ke, r, G = _trace_inputs(case, seed)
    units, nf, b = _units(case)
    idx = _gather(units, b)
    R = G.clone().index_add_(0, idx.reshape(-1), r.reshape(-1))
    Kh = Ke.double().cpu().numpy()
    near = [set() for _ in range(nf)]
    for row in units:
        for f in row:
            near[f].update(int(g) for g in row)
    colour = [-1] * nf
    for f in range(nf):
        used = {colour[g] for g in near[f]}
        colour[f] = next(c for c in range(len(used) + 1) if c not in used)
    order = sorted(range(nf), key=lambda f: (colour[f], f))
    pos = {f: i for i, f in enumerate(order)}
    blk = {}
    for e, row in enumerate(units):
        for a, f in enumerate(row):
            for c, g in enumerate(row):
                v = Kh[e, a * b:(a + 1) * b, c * b:(c + 1) * b]
                k = (pos[int(f)], pos[int(g)])
                blk[k] = blk[k] + v if k in blk else v.copy()
    cols = [sorted(pos[g] for g in near[f]) for f in order]
    K = np.stack([blk[i, j].T for i in range(nf) for j in cols[i]])
    for i in range(nf):
        for k in cols[i]:
            if k >= i:
                break
            lik = blk[i, k] = blk[i, k] @ blk[k, k]     # pivots are held inverted
            for j in cols[k]:
                if j > k and (i, j) in blk:
                    blk[i, j] = blk[i, j] - lik @ blk[k, j]
        blk[i, i] = np.linalg.inv(blk[i, i])
    M = np.stack([blk[i, j].T for i in range(nf) for j in cols[i]])
    return {"K": torch.from_numpy(K), "R": R, "M": torch.from_numpy(M)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "condense":
        return _exact_condense(case, seed)
    if kind == "factor":
        return _exact_factor(case, seed)
    if kind == "batch":
        out = []
        for i, (dims, p) in enumerate(_group(case)):
            c = _case(None, "newton", dims, p, case["prec"])
            d = _blocks(c, seed, "ABCDF", mesh_id=i)
            G = sdev.gen_trace_rhs(ElementSpec(p), seed, i, _mesh(c).n_face)
            out.append(_exact_newton(d, G, _gather(_units(c)[0], ElementSpec(p).b)))
        return out
    units, count, b = _units(case)
    idx = _gather(units, b)
    if kind == "iedg":
        Ke, r, G = _trace_inputs(case, seed)
        R = G.clone().index_add_(0, idx.reshape(-1), r.reshape(-1))
        return {"M": None, "x": _solve_trace(Ke.double(), idx, R)}
    d, G = _system(case, seed)
    if kind in ("rhs", "newton"):
        return _exact_newton(d, G, idx)
    spec, E = ElementSpec(case["p"]), idx.shape[0]
    g = torch.Generator(device="cuda").manual_seed(seed)
    z = torch.randn((E, spec.n), dtype=torch.float64, device="cuda", generator=g)
    u = torch.randn(count * b, dtype=torch.float64, device="cuda", generator=g)
    zc, uc = z[:, :, None], u[idx][:, :, None].contiguous()
    rF = d["F"] - (torch.matmul(d["A"], zc) + torch.matmul(d["B"], uc))[:, :, 0]
    q = (torch.matmul(d["C"], zc) + torch.matmul(d["D"], uc))[:, :, 0]
    rG = G.clone().index_add_(0, idx.reshape(-1), q.reshape(-1), alpha=-1.0)
    sums = torch.stack([rF.square().sum(), rG.square().sum(), d["F"].square().sum(), G.square().sum()])
    return {"rF": rF, "rG": rG, "sums": sums}
