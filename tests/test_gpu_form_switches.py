"""Both sides of every switch on the number of rows or elements: SpMV (512
rows), sweeps (512 rows a level), face-block factorisation (256 rows a level)
and element solves (512 elements), at block and element sizes whose remainders
(columns past a multiple of 8 or 16, rows past a multiple of 64, no vector
access) a form of its own handles.

Trace system: groups of S units that share nothing, so every level has one row
a group, BILU(0) is the block LU of each group's dense matrix and its
application the dense solve, checked by its residual.  Tolerance: S b terms of one rounding each
(2^-53, FP32 factors 2^-24), times 16 for the condition (diagonal 1.5,
off-diagonal part of norm 0.2) and the growth of the pivot inverses; SpMV
accumulates in FP64 in both.  Element solves: factors are data, so the rows'
residuals are FP64 roundings of n terms in both."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1605_01020_amd.api")
from paper_1605_01020_amd import F64, F32  # noqa: E402

S = 7


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = api.Context()
    yield c
    torch.cuda.synchronize()


def _rel(a, b):
    return (torch.linalg.norm(a - b) / torch.linalg.norm(b)).item()


@pytest.mark.parametrize("b", [9, 20, 45, 80, 125])
def test_trace_operators_either_side_of_the_row_switches(ctx, b):
    g = torch.Generator(device="cuda").manual_seed(b)
    most = 513
    t = S * b
    Ke = torch.randn(most, t, t, dtype=torch.float64, device="cuda", generator=g) * (0.1 / t ** 0.5)
    Ke += 1.5 * torch.eye(t, dtype=torch.float64, device="cuda")
    x = torch.randn(most, t, dtype=torch.float64, device="cuda", generator=g)
    # 73 and 74 groups: 511 and 518 rows in all
    for E in (73, 74, 256, 257, 511, 512, 513):
        mesh = api.Mesh(ctx, np.arange(E * S, dtype=np.int32).reshape(E, S), E * S, b, ordering="natural", slots=True)
        q = mesh.query()
        assert mesh.n_levels == S and (np.diff(q["level_ptr"]) == E).all()
        assert (q["col_face"] == np.repeat(np.arange(E * S).reshape(E, S), S, 0).ravel()).all()
        blocks = Ke[:E].reshape(E, S, b, S, b).permute(0, 1, 3, 4, 2).reshape(-1, b, b)  # column-major blocks
        for prec, dt, eps in ((F64, torch.float64, 2.0 ** -53), (F32, torch.float32, 2.0 ** -24)):
            print(f"[gpu-test] rows {E} a level, b={b} prec={int(prec)}", flush=True)
            K = blocks.to(dt).contiguous()
            dense = Ke[:E].to(dt).double()
            xs = x[:E].flatten().contiguous()
            y = api.spmv(ctx, mesh, K, xs, prec=prec)
            assert _rel(y, (dense * x[:E, None, :]).sum(2).flatten()) <= 4 * t * 2.0 ** -53
            M = api.factor_ilu0(ctx, mesh, K, prec=prec)
            ctx.sync_status()
            tol = 16 * t * eps
            got = api.ilu0_apply(ctx, mesh, M, xs, prec=prec)
            # group by group: a wrong row cannot hide in the norm of all
            res = (dense * got.reshape(E, 1, t)).sum(2) - x[:E]
            assert (torch.linalg.norm(res, dim=1) / torch.linalg.norm(x[:E], dim=1)).max().item() <= tol
            again = xs.clone()  # in place
            assert torch.equal(api.ilu0_apply(ctx, mesh, M, again, prec=prec, y=again), got)
        mesh.close()


@pytest.mark.parametrize("n,t", [(4, 2), (68, 30), (160, 120), (540, 270)])
@pytest.mark.parametrize("prec,dt", [(F64, torch.float64), (F32, torch.float32)])
def test_element_solves_either_side_of_the_element_switch(ctx, n, t, prec, dt):
    g = torch.Generator(device="cuda").manual_seed(n)
    most = 514

    def r(*s):
        return torch.randn(*s, dtype=torch.float64, device="cuda", generator=g)
    T = r(most, n, n) * (0.5 / n ** 0.5) + 2 * torch.eye(n, dtype=torch.float64, device="cuda")
    perm = torch.argsort(torch.rand(most, n, device="cuda", generator=g), dim=1)
    U12, L21 = r(most, n, t) / t ** 0.5, r(most, t, n) / n ** 0.5
    T, U12, L21 = (v.to(dt) for v in (T, U12, L21))
    F, u = r(most, n), r(most, t)
    put = perm[:, :, None].expand(-1, -1, n)
    fac = {"LU": torch.empty_like(T).scatter_(1, put, T), "perm": perm.int(), "L21": L21,
           "U12": torch.empty_like(U12).scatter_(1, perm[:, :, None].expand(-1, -1, t), U12)}
    L = torch.tril(T.double(), -1) + torch.eye(n, dtype=torch.float64, device="cuda")
    U = torch.triu(T.double())
    tol = 8 * (n + t) * 2.0 ** -53
    kept = {}
    for E in (511, 512, 513, 514):
        print(f"[gpu-test] element solves E={E} n={n} t={t} prec={int(prec)}", flush=True)
        f = {k: v[:E].contiguous() for k, v in fac.items()}
        w, rr = api.condense_rhs(ctx, f, F[:E].contiguous(), prec=prec)
        wp, Fp = (v.gather(1, perm[:E]) for v in (w, F[:E]))
        scale = torch.linalg.norm(Fp, dim=1)
        assert (torch.linalg.norm((L[:E] * wp[:, None, :]).sum(2) - Fp, dim=1) / scale).max().item() <= tol
        want = -(L21[:E].double() * wp[:, None, :]).sum(2)
        assert (torch.linalg.norm(rr - want, dim=1) / (torch.linalg.norm(want, dim=1) + scale)).max().item() <= tol
        mesh = api.Mesh(ctx, np.arange(E, dtype=np.int32)[:, None], E, t, ordering="natural", slots=True) if t <= 128 else \
            api.Mesh(ctx, np.arange(3 * E, dtype=np.int32).reshape(E, 3), 3 * E, t // 3, ordering="natural", slots=True)
        z = api.backsolve_local(ctx, mesh, f, u[:E].flatten().contiguous(), prec=prec, w=w)
        rhs = wp - (U12[:E].double() * u[:E, None, :]).sum(2)
        err = torch.linalg.norm((U[:E] * z[:, None, :]).sum(2) - rhs, dim=1) / torch.linalg.norm(rhs, dim=1)
        assert err.max().item() <= tol
        mesh.close()
        kept[E] = (w, rr, z)
    for E in (512, 513, 514):
        for a, v in zip(kept[511], kept[E]):
            assert _rel(v[:511], a) <= tol
