"""Zero, infinite and subnormal pivots, overflows and infinities: what IEEE
arithmetic gives for them, step by step, is what the kernels give."""
import numpy as np
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1605_01020_amd.api")
from paper_1605_01020_amd import F64, F32, BF16  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = api.Context()
    yield c
    torch.cuda.synchronize()


def _back(U, y):
    """U z = y from the last row up: a quotient, then one product and one
    difference for every row above."""
    z = y.copy()
    with np.errstate(all="ignore"):
        for k in range(len(z) - 1, -1, -1):
            z[k] /= U[k, k]
            z[:k] -= U[:k, k] * z[k]
    return z


# 1 and 513 elements: both widths of the workgroup; 68 rows: two blocks of the
# triangle.  Every value is a power of two
# or zero and no row sums more than two of them, so the order cannot show.
@pytest.mark.parametrize("E", [1, 513])
@pytest.mark.parametrize("prec,dtype", [(F64, np.float64), (F32, np.float32)])
def test_backsolve_pivots_out_of_range(ctx, E, prec, dtype):
    n, b = 68, 2
    tiny = np.float64(5e-324) if prec == F64 else np.float64(2.0 ** -149)
    cases = {"infinite pivot": (3, np.inf, 4.0), "zero pivot": (3, 0.0, 4.0), "zero over zero": (66, 0.0, 0.0),
             "overflow": (5, tiny, 2.0 ** 1023), "infinite value": (2, 4.0, np.inf),
             "smallest pivot": (66, tiny, 2.0 ** -1060), "smallest pivot, zero": (7, tiny, 0.0),
             "largest pivot": (65, 2.0 ** (1023 if prec == F64 else 127), 2.0 ** 1000),
             "ordinary": (0, 2.0, 8.0)}
    mesh = api.Mesh(ctx, np.arange(E)[:, None], E, b, slots=True)
    for name, (row, pivot, value) in cases.items():
        print(f"[gpu-test] back-substitution, {name} E={E} prec={int(prec)}", flush=True)
        U = np.diag(np.full(n, 2.0))
        U[0, 65], U[1, 64], U[1, 7], U[2, 3] = 0.25, 4.0, 0.5, 0.5
        y = np.zeros(n)
        y[0] = 1.0
        U[row, row], y[row] = pivot, value  # (rows below it are zero: it meets its value alone)
        ref = _back(U, y)
        fac = {"LU": dev(np.repeat(U[None].astype(dtype), E, 0)),
               "perm": dev(np.repeat(np.arange(n, dtype=np.int32)[None], E, 0)),
               "U12": dev(np.zeros((E, n, b), dtype)),
               "w": dev(np.repeat(y[None], E, 0))}
        z = api.backsolve_local(ctx, mesh, fac, torch.zeros(E * b, dtype=torch.float64, device="cuda"), prec=prec)
        np.testing.assert_array_equal(z.cpu().numpy(), np.broadcast_to(ref, (E, n)), err_msg=name)


# sizes and widths at which every product with L_pp^{-1} occurs: inside a panel,
# between a 128-wide panel's halves, in the panel rows, and (small t) with the
# inverse formed again there
@pytest.mark.parametrize("n,t", [(20, 30), (68, 130), (140, 6), (196, 112)])
def test_condense_rows_before_a_bad_pivot_keep_their_values(ctx, n, t):
    """The rows of U, U12 and w at positions before p do not depend on row p:
    with an infinity in that row, or no pivot at p at all, they have the bits
    they have without."""
    g = torch.Generator().manual_seed(7 * n + t)

    def r(*s):
        return torch.randn(*s, dtype=torch.float64, generator=g)
    A = (r(n, n) / n ** 0.5 + 2 * torch.eye(n, dtype=torch.float64)).cuda()
    B, C, D, F = (x.cuda() for x in (r(n, t) / n ** 0.5, r(t, n) / n ** 0.5, r(t, t), r(n)))
    for prec, widths in ((F64, [(8, 64), (16, 64)]), (F32, [(8, 64), (16, 64), (8, 128), (16, 128)]),
                         (BF16, [(16, 64), (16, 128)])):
        for lw, ct in widths:
            api.set_leaf_width(ctx, n, lw, prec=prec)
            api.set_panel_width(ctx, n, ct, prec=prec)
            o = api.condense(ctx, *(x[None].contiguous() for x in (A, B, C, D, F)), prec=prec)
            ctx.sync_status()
            ref = {k: v[0] for k, v in o.items()}
            perm = ref["perm"].long()
            spots = sorted({min(x, n - 1) for x in (3, 6, 13, 18, 35, 67, 75, 110, 131, n - 1)})
            As, ps, cs = [], [], []
            for p in spots:
                M = A.clone()  # no pivot for column p: of rows before p, only that column changes
                M[:, p] = 0.0
                As.append(M), ps.append(p), cs.append(p)
                for c in spots:
                    if c > p:
                        M = A.clone()
                        M[perm[p], c] = float("inf")
                        # (the panel rows' solve takes whole 16 x 16 blocks: that column is left out)
                        As.append(M), ps.append(p), cs.append(c if c >= (p // ct + 1) * ct else None)
            E = len(As)
            print(f"[gpu-test] bad pivots n={n} t={t} prec={int(prec)} widths {lw}/{ct} elements {E}", flush=True)
            o = api.condense(ctx, torch.stack(As), *(x.expand(E, *x.shape).contiguous() for x in (B, C, D, F)), prec=prec)
            with pytest.raises(Exception, match="singular"):
                ctx.sync_status()
            for e, (p, c) in enumerate(zip(ps, cs)):
                rows = perm[:p]
                assert torch.equal(o["perm"][e, :p].long(), rows)
                for k in ("U12", "w"):
                    assert torch.equal(o[k][e][rows], ref[k][rows]), (k, lw, ct, p, c)
                got, want = torch.triu(o["LU"][e][rows]), torch.triu(ref["LU"][rows])
                if c is not None:
                    got[:, c], want[:, c] = 0.0, 0.0
                assert torch.equal(got.isfinite(), want.isfinite()) and torch.equal(got, want), ("U", lw, ct, p, c)
