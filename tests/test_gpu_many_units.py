"""Meshes of more rows than one launch of 512-thread workgroups can have (its
threads are counted in 32 bits: 8,388,607 workgroups), with blocks of one dof:
the trace operators of elements that share nothing are exact by inspection."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_1605_01020_amd.api")
from paper_1605_01020_amd import F64, F32  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = api.Context()
    yield c
    torch.cuda.synchronize()


def test_trace_operators_past_a_launch_of_512_threads(ctx):
    E = 2 ** 23 + 5
    print(f"[gpu-test] {E} units of one dof", flush=True)
    mesh = api.Mesh(ctx, np.arange(E, dtype=np.int32)[:, None], E, 1, ordering="natural", slots=True)
    assert mesh.nnzb == E and mesh.n_levels == 1
    k = torch.arange(E, dtype=torch.float64, device="cuda") % 7 - 9.0  # -9 .. -3
    x = torch.arange(E, dtype=torch.float64, device="cuda") % 5 + 1.0
    for prec, dt in ((F64, torch.float64), (F32, torch.float32)):
        K = k.to(dt).reshape(E, 1, 1)
        y = api.spmv(ctx, mesh, K, x, prec=prec)
        assert torch.equal(y, k * x)
        M = api.factor_ilu0(ctx, mesh, K, prec=prec)
        ctx.sync_status()
        assert torch.equal(M.flatten(), (1.0 / k.to(dt)))
        z = api.ilu0_apply(ctx, mesh, M, x, prec=prec)
        assert torch.equal(z, M.flatten().double() * x)
    mesh.close()


def test_residual_past_a_launch_of_128_threads(ctx):
    """Units and elements together above 33,554,431, neither of them alone."""
    E, S, n = 8_400_000, 3, 4
    print(f"[gpu-test] {E} elements of {S} units of one dof", flush=True)
    mesh = api.Mesh(ctx, np.arange(E * S, dtype=np.int32).reshape(E, S), E * S, 1, ordering="natural", slots=True)
    small = torch.arange(E, dtype=torch.float64, device="cuda") % 3 + 1.0

    def ints(*shape):  # (the element's small integer, times a pattern within the element)
        m = torch.arange(int(np.prod(shape)), dtype=torch.float64, device="cuda").reshape(1, *shape) % 4 - 1.0
        return (small.reshape(-1, *[1] * len(shape)) * m).contiguous()
    A, B, C, D, F, z = ints(n, n), ints(n, S), ints(S, n), ints(S, S), ints(n), ints(n)
    u, G = ints(S).flatten(), ints(S).flatten() + 1.0
    rF, rG, sums = api.residual_full(ctx, mesh, A, B, C, D, F, G, z, u)
    ue = u.reshape(E, S)
    wF = F - (A * z[:, None, :]).sum(2) - (B * ue[:, None, :]).sum(2)
    wG = G - ((C * z[:, None, :]).sum(2) + (D * ue[:, None, :]).sum(2)).flatten()
    assert torch.equal(rF, wF) and torch.equal(rG, wG)
    # sums of small integers: exact
    assert sums.tolist() == [v.square().sum().item() for v in (wF, wG, F, G)]
    mesh.close()
