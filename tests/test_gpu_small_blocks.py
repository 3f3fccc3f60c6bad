"""GPU parity of the node-block BILU(0) (blocks of 1 to 8) and its sweeps.

Meshes whose rows have from one to some 200 blocks, so that a row's chain of
lower slots and a slot's list of updates cover less than one, exactly and more
than the units a workgroup fetches ahead; both precisions.  Tolerances: the
factor blocks are sums of at most 200 products of blocks of norm about 1 whose
pivots are dominated by D (condition below 10), so 200 x 10 x 2^-53 < 1e-11 in
FP64 and 200 x 10 x 2^-24 < 2e-4 in FP32; a sweep adds chains of the same
length."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, bsr_from_oracle, oracle_from_bsr, rel
from synth import StructuredHexMesh

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


@pytest.mark.parametrize("b", [1, 2, 3, 4, 6, 7, 8])
@pytest.mark.parametrize("dims,p", [((1, 1, 1), 1), ((2, 1, 1), 1), ((2, 2, 2), 2), ((2, 2, 1), 3)])
def test_small_block_factor_and_sweeps(ctx, b, dims, p):
    hm = StructuredHexMesh(*dims)
    nodes, count = hm.iedg_trace_nodes(p)
    print(f"[gpu-test] node blocks b={b} dims={dims} p={p} nodes={count}", flush=True)
    tm = oracle.TraceMesh(nodes, count, b)
    t = nodes.shape[1] * b
    rng = np.random.default_rng(100 * b + p)
    Ks = [1.5 * np.eye(t) + rng.standard_normal((t, t)) * (0.1 / np.sqrt(t)) for _ in range(hm.n_elem)]
    K, _ = oracle.assemble(tm, Ks, [np.zeros(t)] * hm.n_elem, np.zeros(count * b))
    mesh = api.Mesh(ctx, nodes, count, b, slots=True)
    q = mesh.query()
    fac = oracle.bilu0(tm, K, q["order"])
    x = rng.standard_normal(count * b)
    y = oracle.bilu0_apply(tm, fac, x)
    for prec, dt, tol in ((F64, torch.float64, 1e-11), (F32, torch.float32, 2e-4)):
        Kd = dev(bsr_from_oracle(mesh, K, q), dt)
        Md = api.factor_ilu0(ctx, mesh, Kd, prec=prec)
        ctx.sync_status()
        got = oracle_from_bsr(mesh, Md.cpu().numpy().astype(np.float64), q)
        scale = max(np.abs(v).max() for v in K.values())
        for key, Lb in fac["L"].items():
            assert np.abs(got[key] - Lb).max() <= tol * scale, key
        for i, Ui in fac["Uinv"].items():
            assert np.abs(got[(i, i)] - Ui).max() <= tol * np.abs(Ui).max(), i
        assert rel(api.ilu0_apply(ctx, mesh, Md, dev(x), prec=prec).cpu().numpy(), y) <= tol
