"""Host-side logic of the batched and serving forms (no GPU)."""
import numpy as np
import pytest

from synth.matrices import workload, MeshCase


def test_plan_groups_packs_every_mesh_once_under_budget():
    from paper_1605_01020_amd.batch import plan_groups, Simulation
    wl = workload(3)
    budget = 200e9
    groups = plan_groups(wl.meshes, budget)
    ids = sorted(c.mesh_id for g in groups for c in g)
    assert ids == list(range(len(wl.meshes)))
    for g in groups:
        assert sum(Simulation.footprint(c) for c in g) <= budget
    with pytest.raises(ValueError):
        plan_groups(wl.meshes, 1e9)


def test_nnzb_estimate_matches_structure_table():
    # nonzero face blocks of K for the meshes of the batched configuration
    from paper_1605_01020_amd.batch import _nnzb_estimate
    from synth.mesh import StructuredHexMesh
    for dims, nnzb in (((4, 4, 4), 2160), ((16, 16, 8), 68096), ((6, 6, 6), 7236), ((8, 8, 4), 8576),
                       ((12, 12, 6), 28800)):
        assert _nnzb_estimate(StructuredHexMesh(*dims)) == nnzb


def test_poisson_requests_are_seeded_and_poisson():
    from paper_1605_01020_amd.serve import poisson_requests
    a = poisson_requests(7, 4000, 50.0, 64)
    b = poisson_requests(7, 4000, 50.0, 64)
    assert [(r.sim, r.rhs, r.arrival) for r in a] == [(r.sim, r.rhs, r.arrival) for r in b]
    gaps = np.diff([r.arrival for r in a])
    assert abs(gaps.mean() - 1 / 50.0) < 0.1 / 50.0          # exponential mean 1/rate
    assert abs(gaps.std() - 1 / 50.0) < 0.1 / 50.0            # and std 1/rate
    sims = np.array([r.sim for r in a])
    assert sims.min() == 0 and sims.max() == 63
    # right-hand side ids count per simulation from 1
    seen = {}
    for r in a:
        seen[r.sim] = seen.get(r.sim, 0) + 1
        assert r.rhs == seen[r.sim]


class _Stream:
    """Stands in for a stream: notes what is queued and whom it waits for."""

    def __init__(self, log):
        self.log = log

    def wait_stream(self, other):
        self.log.append(("wait", self, other))


class _Sim:
    def __init__(self, log, streams, n_trace, gm=None, mesh=None, fails=False):
        self.log, self.streams, self.fails = log, streams, fails
        self.gm = [object()] if gm is None else gm
        self.mesh = type("M", (), {"n_trace": n_trace})() if mesh is None else mesh

    def enqueue_after_condense(self):
        if self.fails:
            raise RuntimeError("refused")
        self.log.append(("solve", self, self.streams[-1]))


def _group(monkeypatch, sims, log, streams):
    """A BatchGroup over stand-ins: no library, no GPU."""
    import contextlib
    from paper_1605_01020_amd import batch

    @contextlib.contextmanager
    def on(st):
        streams.append(st)
        try:
            yield
        finally:
            streams.pop()

    monkeypatch.setattr(batch.torch.cuda, "current_stream", lambda: streams[-1])
    monkeypatch.setattr(batch.torch.cuda, "stream", on)
    g = batch.BatchGroup.__new__(batch.BatchGroup)
    g.sims, g.plans = sims, []
    g.branches = g._branches()
    g.streams = [_Stream(log) for _ in g.branches[1:]]
    return g


@pytest.mark.parametrize("failing", [None, 0, 1, 2, 4])
def test_batch_group_joins_every_branch(monkeypatch, failing):
    """Every stream that was forked from the caller's is joined to it at the
    end, also when a mesh's solve is refused on any branch."""
    log = []
    here = _Stream(log)
    streams = [here]
    sims = [_Sim(log, streams, 100 - i, fails=i == failing) for i in range(5)]
    g = _group(monkeypatch, sims, log, streams)
    if failing is None:
        g.enqueue()
    else:
        with pytest.raises(RuntimeError, match="refused"):
            g.enqueue()
    assert streams == [here]
    used = {e[2] for e in log if e[0] == "solve"} - {here}
    for st in used | {s for s in g.streams if ("wait", s, here) in log}:
        last = max((i for i, e in enumerate(log) if e[0] == "solve" and e[2] is st), default=-1)
        assert ("wait", here, st) in log[last + 1:], "a branch is left unjoined"
    if failing is None:
        assert len([e for e in log if e[0] == "solve"]) == 5 and len(g.streams) == 3


def test_batch_group_branches(monkeypatch):
    """Meshes that share a workspace stay on one branch, in their order: a
    shared mesh, a shared GMRES state, and chains of both."""
    log, streams = [], [None]

    def sim(n, **k):
        return _Sim(log, streams, n, **k)

    def deal(sims):
        g = _group(monkeypatch, sims, log, streams)
        assert sorted(map(id, sims)) == sorted(id(s) for b in g.branches for s in b)
        assert all(g.branches) and len(g.branches) <= g.BRANCHES
        return {id(s): k for k, b in enumerate(g.branches) for s in b}, g.branches

    assert deal([])[1] == []
    assert len(deal([sim(5)])[1]) == 1
    assert len(deal([sim(5), sim(4), sim(3)])[1]) == 3
    assert len(deal([sim(n) for n in range(9, 0, -1)])[1]) == 4
    a, b = sim(7), sim(6)
    c = sim(5, mesh=a.mesh)                    # a's mesh
    d = sim(4, gm=[b.gm[0], object()])         # b's GMRES state
    where, br = deal([a, b, c, d])
    assert where[id(a)] == where[id(c)] != where[id(b)] == where[id(d)]
    assert all(x.index(p) < x.index(q) for x in br for p, q in ((a, c), (b, d)) if p in x)
    e = sim(3, gm=[a.gm[0], d.gm[1]])          # joins both chains
    where, br = deal([a, b, c, d, e, sim(2)])
    assert len({where[id(s)] for s in (a, b, c, d, e)}) == 1 and len(br) == 2
    one = next(x for x in br if a in x)
    for p, q in ((a, c), (b, d), (a, e), (d, e)):
        assert one.index(p) < one.index(q)


def test_autotuner_keeps_a_choice_within_its_margin():
    from paper_1605_01020_amd import autotune
    t = {(8, 64): 1.0, (16, 64): 1.015, (8, 128): 1.03}
    assert autotune.choose(t) == (8, 64)
    assert autotune.choose(t, (16, 64)) == (16, 64)      # within 2% of the fastest
    assert autotune.choose(t, (8, 128)) == (8, 64)       # not
    assert autotune.choose(t, (16, 128)) == (8, 64)      # not built
    # every stored choice is the fastest of its row or within the margin
    import json
    with open(autotune.TUNING_PATH) as f:
        for e in json.load(f)["entries"]:
            ms = {tuple(map(int, k.split("/"))): v for k, v in e["ms"].items()}
            kept = (e["leaf_width"], e["panel_width"])
            assert autotune.choose(ms, kept) == kept, e
