"""Edges of the rank-k step's dispatch on the GPU: the spaced top-k selection where
an excluded window covers more score chunks than the selecting workgroup has
waves, where near-ties lie in different chunks (a chunk is then scanned), and
with a spacing beyond the grid; and the rank-32 FP32 update at a size from which
it takes 256 rows per workgroup.

Tolerances: selections are exact (the oracle's rule on the scores the GPU
computed from); the updated G is held to the complex64 drift bound of k updates
(tests/parity.py), E and the FP64 diagonal to 5e-6 as in the rank-k tests.
"""
import numpy as np
import pytest

from oracle import greedy as og, state as ost
from parity import c64_drift_tol, rel_elem as _rel
import workloads as W

pytestmark = pytest.mark.gpu


def _job(p, **kw):
    from paper_2202_05388_amd.job import Job
    print(f"[case] {p.name} {p.ny}x{p.nx} mon={p.n_mon} {p.dtype} {kw}", flush=True)
    return Job(p, device="cuda:0", **kw)


@pytest.mark.parametrize("ny,nx,n_eps,k,spacing,tau", [
    (40, 41, 2, 12, 9, 1e-9),      # 17 x 17 windows over up to 4 of 7 chunks
    (9, 190, 3, 20, 5, 1e-9),      # long rows: a window row per chunk, every chunk touched
    (40, 41, 2, 32, 2, 0.02),      # wide band: the winner lies in a chunk below the best one's
    (33, 31, 8, 16, 3, 0.02),
    (16, 16, 2, 8, 1000, 1e-9),    # one chunk, a spacing beyond the grid: a single pick
    (23, 29, 2, 32, 0, 1e-9),
])
def test_topk_selection_edges(ny, nx, n_eps, k, spacing, tau):
    table = (1.0, 12.25, 2.25, 4.0, 6.25, 9.0, 3.0, 1.5)[:n_eps]
    p = W.tiny(ny, nx, n_mon=8, dtype="c128", cand_mask=(1 << n_eps) - 1, eps_table=table)
    N = p.n
    idx = W.random_material_idx(p, 7)
    idx[np.random.default_rng(3).random(N) < 0.7] = 0
    G, E = ost.dense_state(p, ost.eps_of(p, idx))
    job = _job(p)
    job.upload_state(G, E, np.diagonal(G[:N]), idx)
    job.score(topk=k, min_spacing=spacing, tau=tau)
    got = job.read_picks(k)
    F = og.scores_closed_form(p, E, np.diagonal(G[:N]), G[N + p.fom_monitor], idx)
    ref = og.select_rank_k(F, ost.fom_of_state(p, E), tau, k, spacing, p.nx)
    assert [(a, b) for a, b, _, _ in got if a >= 0] == [(r.pixel, r.eps_idx) for r in ref]
    assert len(ref) >= 1 and all(a < 0 for a, _, _, _ in got[len(ref):])
    # the score array marks the window of every pick that another could have followed
    marked = np.zeros((ny, nx), bool)
    w = max(spacing - 1, 0)
    for r in ref[: k - 1]:
        y, x = divmod(r.pixel, nx)
        marked[max(y - w, 0): y + w + 1, max(x - w, 0): x + w + 1] = True
    assert np.all(np.isneginf(job.scores()[marked.reshape(-1)]))


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_rank_32_update_large(precision):
    """77 x 76 pixels: 5852 columns, 23 x 46 = 1058 workgroups of 256 rows, ragged in both directions."""
    from paper_2202_05388_amd import _lib as L
    p = W.tiny(77, 76, n_mon=8, dtype="c64")
    N, s = p.n, 24
    from oracle import greens
    G, E = greens.build_G0(p), greens.incident_field(p)
    idx = np.zeros(N, np.uint8)
    pix = np.random.default_rng(1).choice(N, s, replace=False)
    Gd, Ed = ost.update_region(p, G, E, ost.eps_of(p, idx), pix, np.full(s, p.eps_table[1]))
    job = _job(p)
    job.upload_state(G, E, np.diagonal(G[:N]), idx)
    for t, j in enumerate(pix):
        job.set_pick(int(j), 1, slot=t)
    job.apply_rank_k(s, precision=L.GFO_FP32 if precision == "fp32" else L.GFO_BF16)
    G1, E1, d1, i1 = job.host_state()
    assert job.status() == 0 and sorted(np.flatnonzero(i1)) == sorted(int(j) for j in pix)
    if precision == "fp32":
        assert _rel(G1, Gd) <= c64_drift_tol(s)
    else:
        assert _rel(G1 - G, Gd - G, floor=1.0) <= 1e-2
    assert _rel(E1, Ed) <= 5e-6
    assert _rel(d1, np.diagonal(Gd[:N])) <= 5e-6


def test_records_of_32_with_repeats():
    """32 records of which a pixel's first valid one counts (no-ops, sentinels and pixels or
    materials out of range between them): the same bits as the counted ones alone."""
    from paper_2202_05388_amd import _lib as L
    p = W.tiny(12, 13, n_mon=5, dtype="c64").replace(eps_table=(1.0, 12.25, 4.0))
    rng = np.random.default_rng(3)
    recs, counted = [], []
    for j in rng.choice(p.n, 14, replace=False):
        e = int(rng.integers(1, 3))
        recs += [(int(j), 0), (int(j), e)]                  # a no-op, then the move
        counted.append((int(j), e))
    recs = recs[:9] + [(-1, -1), (recs[3][0], 2), (p.n, 1), (recs[1][0], 3)] + recs[9:]
    recs = recs[:31] + [(recs[1][0], 3 - recs[1][1])]       # the last: the first pixel once more
    seen = {j for j, e in recs if 0 <= j < p.n and 0 < e < 3}
    counted = [c for c in counted if c[0] in seen]
    a, b = _job(p), _job(p)
    for job, rs in ((a, recs), (b, counted)):
        job.init()
        for t, (j, e) in enumerate(rs):
            job.set_pick(j, e, slot=t)
        job.apply_rank_k(len(rs), precision=L.GFO_FP32)
    assert len(recs) == 32 and np.array_equal(a.history(), b.history())
    assert [tuple(x) for x in a.history()] == counted
    for x, y in zip(a.host_state(), b.host_state()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n_eps", [3, 4, 5, 7])
def test_topk_selection_materials(n_eps):
    """A kernel for each of two, three and four materials, one for more (its loads clamped
    to the table's last entry)."""
    test_topk_selection_edges(21, 37, n_eps, 14, 4, 1e-9)
    test_topk_selection_edges(21, 37, n_eps, 9, 3, 0.02)
