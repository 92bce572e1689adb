"""Region scores where the split over threads and the batches of pending terms end:
region counts around one workgroup's, up to eight materials, 1 to 40 pending terms,
more regions than one pass of the summaries."""
import numpy as np
import pytest

from oracle import regions as orr
from oracle import state as ost
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,n_eps,terms", [
    (2, 2, 2, 0), (2, 30, 5, 0), (2, 32, 4, 0), (2, 34, 8, 0), (2, 130, 8, 0), (10, 26, 3, 0),
    (16, 18, 2, 1), (16, 18, 2, 15), (16, 18, 6, 16), (16, 18, 2, 17), (18, 16, 8, 33), (16, 18, 2, 40)])
def test_region_scores_at_the_edges(ny, nx, n_eps, terms):
    """Tolerance as for any FP64 solve of a 4 x 4 system of condition below 1e3:
    1e-10 of each score.  The pick is the lowest index within the tie band."""
    from paper_2202_05388_amd.job import Job
    from paper_2202_05388_amd import _lib as L
    table = (1.0, 12.25, 2.25, 4.0, 6.0, 1.5, 9.0, 3.0)[:n_eps]
    p = W.tiny(ny, nx, n_mon=3, pitch=0.025, mon_distance=0.5, dtype="c128", tau=1e-9, region=2,
               cand_mask=W.MASK_BOTH).replace(eps_table=table)
    print(f"[case] {ny}x{nx} n_eps {n_eps} terms {terms}", flush=True)
    idx = np.random.default_rng(ny * nx + n_eps).integers(0, n_eps, p.n).astype(np.uint8)
    job = Job(p, device="cuda:0", delay=64 if terms else 0)
    job.init()
    G, E = ost.dense_state(p, ost.eps_of(p, idx))
    job.upload_state(G, E, np.diagonal(G[: p.n]).copy(), idx)
    if terms:
        job.run_greedy(terms, poll_every=terms)
        assert job.state.pending_calls == terms
        idx = job.eps_idx.cpu().numpy()
    mask = (1 << n_eps) - 1
    fom = job.fom()
    L.score_regions(job.prob, job.state, 2, mask, p.tau, job.picks.data_ptr(), 0)
    q = p.replace(cand_mask=mask)
    ev = orr._RegionEvaluator(q, 2, "T1")
    Eo, row, G_VV = ev(idx)
    F = orr.region_scores(q, 2, Eo, G_VV, row, idx)
    K = orr.n_regions(q, 2)
    F_gpu = job.scores().reshape(-1)[: K * n_eps].reshape(K, n_eps)
    fin = np.isfinite(F)
    assert np.array_equal(np.isfinite(F_gpu), fin)
    assert np.allclose(F_gpu[fin], F[fin], rtol=1e-10, atol=0)
    best = F_gpu.max()
    pixel, e, fom_new, _ = job.read_picks(1)[0]
    if best > fom * (1 + p.tau):
        band = best - p.tau * abs(best)
        first = int(np.nonzero(F_gpu.reshape(-1) >= band)[0][0])
        assert (pixel, e) == divmod(first, n_eps) and fom_new == F_gpu.reshape(-1)[first]
    else:
        assert pixel == -1
    assert job.status() == 0


def test_more_regions_than_one_pass():
    """16,500 regions: two sixteens per workgroup.  In the empty design every region has
    the same 4 x 4 block; the scores are a batched FP64 solve on the host of the stored
    complex64 entries, the same data: 1e-9 of each score (condition below 1e3)."""
    from paper_2202_05388_amd.job import Job
    from paper_2202_05388_amd import _lib as L
    p = W.tiny(2, 33000, n_mon=1, pitch=0.025, mon_distance=0.5, dtype="c64", tau=1e-6, region=2,
               cand_mask=W.MASK_BOTH)
    job = Job(p, device="cuda:0", delay=16)
    job.init()
    L.score_regions(job.prob, job.state, 2, p.cand_mask, p.tau, job.picks.data_ptr(), 0)
    N, nx = p.n, p.nx
    V = np.array([[2 * b, 2 * b + 1, nx + 2 * b, nx + 2 * b + 1] for b in range(nx // 2)])
    top = job.G[0:2, :N].cpu().numpy().astype(np.complex128)       # rows 0 and 1: pixels (0, 0), (0, 1)
    d = complex(job.diag64[0].cpu())
    h, v, x, y = top[0, 1], top[0, nx], top[0, nx + 1], top[1, nx]
    block = np.array([[d, h, v, x], [h, d, y, v], [v, y, d, h], [x, v, h, d]])
    row = job.G[N, :N].cpu().numpy().astype(np.complex128)
    E = job.E.cpu().numpy().astype(np.complex128)
    b = (2 * np.pi / p.wavelength) ** 2 * (p.eps_table[1] - p.eps_table[0])
    sol = np.linalg.solve(np.eye(4) - b * block, E[V].T).T
    F = np.abs(E[N] + b * (row[V] * sol).sum(axis=1)) ** 2
    F_gpu = job.scores().reshape(-1)[: 2 * len(V)].reshape(-1, 2)
    assert np.isneginf(F_gpu[:, 0]).all() and np.allclose(F_gpu[:, 1], F, rtol=1e-9, atol=0)
    best = F_gpu.max()
    pixel, e, fom_new, _ = job.read_picks(1)[0]
    first = int(np.nonzero(F_gpu[:, 1] >= best - p.tau * best)[0][0])
    assert best > job.fom() * (1 + p.tau) and (pixel, e) == (first, 1) and fom_new == F_gpu[first, 1]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("table", [(1.0, 12.25), (1.0, 12.25, 5.0)])
@pytest.mark.parametrize("ny,nx,moves,kw", [
    (130, 128, 0, {}),                                # 4160 regions, the last workgroup partial
    (130, 128, 1, {"delay": 16, "packed": True}),     # one pending term
    (130, 130, 5, {"delay": 16}),                     # a last batch of one term (complex64: a thread per region)
    (258, 256, 40, {"delay": 64, "packed": True})])   # beyond 16384 regions: two sixteens per workgroup
def test_region_forms_agree(dtype, table, ny, nx, moves, kw):
    """The thread-per-region form (many regions, few terms, two or three materials) and the
    form of twelve threads per region: a table with two more entries that are no
    candidates takes the other one, with the same scores, bit for bit."""
    import torch
    from paper_2202_05388_amd import _lib as L
    from paper_2202_05388_amd.job import Job
    if dtype == "c128" and moves == 5:
        pytest.skip("complex128 takes one form for both tables there")
    print(f"[case] {ny}x{nx} {dtype} {len(table)} materials, {moves} terms, {kw}", flush=True)
    got = []
    n = (ny // 2) * (nx // 2)
    for eps in (table, table + (2.0, 3.0)):
        p = W.tiny(ny, nx, n_mon=3, dtype=dtype, eps_table=eps, cand_mask=(1 << len(table)) - 1, tau=1e-6)
        job = Job(p, device="cuda:0", **kw)
        job.init()
        for i in range(moves):
            job.set_pick(977 * (i + 1) % p.n, 1)
            job.apply()
        assert job.state.pending_calls == moves
        L.score_regions(job.prob, job.state, 2, p.cand_mask, p.tau, job.picks.data_ptr(),
                        torch.cuda.current_stream().cuda_stream)
        off = L.scores_offset(job.prob, job.kmax, job.ld)
        s = job.work[off: off + 8 * n * len(eps)].view(torch.float64).view(n, len(eps))
        got.append((s[:, :len(table)].clone(), job.read_picks(1)[0], job.status()))
        del job
    (sa, pa, ta), (sb, pb, tb) = got
    assert torch.equal(sa, sb) and pa == pb and ta == tb == 0 and pa[0] >= 0
