"""The refresh product's tiles: whole ones of design rows, ragged ones, ones that hold
monitor rows; pixel coordinates on grids from one column to one row."""
import numpy as np
import pytest

from oracle import greens, state as ost
import workloads as W
from parity import rel_elem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("ny,nx,n_mon,flips,kw", [
    (1, 130, 1, 5, {}), (130, 1, 2, 4, {}), (64, 3, 64, 13, {"delay": 16}), (16, 16, 65, 60, {}),
    (33, 8, 3, 31, {"delay": 16, "packed": True}), (20, 19, 130, 100, {"upper": True})])
def test_refresh_tiles(dtype, ny, nx, n_mon, flips, kw):
    """Tolerance: 100 u kappa of the core, u = 2^-53, as two FP64 solves of one system
    differ by a modest multiple of u kappa (complex64: plus one rounding); at least
    1e-11, what the Bessel functions of two libraries differ by against the floor of
    1e-3 of the largest entry."""
    from paper_2202_05388_amd.job import Job
    p = W.tiny(ny, nx, n_mon=n_mon, dtype=dtype)
    print(f"[case] {ny}x{nx} n_mon {n_mon} {dtype} {flips} flipped {kw}", flush=True)
    rng = np.random.default_rng(ny + 7 * nx)
    idx = np.zeros(p.n, np.uint8)
    idx[rng.choice(p.n, flips, replace=False)] = 1
    job = Job(p, device="cuda:0", kmax=flips, **kw)
    job.init()
    import torch
    job.eps_idx.copy_(torch.from_numpy(idx))
    job.refresh()
    G, E, d, idx2 = job.host_state()
    eps = ost.eps_of(p, idx)
    Gd, Ed = ost.dense_state(p, eps)
    alpha = greens.alpha_of(p, eps)
    V = np.nonzero(alpha != 0)[0]
    kappa = np.linalg.cond(np.diag(1.0 / alpha[V]) - greens.build_G0(p)[np.ix_(V, V)])
    tol64 = max(1e-11, 100 * 2.0 ** -53 * kappa)
    tol = tol64 if dtype == "c128" else 3e-7 + tol64
    assert rel_elem(G, Gd) <= tol and rel_elem(E, Ed) <= tol
    assert rel_elem(d, np.diagonal(Gd[:p.n])) <= tol64
    assert np.array_equal(idx, idx2) and job.status() == 0


@pytest.mark.parametrize("ny,nx,n_mon,flips", [(64, 64, 33, 180), (83, 77, 5, 300)])
def test_c64_refresh_is_c128_rounded_once(ny, nx, n_mon, flips):
    """The refresh computes in FP64 with the same instructions for either storage type:
    complex64 storage holds the complex128 result rounded once, entry for entry, and the
    same FP64 diagonal."""
    import torch
    from paper_2202_05388_amd.job import Job
    print(f"[case] {ny}x{nx} n_mon {n_mon} {flips} flipped", flush=True)
    idx = np.zeros(ny * nx, np.uint8)
    idx[np.random.default_rng(flips).choice(ny * nx, flips, replace=False)] = 1
    jobs = []
    for dtype in ("c128", "c64"):
        job = Job(W.tiny(ny, nx, n_mon=n_mon, dtype=dtype), device="cuda:0", kmax=flips)
        job.init()
        job.eps_idx.copy_(torch.from_numpy(idx))
        job.refresh()
        jobs.append(job)
    a, b = jobs
    assert torch.equal(a.diag64, b.diag64)
    assert torch.equal(a.E.to(torch.complex64), b.E)
    assert int((a.G.to(torch.complex64) != b.G).sum()) == 0


def test_refresh_large_panel_product():
    """14,762 pixels, 1,034 of them flipped: Z = U M on the 128 x 128 tiles (1,044 of them),
    with ragged rows and columns and a last chunk of four k.  Every 100th design row and
    the monitor rows against G0 + G0[:, V] M G0[V, :] from the device's own G0.
    Tolerance as above: 100 u kappa."""
    import torch
    from paper_2202_05388_amd.job import Job
    p = W.tiny(122, 121, n_mon=5, dtype="c128")
    N, k = p.n, 1034
    idx = np.zeros(N, np.uint8)
    idx[np.random.default_rng(7).choice(N, k, replace=False)] = 1
    V = np.flatnonzero(idx)
    rows = np.concatenate([np.arange(3, N, 100), np.arange(N, N + 5)])
    print(f"[case] 122x121 c128, {k} flipped, {len(rows)} rows compared", flush=True)
    job = Job(p, device="cuda:0", kmax=k)
    job.init()
    at = torch.from_numpy(rows).cuda()
    G0V = job.G[torch.from_numpy(V).cuda(), :N].cpu().numpy()         # k x N, and its transpose by symmetry
    G0r, Einc = job.G[at, :N].cpu().numpy(), job.E.cpu().numpy()
    job.eps_idx.copy_(torch.from_numpy(idx))
    job.refresh()
    G, E, d = job.G[at, :N].cpu().numpy(), job.E.cpu().numpy()[rows], job.diag64.cpu().numpy()
    alpha = greens.alpha_of(p, ost.eps_of(p, idx))[V]
    core = np.diag(1.0 / alpha) - G0V[:, V]
    Z = np.linalg.solve(core.T, G0r[:, V].T).T
    Gd, Ed = G0r + Z @ G0V, Einc[rows] + Z @ Einc[V]
    tol = max(1e-12, 100 * 2.0 ** -53 * np.linalg.cond(core))
    own = rows[rows < N]
    err = [rel_elem(G, Gd), rel_elem(E, Ed), rel_elem(d[own], Gd[np.arange(len(own)), own])]
    print("G, E, diag64", *("%.3g" % e for e in err), "bound %.3g" % tol, flush=True)
    assert max(err) <= tol and job.status() == 0
