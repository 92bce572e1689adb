"""The refresh's blocked inverse at the edges of its panel sizes: one row per thread
up to 512 flipped pixels (panels of 16 columns), two, three and four per thread up to
1024, 1536 and 2048 (panels of 32 in subpanels of 8), one launch per column beyond; the last panel
partial or whole, fewer rows than a wave and more.  A mirror-symmetric structure
has rows of equal modulus, so pivots are chosen among exact ties.

The reference is the dense re-solve from the device's own G0 (held to the oracle's
at 1e-13 by the init tests): kappa also multiplies the last bits in which the two
Bessel libraries differ, which here come to more than the solves' own rounding.

Tolerance: 100 u kappa of the core, as for the other large flipped sets (two FP64
solves of one system differ by a modest multiple of u kappa), at least 1e-12.
"""
import numpy as np
import pytest

from oracle import greens, state as ost
from parity import rel_elem as _rel
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,k,mirror", [
    (1, 3, 2, False),          # kp = 4: fewer rows than the panel is wide
    (5, 7, 16, False),         # one whole panel
    (5, 7, 17, False),         # kp = 20: a second panel of 4 columns
    (9, 9, 64, True),
    (9, 9, 66, True),          # a second wave with 4 rows
    (24, 24, 512, False),      # eight waves, the last of one row per thread
    (24, 24, 513, True),       # two rows per thread, kp = 516: a last panel of 4 columns
    (31, 32, 900, True),
    (33, 33, 1024, False),     # eight waves of two rows, all full
    (33, 33, 1025, True),      # three rows per thread
    (36, 35, 1153, False),     # seven waves of three rows, kp = 1156
    (40, 39, 1536, False),
    (40, 40, 1540, True),      # four rows per thread
    (47, 45, 2050, False),     # beyond 2048: one launch per column
])
def test_refresh_panel_edges(ny, nx, k, mirror):
    import torch
    from paper_2202_05388_amd.job import Job
    p = W.tiny(ny, nx, n_mon=5, dtype="c128")
    N = p.n
    if mirror:
        idx = W.mirror_symmetric_eps_idx(p, k / N, 5)
    else:
        idx = np.zeros(N, np.uint8)
        idx[np.random.default_rng(k).choice(N, k, replace=False)] = 1
    V = np.flatnonzero(idx)
    print(f"[case] {ny}x{nx} k={len(V)} mirror={mirror}", flush=True)
    job = Job(p, device="cuda:0", kmax=len(V))
    job.init()
    G0 = job.host_state()[0]
    job.eps_idx.copy_(torch.from_numpy(idx))
    job.refresh()
    G, E, d, _ = job.host_state()
    eps = ost.eps_of(p, idx)
    Gd, Ed = ost.dense_state(p, eps, G0)
    core = np.diag(1.0 / greens.alpha_of(p, eps)[V]) - G0[np.ix_(V, V)]
    tol = max(1e-12, 100 * 2.0 ** -53 * np.linalg.cond(core))
    print(f"G {_rel(G, Gd):.3g}, E {_rel(E, Ed):.3g}, bound {tol:.3g}", flush=True)
    assert job.status() == 0
    assert _rel(G, Gd) <= tol and _rel(E, Ed) <= tol
    assert _rel(d, np.diagonal(Gd[:N])) <= tol


@pytest.mark.parametrize("k", [600, 1100, 1600])   # two, three and four rows per thread
def test_refresh_panels_repeat(k):
    """The panels pass a wave's rows between its lanes through LDS: the same structure
    gives the same bits, whatever ran before on the same buffers."""
    import torch
    from paper_2202_05388_amd.job import Job
    p = W.tiny(41, 43, n_mon=5, dtype="c128")
    job = Job(p, device="cuda:0", kmax=k)
    job.init()
    runs = []
    for seed in (1, 2, 1):
        idx = np.zeros(p.n, np.uint8)
        idx[np.random.default_rng(seed).choice(p.n, k, replace=False)] = 1
        job.eps_idx.copy_(torch.from_numpy(idx))
        print(f"[case] repeat k={k}, structure {seed}", flush=True)
        job.refresh()
        runs.append([x.clone() for x in (job.G, job.E, job.diag64)])
    assert job.status() == 0
    assert all(torch.equal(a, b) for a, b in zip(runs[0], runs[2]))
