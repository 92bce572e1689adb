"""init_G0 at the edges of its blocks: rows in fours within a grid row, two columns
per thread across the end of a grid row, the monitor columns, grids taller than one
launch's row blocks."""
import numpy as np
import pytest

from oracle import greens, state as ost
import workloads as W
from parity import rel_elem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("ny,nx,n_mon", [(1, 1, 1), (5, 1, 2), (1, 3, 1), (3, 4, 3), (4, 5, 1),
                                         (7, 7, 4), (2, 257, 2), (9, 63, 5), (129, 4, 2)])
@pytest.mark.parametrize("kw", [{}, {"delay": 16}, {"delay": 16, "packed": True}])
def test_fill_edges(dtype, ny, nx, n_mon, kw):
    """Tolerance: an entry is one FP64 Bessel value, off by a few u of its size near
    1 (arguments up to 1e2 add 1e2 u; against the floor of 1e-3 of the largest entry
    that is 1e5 u = 1e-11), rounded once to storage (complex64: 2^-24 per part)."""
    from paper_2202_05388_amd.job import Job
    p = W.tiny(ny, nx, n_mon=n_mon, dtype=dtype)
    print(f"[case] {ny}x{nx} mon={n_mon} {dtype} {kw}", flush=True)
    job = Job(p, device="cuda:0", **kw)
    job.init()
    G, E, d, idx = job.host_state()
    G0 = greens.build_G0(p)
    tol = 1e-11 if dtype == "c128" else 2e-7
    assert G.shape == G0.shape and rel_elem(G, G0) <= tol
    assert rel_elem(E, ost.dense_state(p, ost.eps_of(p, idx))[1]) <= tol
    assert rel_elem(d, np.diagonal(G0[:p.n])) <= 1e-11
    assert (idx == 0).all() and job.status() == 0


def test_fill_taller_than_one_launch():
    """66,000 rows of one pixel: more row blocks than the launch has workgroups.
    G[p, q] depends on |p - q| alone and comes from the same table entry: equal bits."""
    import torch
    from paper_2202_05388_amd.job import Job
    p = W.tiny(66000, 1, n_mon=1, dtype="c64")
    job = Job(p, device="cuda:0", delay=16)
    job.init()
    torch.cuda.synchronize()
    N = p.n
    for r in (1, 3, 4, 511, 65023, 65027, 65028, 65534, 65535, 65536, N - 1):
        assert torch.equal(job.G[r, r:N], job.G[0, :N - r]), r


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n_mon", [1, 63, 64, 65, 130])
def test_monitor_counts(dtype, n_mon):
    """Monitors as a kernel argument (up to 64) and through a copy: the matrix as above,
    and the coordinates that a refresh of one flipped pixel reads afterwards."""
    import torch
    from paper_2202_05388_amd.job import Job
    p = W.tiny(6, 9, n_mon=n_mon, dtype=dtype)
    print(f"[case] n_mon {n_mon} {dtype}", flush=True)
    job = Job(p, device="cuda:0", kmax=1)
    job.init()
    tol = 1e-11 if dtype == "c128" else 3e-7
    assert rel_elem(job.host_state()[0], greens.build_G0(p)) <= tol
    idx = np.zeros(p.n, np.uint8)
    idx[17] = 1
    job.eps_idx.copy_(torch.from_numpy(idx))
    job.refresh()
    G, E, _, _ = job.host_state()
    Gd, Ed = ost.dense_state(p, ost.eps_of(p, idx))
    assert rel_elem(G, Gd) <= tol and rel_elem(E, Ed) <= tol and job.status() == 0


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("ny,nx", [(1, 1025), (257, 1), (513, 1), (2, 511), (3, 171), (512, 2)])
@pytest.mark.parametrize("kw", [{}, {"delay": 16}, {"delay": 16, "packed": True}])
def test_fill_block_edges(dtype, ny, nx, kw):
    """Around the ends of a workgroup's columns (complex64 512, complex128 256), and a grid
    of one column (filled as one of one row).  Tolerance as above."""
    from paper_2202_05388_amd.job import Job
    p = W.tiny(ny, nx, n_mon=2, dtype=dtype)
    print(f"[case] {ny}x{nx} {dtype} {kw}", flush=True)
    job = Job(p, device="cuda:0", **kw)
    job.init()
    assert rel_elem(job.host_state()[0], greens.build_G0(p)) <= (1e-11 if dtype == "c128" else 2e-7)


def test_fill_walks_the_segments():
    """53,334 rows of three pixels, band-packed (102 GB): more pairs of segments than the
    launch has lines of workgroups.  G[p, q] of pixels the same distance apart comes from the
    same table entry: equal bits."""
    import torch
    from paper_2202_05388_amd.job import Job
    p = W.tiny(53334, 3, n_mon=1, dtype="c64")
    torch.cuda.empty_cache()
    job = Job(p, device="cuda:0", delay=16, packed=True)
    job.init()
    torch.cuda.synchronize()
    bands = job._bands()

    def row(r, n):                       # entries [r, r + n) of design row r
        r0, _, c0, off, stride = bands[r // 64]
        at = off + (r - r0) * stride + r - c0
        return job.G[at: at + n]
    N = p.n
    for iy in (0, 1, 2, 12345, 26626, 26627, 26666, 26667, 26668, 26706, 26707, 40000, 53332, 53333):
        for ix in range(3):
            n = N - 3 * iy - ix
            assert torch.equal(row(3 * iy + ix, n), row(ix, n)), (iy, ix)
