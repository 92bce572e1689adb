"""The split-product flush over lists of tiles long enough that an XCD's workgroups
walk them in rounds, and at 65 to 128 terms (one workgroup per compute unit), against
the pair flush: upper triangle and monitor rows after the same moves."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,n_mon,steps,delay,packed", [
    (30, 34, 70, 66, 128, False),      # fewer tiles than workgroups, two monitor bands
    (30, 34, 70, 66, 128, True),
    (64, 64, 1, 80, 128, True),        # some 8 to 9 tiles per workgroup, one cut
    (128, 128, 64, 100, 128, False),   # rounds of 16 tiles, then the even cut
    (129, 130, 65, 70, 96, True),      # the same, ragged
    (184, 184, 16, 20, 32, False),     # rounds of 32 tiles at two workgroups per compute unit
])
def test_rounds_equal_pair_flush(ny, nx, n_mon, steps, delay, packed):
    """Tolerance: K terms summed in FP32 in another order and from split products,
    each off by a few u of its size: 4 K u of the largest entry, u = 2^-24."""
    import torch
    from paper_2202_05388_amd import _lib as L
    from paper_2202_05388_amd.job import Job
    p = W.tiny(ny, nx, n_mon=n_mon, dtype="c64", cand_mask=W.MASK_BOTH, tau=1e-6)
    names = L.flush_variants()
    old = L.flush_get_variant()
    jobs = []
    try:
        for name in ("up_pair4_3m_nt", "up_bandseg_s3"):
            L.flush_set_variant(names.index(name))
            print(f"[case] {ny}x{nx} n_mon {n_mon}: {steps} moves, flush {name}, packed {packed}", flush=True)
            job = Job(p, device="cuda:0", delay=delay, packed=packed)
            job.init()
            job.run_greedy(steps, poll_every=steps)
            assert job.state.pending_calls == steps
            job.flush()
            torch.cuda.synchronize()
            jobs.append(job)
    finally:
        L.flush_set_variant(old)
    a, b = (j.G for j in jobs)
    tol = 4 * steps * 2.0 ** -24
    if packed:                       # the whole matrix as the caller reads it
        a, b = (torch.from_numpy(j.host_state()[0]) for j in jobs)
    N = p.n
    for r in range(0, a.shape[0], 1024):
        x, y = a[r:r + 1024, :N], b[r:r + 1024, :N]
        if r < N:                    # the design rows' upper triangle, the monitor rows whole
            keep = torch.arange(N, device=x.device)[None, :] >= torch.arange(r, r + x.shape[0], device=x.device)[:, None]
            keep |= (torch.arange(r, r + x.shape[0], device=x.device) >= N)[:, None]
            x, y = torch.where(keep, x, 0), torch.where(keep, y, 0)
        assert float((x - y).abs().max()) <= tol * float(x.abs().max()), r
    assert (jobs[0].history() == jobs[1].history()).all()


@pytest.mark.parametrize("ny,nx,n_mon,steps,delay,packed", [
    (7, 9, 1, 1, 16, False), (7, 9, 70, 8, 16, False), (8, 8, 64, 9, 64, True), (16, 20, 65, 31, 64, True),
    (24, 26, 3, 32, 64, False), (30, 34, 130, 33, 64, False), (64, 64, 2, 64, 128, True),
    (63, 65, 2, 65, 128, False), (96, 97, 70, 100, 128, True)])
def test_c128_flush_equals_eager(ny, nx, n_mon, steps, delay, packed):
    """complex128: the counts around the phases of 8 terms and the rounds of 32, one
    tile to several rounds of tiles per workgroup, ragged bands, one to three monitor
    bands.  Tolerance: K terms summed in FP64, each off by a few u of the largest entry,
    on either side: 8 K u, u = 2^-53."""
    import numpy as np
    from paper_2202_05388_amd.job import Job
    from parity import rel_elem
    p = W.tiny(ny, nx, n_mon=n_mon, dtype="c128", cand_mask=W.MASK_BOTH, tau=1e-9)
    print(f"[case] c128 {ny}x{nx} n_mon {n_mon}: {steps} moves, packed {packed}", flush=True)
    a = Job(p, device="cuda:0")
    a.init()
    a.run_greedy(steps, poll_every=steps)
    b = Job(p, device="cuda:0", delay=delay, packed=packed)
    b.init()
    b.run_greedy(steps, poll_every=steps)
    assert b.state.pending_calls == steps or delay == steps
    Gb, Eb, db, ib = b.host_state()
    Ga, Ea, da, ia = a.host_state()
    assert np.array_equal(ia, ib) and np.array_equal(a.history(), b.history())
    assert rel_elem(Gb, Ga, floor=1.0) <= 8 * steps * 2.0 ** -53


@pytest.mark.parametrize("ny,nx,n_mon,steps,packed", [
    (43, 44, 1, 8, False), (46, 47, 70, 33, True), (49, 50, 3, 20, False), (58, 59, 65, 33, False),
    (79, 80, 1, 5, True)])
def test_c128_tiled_flush_equals_eager(ny, nx, n_mon, steps, packed):
    """complex128 between one tile per workgroup of the persistent form and many: few
    terms, or an uneven share, a workgroup per tile.  Tolerance as above."""
    import numpy as np
    from paper_2202_05388_amd.job import Job
    from parity import rel_elem
    p = W.tiny(ny, nx, n_mon=n_mon, dtype="c128", cand_mask=W.MASK_BOTH, tau=1e-9)
    print(f"[case] c128 {ny}x{nx} n_mon {n_mon}: {steps} moves, packed {packed}", flush=True)
    a = Job(p, device="cuda:0")
    a.init()
    a.run_greedy(steps, poll_every=steps)
    b = Job(p, device="cuda:0", delay=64, packed=packed)
    b.init()
    b.run_greedy(steps, poll_every=steps)
    assert b.state.pending_calls == steps
    Gb, _, _, ib = b.host_state()
    Ga, _, _, ia = a.host_state()
    assert np.array_equal(ia, ib) and np.array_equal(a.history(), b.history())
    assert rel_elem(Gb, Ga, floor=1.0) <= 8 * steps * 2.0 ** -53
