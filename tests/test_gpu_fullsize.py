"""Parity at the full workload sizes, in launch shapes of the strip sweep named here (the default
paths, which take the row-scan sweep, are in test_gpu_default_paths.py), element by element against
the FP64 oracle:

* c3 (512 x 512, 64 samples of 128 stratified ordinates): every one of the 64 per-sample fluxes
  and the ensemble's FP64 mean and variance against the oracle's ensemble over the same
  bit-identical sample sets; mirror symmetry of the mean;
* c4 (1024 stratified ordinates, HG g = 0.8 folded, BF16 contraction, tile 8 x 4, band 4): the
  full 256 x 256 solve converges and is mirror symmetric; on a 128 x 128 grid (128 GEMM row
  tiles of 128 cells) three iterations against the oracle's three, and the same set on a ragged
  20 x 20 grid to convergence;
* c5 (200 uneven problems in one persistent launch): a fixed stratified subset of the problems
  (the median problem of each eighth of the cost ranking, the largest problem and a 1024-side
  problem with n >= 400) against the oracle, every problem converged.
"""
import numpy as np
import pytest

import parity
from parity import nrm

import rom_inputs as RI

pytestmark = pytest.mark.gpu

C3_TILE, C3_BAND = (16, 16), 4
C4_TILE, C4_BAND = (8, 4), 4
C5_TILE, C5_BAND = (16, 16), 4


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_12527_amd import rom
    rom.lib()
    return rom


def mirror_err(phi, n):
    P = np.asarray(phi).reshape(n, n)
    return max(nrm(P[:, ::-1], P), nrm(P[::-1, :], P))


def c5_subset(wl):
    """Fixed stratified subset of c5: problems ranked by cells x ordinates, the median problem of
    each eighth of the ranking, plus the costliest problem and the costliest problem with a
    1024-cell side and at least 400 ordinates (deduplicated, ascending cost)."""
    cost = np.array([f.cells * wl.n_ord[k] for k, f in enumerate(wl.fields)])
    order = np.argsort(cost, kind="stable")
    pick = [int(order[(2 * s + 1) * len(order) // 16]) for s in range(8)]
    pick.append(int(order[-1]))
    wide = [int(k) for k in order if max(wl.fields[k].nx, wl.fields[k].ny) == 1024 and wl.n_ord[k] >= 400]
    pick.append(wide[-1])
    return sorted(set(pick), key=lambda k: cost[k])


def test_c3_full_size(R, orc):
    wl = RI.c3()
    f = wl.fields[0]
    h = R.Handle(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
    o = R.si_opts(tol=wl.tol, max_iter=wl.max_iter, tile=C3_TILE, band=C3_BAND, sweep=R.ROM_SWEEP_STRIP)
    phis, st, rc = h.ensemble_samples(wl.samples, wl.seed, R.ROM_ORD_STRATIFIED, 4, 8, opts=o)
    assert rc == 0 and phis.shape == (64, f.nx * f.ny)
    mean, var, est, rc = h.ensemble(wl.samples, wl.seed, R.ROM_ORD_STRATIFIED, 4, 8, o)
    assert rc == 0
    # the ensemble call and the per-sample call solve the same samples with the same kernels
    m = phis.mean(axis=0)
    v = ((phis - m) ** 2).sum(axis=0) / (wl.samples - 1)
    assert np.max(np.abs(mean - m)) <= 1e-12 * np.max(np.abs(m))
    assert np.max(np.abs(var - v)) <= 1e-10 * np.max(np.abs(v))
    assert mirror_err(mean, f.nx) < 1e-5
    # every sample, the mean and the variance against the oracle's ensemble (same sample sets)
    p = orc.Problem(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
    ref = orc.ensemble(p, orc.ORD_STRATIFIED, 4, 8, wl.seed, wl.samples, tol=wl.tol, want_phis=True)
    for k in range(wl.samples):
        parity.check(phis[k], ref["phis"][k], 1e-5, what=f"c3 sample {k}")
    parity.check(mean, ref["mean"], 1e-5, what="c3 mean")
    # FP32 per-sample fluxes (relative error ~1e-6) enter the variance through phi_s - mean,
    # which is a few per cent of phi here: about 2e-6 / 0.03 relative at worst per cell; the
    # FP32 bar normwise (measured 3e-7)
    parity.check(var, ref["var"], 1e-5, cell_tol=1e-4, what="c3 variance")


def test_c4_full_size(R, orc):
    wl = RI.c4()
    f = wl.fields[0]
    h = R.Handle(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
    h.set_scattering(R.ROM_SCAT_HG, wl.g)
    d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, 16, 16, seed=wl.seed)
    assert len(w) == 1024
    h.set_ordinates(d, w)
    o = R.si_opts(tol=wl.tol, max_iter=wl.max_iter, tile=C4_TILE, band=C4_BAND, sweep=R.ROM_SWEEP_STRIP)
    phi, st, rc = h.source_iterate(o)
    assert rc == 0 and st.final_r <= wl.tol
    assert mirror_err(phi, f.nx) < 1e-4  # BF16 angular flux in the contraction
    W = orc.build_W(d, w, orc.SCAT_HG, wl.g, fold=1)
    # 128 x 128: the [16384 x 1024] x [1024 x 1024] BF16 contraction in 128 row tiles, three
    # iterations on both sides
    g = RI.uniform_fields(128, 128, 1.0, 0.8, 0.45, 0.55)
    hm = R.Handle(g.nx, g.ny, g.sigma_t, g.sigma_s, g.q)
    hm.set_scattering(R.ROM_SCAT_HG, wl.g)
    hm.set_ordinates(d, w)
    o3 = R.si_opts(tol=-1.0, max_iter=3, tile=C4_TILE, band=C4_BAND, sweep=R.ROM_SWEEP_STRIP)
    phi_m, st_m, rc = hm.source_iterate(o3)
    assert rc == R.ROM_NOT_CONVERGED and st_m.iters == 3
    pm = orc.Problem(g.nx, g.ny, g.sigma_t, g.sigma_s, g.q)
    ref = orc.source_iterate(pm, d, w, W, tol=-1.0, max_iter=3)
    parity.check(phi_m, ref["phi"], 2e-3, what="c4 path 128x128, 3 iterations")
    # the same ordinate set, kernel, precision and launch shape to convergence on a ragged grid
    g = RI.uniform_fields(20, 20, 1.0, 0.8, 0.45, 0.55)
    hs = R.Handle(g.nx, g.ny, g.sigma_t, g.sigma_s, g.q)
    hs.set_scattering(R.ROM_SCAT_HG, wl.g)
    hs.set_ordinates(d, w)
    phi_s, st_s, rc = hs.source_iterate(o)
    assert rc == 0
    p = orc.Problem(g.nx, g.ny, g.sigma_t, g.sigma_s, g.q)
    parity.si_check(orc, p, d, w, W, phi_s, st_s.iters, wl.tol, 2e-3, what="c4 path 20x20")


def test_c5_full_size(R, orc):
    wl = RI.c5()
    hs, sets = [], []
    for k, f in enumerate(wl.fields):
        h = R.Handle(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
        nz, nt = orc.stratified_spec(wl.n_ord[k])
        d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, nz, nt, seed=wl.problem_seed(k))
        h.set_ordinates(d, w)
        hs.append(h)
        sets.append((d, w))
    o = R.si_opts(tol=wl.tol, max_iter=wl.max_iter, tile=C5_TILE, band=C5_BAND, sweep=R.ROM_SWEEP_STRIP)
    outs, stats, rc = R.solve_batch(hs, o)
    assert rc == 0 and all(s.status == 0 for s in stats)
    sub = c5_subset(wl)
    assert len(sub) >= 8
    assert any(max(wl.fields[k].nx, wl.fields[k].ny) == 1024 and wl.n_ord[k] >= 400 for k in sub)
    for k in sub:
        f = wl.fields[k]
        print(f"c5 problem {k}: {f.nx}x{f.ny}, n = {wl.n_ord[k]}", flush=True)
        p = orc.Problem(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
        parity.si_check(orc, p, sets[k][0], sets[k][1], None, outs[k], stats[k].iters, wl.tol, 1e-5,
                        what=f"c5 problem {k}")
