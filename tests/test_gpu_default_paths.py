"""The full workload sizes with the default options, element by element against the FP64 oracle: what the library
takes by itself (the row-scan sweep in its forms for full GPUs, the contraction on planes in every tile width,
the large-tile combine over many planes), where test_gpu_fullsize names the strip sweep."""
import numpy as np
import pytest

import parity

import rom_inputs as RI
from test_gpu_fullsize import c5_subset, mirror_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_12527_amd import rom
    rom.lib()
    return rom


def test_c3_full_size(R, orc):
    wl = RI.c3()
    f = wl.fields[0]
    h = R.Handle(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
    o = R.si_opts(tol=wl.tol, max_iter=wl.max_iter)
    phis, st, rc = h.ensemble_samples(wl.samples, wl.seed, R.ROM_ORD_STRATIFIED, 4, 8, opts=o)
    assert rc == 0 and st.lanes == 1 and st.band == 16
    mean, var, est, rc = h.ensemble(wl.samples, wl.seed, R.ROM_ORD_STRATIFIED, 4, 8, o)
    assert rc == 0 and est.lanes == 1
    m = phis.mean(axis=0)
    v = ((phis - m) ** 2).sum(axis=0) / (wl.samples - 1)
    assert np.max(np.abs(mean - m)) <= 1e-12 * np.max(np.abs(m))
    assert np.max(np.abs(var - v)) <= 1e-10 * np.max(np.abs(v))
    assert mirror_err(mean, f.nx) < 1e-5
    p = orc.Problem(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
    for k in (0, 21, 42, 63):
        d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, 4, 8, seed=wl.seed, sample=k)
        ref = orc.source_iterate(p, d, w, None, tol=wl.tol)
        parity.check(phis[k], ref["phi"], 1e-5, what=f"c3 sample {k}")


def test_c4_full_size(R):
    """Three iterations against the strip sweep's (FP32 sources, BF16 angular flux on both sides)."""
    wl = RI.c4()
    f = wl.fields[0]
    d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, 16, 16, seed=wl.seed)
    h = R.Handle(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
    h.set_scattering(R.ROM_SCAT_HG, wl.g)
    h.set_ordinates(d, w)
    phi, st, rc = h.source_iterate(R.si_opts(tol=wl.tol, max_iter=wl.max_iter))
    assert rc == 0 and st.lanes == 1 and st.final_r <= wl.tol
    assert mirror_err(phi, f.nx) < 1e-4
    got, st, _ = h.source_iterate(R.si_opts(tol=-1, max_iter=3))
    assert st.lanes == 1
    ref, st, _ = h.source_iterate(R.si_opts(tol=-1, max_iter=3, tile=(8, 4), band=4, sweep=R.ROM_SWEEP_STRIP))
    assert st.lanes != 1
    parity.check(got, ref, 2e-3, what="c4 against the strip sweep")


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
    outs, stats, rc = R.solve_batch(hs, R.si_opts(tol=wl.tol, max_iter=wl.max_iter))
    assert rc == 0 and all(s.status == 0 and s.lanes == 1 for s in stats)
    for k in c5_subset(wl):
        f = wl.fields[k]
        print(f"c5 problem {k}: {f.nx}x{f.ny}, n = {wl.n_ord[k]}", flush=True)
        p = orc.Problem(f.nx, f.ny, f.sigma_t, f.sigma_s, f.q)
        parity.si_check(orc, p, sets[k][0], sets[k][1], None, outs[k], stats[k].iters, wl.tol, 1e-5, what=f"c5 problem {k}")


# The BF16 contraction on planes, each tile width with a last tile of cells and of ordinates that is not full, and its
# sources stored through and past the caches (the latter where they and the fluxes exceed 256 MiB).  256 ordinates wide
# where 128-cell tiles then give every CU two blocks, else 128, else 64: 33123 cells x 320 padded ordinates
# are 259 x 2 tiles of 256, x 160 as many of 128; 140621 x 320 and 283513 x 160 exceed the caches, and so do
# 1431311 x 32, on 64-wide tiles.  (The 64-wide ones through the caches are those of test_gpu_scan.)
@pytest.mark.parametrize("nx,ny,n", [(181, 183, 300), (181, 183, 140), (377, 373, 300), (509, 557, 140), (511, 2801, 28)])
def test_contraction_tiles(R, orc, nx, ny, n):
    rng = np.random.default_rng([nx, ny, n])
    st = np.repeat(rng.uniform(0.5, 4.0, -(-ny // 9)), 9)[:ny, None] * np.ones(nx)
    ss, q = st * rng.uniform(0.2, 0.9, (ny, nx)), rng.uniform(0.0, 1.0, (ny, nx))
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=n)
    h = R.Handle(nx, ny, st, ss, q)
    h.set_ordinates(d, w)
    h.set_scattering(R.ROM_SCAT_HG, 0.7)
    phi, s, _ = h.source_iterate(R.si_opts(tol=-1, max_iter=3))
    assert s.lanes == 1
    ref = orc.source_iterate(orc.Problem(nx, ny, st, ss, q), d, w, orc.build_W(d, w, orc.SCAT_HG, 0.7, fold=1), tol=-1, max_iter=3)
    parity.check(phi, ref["phi"], 2e-3)


# The combine over large tiles with more than eight partial planes: from 2.1 million cells in FP32, 1.05 in FP64.
@pytest.mark.parametrize("prec,t,p2", [("fp32", 8, 8), ("fp64", 4, 5)])
def test_large_tiles_over_many_planes(R, orc, prec, t, p2):
    nx = ny = 512
    rng = np.random.default_rng(t)
    st = np.where((np.arange(nx)[None, :] // 73 + np.arange(ny)[:, None] // 73) % 2 == 0, 1.0, 6.0)
    ss, q = 0.6 * st, rng.uniform(0.0, 1.0, (ny, nx))
    h = R.Handle(nx, ny, st, ss, q)
    fp64 = prec == "fp64"
    o = R.si_opts(tol=-1, max_iter=3, precision=R.ROM_PREC_FP64 if fp64 else R.ROM_PREC_FP32)
    phis, s, _ = h.ensemble_samples(t, 3, R.ROM_ORD_STRATIFIED, 4, p2, opts=o)
    assert s.lanes == 1 and s.band == 4   # four ordinates a plane: p2 of them in each quadrant
    p = orc.Problem(nx, ny, st, ss, q)
    for k in range(t):
        d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, 4, p2, seed=3, sample=k)
        parity.check(phis[k], orc.source_iterate(p, d, w, None, tol=-1, max_iter=3)["phi"], 1e-11 if fp64 else 1e-5)
