"""GPU parity of the row-scan sweep kernel (chosen by librom only) against the FP64 oracle.

ROM_SWEEP_SCAN=k takes the k-th row-scan shape of a problem: the single-ordinate forms first, then
(FP32 isotropic step sweeps) the form for full GPUs with 8 and 16 wavefronts per workgroup.  Widths sit at
the edges of the shapes (lane groups of 16, 32 and 64, 1 to 16 cells per lane, one and two strips per
row, rows that end inside a 16-byte store), heights at the edges of a batch of rows; sigma_t changes
in every row, in bands of rows, or not at all.  Bars as in the other parity tests at a fixed iteration
count: FP32 1e-5 (per cell 1e-4), FP64 1e-11."""
import numpy as np
import pytest

import parity

pytestmark = pytest.mark.gpu

FACES = ("left", "right", "bottom", "top")


@pytest.fixture(scope="module")
def R():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_12527_amd import rom
    rom.lib()
    return rom


def problem(rng, nx, ny, medium):
    if medium == "random":
        st = rng.uniform(0.2, 8.0, (ny, nx))
    elif medium == "bands":
        st = np.repeat(rng.uniform(0.2, 8.0, -(-ny // 7)), 7)[:ny, None] * (1.0 + np.arange(nx) // 5 % 2)
    else:
        st = np.full((ny, nx), 1.3)
    return st.ravel(), (st * rng.uniform(0.0, 0.9, (ny, nx))).ravel(), rng.uniform(0.0, 1.0, nx * ny)


def shapes(fp64, nx):
    """How many row-scan shapes a problem of that width has."""
    return (2 if nx <= 128 else 1) + (0 if fp64 else 2)


def compare(R, orc, nx, ny, n, prec, medium, inflow, angular=False):
    rng = np.random.default_rng([nx, ny, n])
    st, ss, q = problem(rng, nx, ny, medium)
    infl = {f: rng.uniform(0, 1, ny if f in FACES[:2] else nx) for f in FACES} if inflow else None
    box = (0.0, 1.5, 0.0, 0.7)
    h = R.Handle(nx, ny, st, ss, q, box=box, inflow=infl)
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=nx + ny)
    h.set_ordinates(d, w)
    ang = None
    if angular:
        ang = {0: rng.uniform(0, 1, (n, ny)), 3: rng.uniform(0, 1, (n, nx))}
        for f, v in ang.items():
            h.set_inflow_angular(f, v)
    fp64 = prec == "fp64"
    phi, s, _ = h.source_iterate(R.si_opts(tol=-1, max_iter=4, precision=R.ROM_PREC_FP64 if fp64 else R.ROM_PREC_FP32))
    assert s.sweep == R.ROM_SWEEP_DIAG and s.lanes == 1  # a row-scan sweep
    assert s.sweeps == 4 and s.sweep_ms > 0
    p = orc.Problem(nx, ny, st, ss, q, box=box, inflow=infl, inflow_angular={FACES[f]: v for f, v in ang.items()} if ang else None)
    ref = orc.source_iterate(p, d, w, None, tol=-1, max_iter=4)["phi"]
    parity.check(phi, ref, 1e-11 if fp64 else 1e-5)


WIDTHS = [1, 3, 16, 63, 64, 65, 127, 128, 130, 192, 256, 257, 300, 320, 384, 385, 511, 512, 513, 700, 768, 769, 1023, 1024]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx", WIDTHS)
def test_widths(R, orc, monkeypatch, nx, prec):
    for k in range(shapes(prec == "fp64", nx)):
        monkeypatch.setenv("ROM_SWEEP_SCAN", str(k + 1))
        for ny, n, medium, inflow in ((33, 29, "random", False), (16, 41, "bands", True), (1, 3, "uniform", False)):
            compare(R, orc, nx, ny, n, prec, medium, inflow)


@pytest.mark.parametrize("ny", [2, 7, 8, 9, 23])
@pytest.mark.parametrize("nx,n", [(20, 70), (100, 140), (200, 9), (600, 33)])
def test_heights_and_angular_inflow(R, orc, monkeypatch, nx, ny, n):
    for k in range(shapes(False, nx)):
        monkeypatch.setenv("ROM_SWEEP_SCAN", str(k + 1))
        compare(R, orc, nx, ny, n, "fp32", "bands", False, angular=True)


@pytest.mark.parametrize("nx,ny", [(48, 31), (90, 20), (257, 12)])
def test_sixteen_wavefronts(R, orc, monkeypatch, nx, ny):
    n = 2052
    monkeypatch.setenv("ROM_SWEEP_SCAN", str(shapes(False, nx)))
    compare(R, orc, nx, ny, n, "fp32", "bands", True)


@pytest.mark.parametrize("k", [1, 2, 3])
def test_uneven_batch_and_new_ordinates(R, orc, monkeypatch, k):
    """A batch of every width class in one launch; then other ordinates (counts kept) on the same plan."""
    monkeypatch.setenv("ROM_SWEEP_SCAN", str(k))
    rng = np.random.default_rng(5)
    hs, ps, opts = [], [], R.si_opts(tol=-1, max_iter=3)
    for nx, ny in ((40, 19), (100, 33), (256, 9), (350, 21), (512, 8), (700, 17), (1024, 10)):
        st, ss, q = problem(rng, nx, ny, "bands")
        hs.append(R.Handle(nx, ny, st, ss, q))
        ps.append(orc.Problem(nx, ny, st, ss, q))
    for seed in (1, 2):
        sets = [R.generate_ordinates(R.ROM_ORD_STRATIFIED, 1 + i % 3, 3, seed=seed, sample=i) for i in range(len(hs))]
        for h, (d, w) in zip(hs, sets):
            h.set_ordinates(d, w)
        outs, stats, _ = R.solve_batch(hs, opts)
        for p, (d, w), phi, s in zip(ps, sets, outs, stats):
            assert s.lanes == 1
            parity.check(phi, orc.source_iterate(p, d, w, None, tol=-1, max_iter=3)["phi"], 1e-5)


@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_ensemble(R, orc, monkeypatch, k):
    monkeypatch.setenv("ROM_SWEEP_SCAN", str(k))
    rng = np.random.default_rng(9)
    st, ss, q = problem(rng, 50, 37, "bands")
    h = R.Handle(50, 37, st, ss, q)
    p = orc.Problem(50, 37, st, ss, q)
    for seed in (3, 4):  # the second call refreshes the plan's tables
        phis, s, _ = h.ensemble_samples(5, seed, R.ROM_ORD_STRATIFIED, 2, 3, opts=R.si_opts(tol=-1, max_iter=4))
        assert s.lanes == 1
        for i in range(5):
            d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, 2, 3, seed=seed, sample=i)
            parity.check(phis[i], orc.source_iterate(p, d, w, None, tol=-1, max_iter=4)["phi"], 1e-5)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kernel", ["linear", "normalized", "iso"])
@pytest.mark.parametrize("scheme", ["step", "dd"])
@pytest.mark.parametrize("nx,n", [(1, 5), (40, 12), (64, 37), (65, 16), (100, 50), (128, 7), (200, 21), (256, 4), (300, 18), (511, 9)])
def test_moment_planes_and_diamond_difference(R, orc, monkeypatch, nx, n, scheme, kernel, prec):
    """The linear kernel's three (normalized on an asymmetric set: four) moment planes, both schemes;
    up to 16 ordinates the 16-lane form has one wavefront per workgroup, above four."""
    if kernel == "iso" and scheme == "step":
        pytest.skip("test_widths")
    fp64 = prec == "fp64"
    rng = np.random.default_rng([nx, n])
    ny = 19
    st, ss, q = problem(rng, nx, ny, "random" if nx % 2 else "bands")
    inflow = {"left": rng.uniform(0, 1, ny), "top": rng.uniform(0, 1, nx)} if n % 3 else None
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=n)
    W = None
    if kernel != "iso":
        norm = kernel == "normalized"
        W = orc.build_W(d, w, orc.SCAT_LINEAR | (orc.SCAT_NORMALIZE if norm else 0), 0.8, fold=1)
    p = orc.Problem(nx, ny, st, ss, q, inflow=inflow)
    ref = orc.source_iterate(p, d, w, W, scheme=orc.SCHEME_DD if scheme == "dd" else orc.SCHEME_STEP, tol=0.0, max_iter=4)["phi"]
    o = R.si_opts(tol=-1, max_iter=4, precision=R.ROM_PREC_FP64 if fp64 else R.ROM_PREC_FP32,
                  scheme=R.ROM_SCHEME_DD if scheme == "dd" else R.ROM_SCHEME_STEP)
    for k in range(2 if nx <= 128 else 1):
        monkeypatch.setenv("ROM_SWEEP_SCAN", str(k + 1))
        h = R.Handle(nx, ny, st, ss, q, inflow=inflow)
        h.set_ordinates(d, w)
        if kernel != "iso":
            h.set_scattering(R.ROM_SCAT_LINEAR | (R.ROM_SCAT_NORMALIZE if norm else 0), 0.8)
        phi, s, _ = h.source_iterate(o)
        assert s.sweep == R.ROM_SWEEP_STRIP and s.lanes == 1
        parity.check(phi, ref, 1e-11 if fp64 else 1e-5)


def test_the_rule_repeats_itself(R):
    """The shape is a rule of sizes and media: equal problems sum in the same order, bit for bit."""
    rng = np.random.default_rng(3)
    for nx, ny, medium in ((40, 28, "random"), (130, 40, "bands"), (64, 64, "uniform")):
        f = problem(rng, nx, ny, medium)
        d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, 3, 4, seed=6)
        got = []
        for _ in range(2):
            h = R.Handle(nx, ny, *f)
            h.set_ordinates(d, w)
            phi, s, _ = h.source_iterate()
            assert s.lanes == 1
            got.append(phi)
        assert np.array_equal(*got)


# Dense kernels: a source plane per ordinate, the angular flux in planes of four (BF16) or one (FP64), the
# contraction on those planes.  Widths at the edges of the shapes, cell counts that end inside a
# 16-byte store and a 128-byte line, ordinates that leave part of a plane and of a K step.  A caller's unsymmetric kernel pins the contraction's orientation.  The
# bars of the other dense-kernel tests: 2e-3 with the BF16 contraction, 1e-11 in FP64.
@pytest.mark.parametrize("nx,ny,n,kind,inflow", [
    (1, 1, 1, "hg", False), (3, 5, 7, "dense", True), (63, 9, 33, "hg", True), (64, 31, 12, "dense", False),
    (65, 17, 70, "dense", True), (129, 8, 40, "hg", False), (200, 16, 300, "dense", True), (257, 7, 20, "dense", False),
    (385, 5, 9, "hg", True), (512, 6, 30, "dense", False)])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_dense_kernels(R, orc, monkeypatch, nx, ny, n, kind, inflow, prec):
    rng = np.random.default_rng([nx, ny, n])
    st, ss, q = problem(rng, nx, ny, "bands")
    infl = {f: rng.uniform(0, 1, ny if f in FACES[:2] else nx) for f in FACES} if inflow else None
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=nx)
    P = rng.uniform(0.2, 1.5, (n, n))
    W = orc.build_W(d, w, orc.SCAT_DENSE, P=P) if kind == "dense" else orc.build_W(d, w, orc.SCAT_HG, 0.7, fold=1)
    ref = orc.source_iterate(orc.Problem(nx, ny, st, ss, q, inflow=infl), d, w, W, tol=-1, max_iter=4)["phi"]
    fp64 = prec == "fp64"
    for k in range(2 if nx <= 64 else 1):
        monkeypatch.setenv("ROM_SWEEP_SCAN", str(k + 1))
        h = R.Handle(nx, ny, st, ss, q, inflow=infl)
        h.set_ordinates(d, w)
        h.set_scattering(R.ROM_SCAT_DENSE if kind == "dense" else R.ROM_SCAT_HG, 0.7, P if kind == "dense" else None)
        for check in (1, 4):   # replays of one iteration, and one replay: only the first starts from q
            o = R.si_opts(tol=-1, max_iter=4, precision=R.ROM_PREC_FP64 if fp64 else R.ROM_PREC_FP32, iters_per_check=check)
            phi, s, _ = h.source_iterate(o)
            assert s.lanes == 1 and s.band == 4
            parity.check(phi, ref, 1e-11 if fp64 else 2e-3)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_dense_batch_of_uneven_problems(R, orc, prec):
    rng = np.random.default_rng(8)
    hs, refs = [], []
    for nx, ny, n in ((40, 33, 12), (130, 9, 70), (65, 20, 300)):
        st, ss, q = problem(rng, nx, ny, "uniform")
        d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=n)
        h = R.Handle(nx, ny, st, ss, q)
        h.set_ordinates(d, w)
        h.set_scattering(R.ROM_SCAT_HG, 0.6)
        hs.append(h)
        refs.append(orc.source_iterate(orc.Problem(nx, ny, st, ss, q), d, w, orc.build_W(d, w, orc.SCAT_HG, 0.6, fold=1), tol=-1,
                                       max_iter=3)["phi"])
    o = R.si_opts(tol=-1, max_iter=3, precision=R.ROM_PREC_FP64 if prec == "fp64" else R.ROM_PREC_FP32)
    for _ in range(2):
        phis, stats, _ = R.solve_batch(hs, o)
        assert stats[0].lanes == 1
        for phi, ref in zip(phis, refs):
            parity.check(phi, ref, 1e-11 if prec == "fp64" else 2e-3)


# Single sweeps: rom_sweep and rom_sweep_noalloc on the row scan agree bit for bit, also for a source that starts
# on an odd element, replayed from a graph, and on either side of the plan size (16 MiB) up to which the row
# scan is taken (512 x 512 in FP32: 40 ordinates below it, 44 beyond).
@pytest.mark.parametrize("nx,ny,n,prec", [(1, 1, 1, "fp32"), (37, 5, 3, "fp64"), (130, 33, 50, "fp32"), (301, 20, 17, "fp64"),
                                          (64, 64, 300, "fp32"), (512, 512, 34, "fp32"), (512, 512, 44, "fp32")])
def test_single_sweeps(R, orc, nx, ny, n, prec):
    import ctypes as C
    import torch
    rng = np.random.default_rng([nx, ny, n])
    st, ss, q = problem(rng, nx, ny, "bands")
    infl = {"left": rng.uniform(0, 1, ny), "top": rng.uniform(0, 1, nx)}
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=1)
    h = R.Handle(nx, ny, st, ss, q, inflow=infl)
    h.set_ordinates(d, w)
    fp64 = prec == "fp64"
    o = R.si_opts(precision=R.ROM_PREC_FP64 if fp64 else R.ROM_PREC_FP32)
    dt = torch.float64 if fp64 else torch.float32
    cells = nx * ny
    src = torch.zeros(cells + 1, dtype=dt, device="cuda")[1:]
    phi = torch.zeros(cells, dtype=dt, device="cuda")

    def call():
        rc = R.lib().rom_sweep_noalloc(h.h, C.c_void_p(src.data_ptr()), C.c_void_p(phi.data_ptr()), o.precision,
                                       C.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == R.ROM_OK

    S = rng.uniform(0, 1, cells)
    src.copy_(torch.tensor(S, dtype=dt))
    call()
    got = phi.double().cpu().numpy()
    assert np.array_equal(got, h.sweep(S, o))
    p = orc.Problem(nx, ny, st, ss, q, inflow=infl)
    parity.check(got, orc.scalar_flux(w, orc.sweep(p, d, S)), 1e-11 if fp64 else 1e-5)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for _ in range(3):
        S = rng.uniform(0, 1, cells)
        src.copy_(torch.tensor(S, dtype=dt))
        phi.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(phi.double().cpu().numpy(), h.sweep(S, o))


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,n", [(1, 3, 1), (7, 11, 60), (61, 67, 66), (64, 33, 500), (31, 9, 2100)])
def test_combine_of_planes(R, orc, nx, ny, n, prec):
    """Cell counts that end inside a 16-byte load and inside a block of the combine, 4 to 64 planes and more (four
    and eight wavefronts, more planes than are loaded at once), one system and three that stop apart."""
    rng = np.random.default_rng([nx, ny, n])
    st, ss, q = problem(rng, nx, ny, "uniform")
    fp64 = prec == "fp64"
    hs, refs, iters = [], [], []
    for k in range(3):
        h = R.Handle(nx, ny, st, ss * (0.2 + 0.4 * k), q)
        d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, max(1, n - k), seed=k)
        h.set_ordinates(d, w)
        hs.append(h)
        ref = orc.source_iterate(orc.Problem(nx, ny, st, ss * (0.2 + 0.4 * k), q), d, w, None, tol=1e-4, max_iter=50)
        refs.append(ref["phi"])
        iters.append(ref["iters"])
    o = R.si_opts(tol=1e-4, max_iter=50, precision=R.ROM_PREC_FP64 if fp64 else R.ROM_PREC_FP32)
    phi, s, _ = hs[1].source_iterate(o)
    assert s.lanes == 1 and s.iters == iters[1]
    parity.check(phi, refs[1], 1e-11 if fp64 else 1e-5)
    phis, stats, _ = R.solve_batch(hs, o)
    assert [x.iters for x in stats] == iters
    for p, ref in zip(phis, refs):
        parity.check(p, ref, 1e-11 if fp64 else 1e-5)


@pytest.mark.parametrize("kernel", ["iso", "linear", "hg"])
@pytest.mark.parametrize("scheme", ["step", "dd"])
@pytest.mark.parametrize("nx,n", [(40, 13), (64, 64), (130, 29), (300, 8)])
def test_sigma_t_beyond_fp32(R, orc, monkeypatch, nx, n, scheme, kernel):
    """A black cell whose sigma_t has no FP32 value lets nothing through; the others keep their flux."""
    if kernel == "hg" and scheme == "dd":
        pytest.skip("dense kernels run the step scheme here")
    ny = 21
    st = np.ones(nx * ny)
    st[5 * nx + nx // 2] = 1e39
    ss, q = np.full(nx * ny, 0.5), np.ones(nx * ny)
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=1)
    W = None if kernel == "iso" else orc.build_W(d, w, orc.SCAT_LINEAR if kernel == "linear" else orc.SCAT_HG, 0.7, fold=1)
    ref = orc.source_iterate(orc.Problem(nx, ny, st, ss, q), d, w, W, tol=-1, max_iter=4,
                             scheme=orc.SCHEME_DD if scheme == "dd" else orc.SCHEME_STEP)["phi"]
    o = R.si_opts(tol=-1, max_iter=4, scheme=R.ROM_SCHEME_DD if scheme == "dd" else R.ROM_SCHEME_STEP)
    forms = 2 if nx <= (64 if kernel == "hg" else 128) else 1
    for k in range(forms + (2 if kernel == "iso" and scheme == "step" else 0)):
        monkeypatch.setenv("ROM_SWEEP_SCAN", str(k + 1))
        h = R.Handle(nx, ny, st, ss, q)
        h.set_ordinates(d, w)
        if kernel != "iso":
            h.set_scattering(R.ROM_SCAT_LINEAR if kernel == "linear" else R.ROM_SCAT_HG, 0.7)
        phi, s, _ = h.source_iterate(o)
        assert s.lanes == 1
        parity.check(phi, ref, 2e-3 if kernel == "hg" else 1e-5)


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("nx,n", [(130, 29), (248, 64), (200, 8)])
def test_a_neighbour_without_fp32_values(R, orc, monkeypatch, nx, n, k):
    """Two lane groups of 32 share a wavefront: beside a batch member whose source is infinite in FP32, one
    whose rows end before the lanes do keeps its flux, bit for bit."""
    import ctypes as C
    monkeypatch.setenv("ROM_SWEEP_SCAN", str(k))
    ny = 9
    st = np.ones(nx * ny)
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=1)
    got = []
    for bad in (1.0, 1e39):
        hs = []
        for q in (1.0, bad):
            h = R.Handle(nx, ny, st, 0.5 * st, q * st)
            h.set_ordinates(d, w)
            hs.append(h)
        outs = [np.zeros(nx * ny) for _ in hs]
        stats = (R.rom_si_stats * 2)()
        o = R.si_opts(tol=1e-5, max_iter=30)
        rc = R.lib().rom_solve_batch((C.c_void_p * 2)(*[h.h for h in hs]), 2, C.byref(o),
                                     (C.c_void_p * 2)(*[x.ctypes.data for x in outs]), stats)
        assert rc == R.ROM_OK or bad > 1.0
        assert stats[0].lanes == 1 and stats[0].status == R.ROM_OK
        got.append(outs[0])
    assert np.array_equal(*got)
    ref = orc.source_iterate(orc.Problem(nx, ny, st, 0.5 * st, st), d, w, None, tol=-1, max_iter=stats[0].iters)["phi"]
    parity.check(got[1], ref, 1e-5)


@pytest.mark.parametrize("scheme", ["step", "dd"])
@pytest.mark.parametrize("nx,ny", [(16, 1000), (64, 1024), (130, 1000), (500, 700)])
def test_long_columns_of_one_medium(R, orc, monkeypatch, nx, ny, scheme):
    """One ordinate along the columns: the flux decays by the same b r in every row, whose rounding error must not
    add up (1e-5 after 1000 rows is 1e-8 a row, a sixth of half an ulp, kept up all the way; the two roundings of
    a row are as good as random while the flux decays, 1.1e-6 after 1000 rows, 5.6e-6 at five sigma).  The bar of
    the other FP32 comparisons, here for every cell as well; twice that for diamond difference, whose face
    values 2 psi - psi_in double a row's rounding."""
    st, z = np.full(nx * ny, 0.1), np.zeros(nx * ny)
    infl = {f: np.ones(ny if f in FACES[:2] else nx) for f in FACES}
    dd = scheme == "dd"
    p = orc.Problem(nx, ny, st, z, z, inflow=infl)
    o = R.si_opts(tol=-1, max_iter=1, scheme=R.ROM_SCHEME_DD if dd else R.ROM_SCHEME_STEP)
    for s in (0.777, -0.777, 0.9, -0.9):
        d, w = np.array([[0.0, s, np.sqrt(1.0 - s * s)]]), np.ones(1)
        ref = orc.scalar_flux(w, orc.sweep(p, d, z, scheme=orc.SCHEME_DD if dd else orc.SCHEME_STEP))
        for k in range((2 if nx <= 128 else 1) + (0 if dd else 2)):
            monkeypatch.setenv("ROM_SWEEP_SCAN", str(k + 1))
            h = R.Handle(nx, ny, st, z, z, inflow=infl)
            h.set_ordinates(d, w)
            phi, stats, _ = h.source_iterate(o)
            assert stats.lanes == 1
            bar = 2e-5 if dd else 1e-5
            parity.check(phi, ref, bar, cell_tol=bar, what=f"{s} form {k + 1}")


@pytest.mark.parametrize("nx,ny", [(16, 1000), (64, 1024), (130, 600), (300, 700)])
def test_tall_grids(R, orc, monkeypatch, nx, ny):
    """The forms on grids far taller than a batch of rows, at the bars of the other FP32 solves."""
    st = np.full(nx * ny, 1.0)
    ss, q = 0.5 * st, np.zeros(nx * ny)
    q.reshape(ny, nx)[ny // 3:ny // 2, nx // 4:] = 1.0
    d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, 2, 4, seed=2)
    ref = orc.source_iterate(orc.Problem(nx, ny, st, ss, q), d, w, None, tol=-1, max_iter=5)["phi"]
    for k in range(shapes(False, nx)):
        monkeypatch.setenv("ROM_SWEEP_SCAN", str(k + 1))
        h = R.Handle(nx, ny, st, ss, q)
        h.set_ordinates(d, w)
        phi, stats, _ = h.source_iterate(R.si_opts(tol=-1, max_iter=5))
        assert stats.lanes == 1
        parity.check(phi, ref, 1e-5)


@pytest.mark.parametrize("shape", [{"diag_rows": 16}, {"diag_rows": 64}, {"diag_k": 2}, {"diag_rows": 16, "diag_k": 1}])
def test_a_named_row_lane_shape_is_kept(R, orc, shape):
    """Rows or ordinates per lane, named with the kernel left open, restrict the choice as before: among the row-lane
    kernel's shapes those, or the strip kernel's, never the row scan."""
    f = problem(np.random.default_rng(1), 48, 40, "uniform")
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, 24, seed=1)
    h = R.Handle(48, 40, *f)
    h.set_ordinates(d, w)
    phi, s, _ = h.source_iterate(R.si_opts(tol=-1, max_iter=4, **shape))
    assert s.lanes != 1
    if s.sweep == R.ROM_SWEEP_DIAG:
        assert s.tile_y == shape.get("diag_rows", s.tile_y) and s.tile_x == shape.get("diag_k", s.tile_x)
    parity.check(phi, orc.source_iterate(orc.Problem(48, 40, *f), d, w, None, tol=-1, max_iter=4)["phi"], 1e-5)


@pytest.mark.parametrize("kernel,dd,top", [("iso", True, 1e37), ("linear", True, 1e37), ("linear", False, 2e37)])
@pytest.mark.parametrize("where", ["q", "inflow", "angular"])
def test_sources_near_the_end_of_fp32(R, orc, kernel, dd, top, where):
    """The weighted fluxes of the strip kernel stay finite where 2 |s| / dy times the flux itself would not."""
    nx, ny, n = 40, 24, 29
    one, z = np.ones(nx * ny), np.zeros(nx * ny)
    d, w = R.generate_ordinates(R.ROM_ORD_IID_SPHERE, n, seed=1)
    q = top * one if where == "q" else z
    infl = {"left": np.full(ny, top)} if where == "inflow" else None
    W = None if kernel == "iso" else orc.build_W(d, w, orc.SCAT_LINEAR, 0.8, fold=1)
    h = R.Handle(nx, ny, one, 0.5 * one, q, inflow=infl)
    h.set_ordinates(d, w)
    ang = None
    if where == "angular":
        h.set_inflow_angular(0, np.full((n, ny), top))
        ang = {"left": np.full((n, ny), top)}
    if kernel != "iso":
        h.set_scattering(R.ROM_SCAT_LINEAR, 0.8)
    phi, s, _ = h.source_iterate(R.si_opts(tol=-1, max_iter=6, scheme=R.ROM_SCHEME_DD if dd else R.ROM_SCHEME_STEP))
    ref = orc.source_iterate(orc.Problem(nx, ny, one, 0.5 * one, q, inflow=infl, inflow_angular=ang), d, w, W, tol=-1, max_iter=6,
                             scheme=orc.SCHEME_DD if dd else orc.SCHEME_STEP)["phi"]
    parity.check(phi, ref, 1e-5)


@pytest.mark.parametrize("kernel,prec", [("iso", "fp64"), ("linear", "fp32")])
def test_partial_planes_that_do_not_fit(R, orc, kernel, prec):
    """Where the allocator has no room for the row scan's partial planes, the solve runs on another kernel, which needs
    a part of them, and a later solve with room takes the row scan."""
    import torch
    nx, ny, n = 200, 180, 256
    f = problem(np.random.default_rng(2), nx, ny, "uniform")
    d, w = R.generate_ordinates(R.ROM_ORD_STRATIFIED, 8, 8, seed=1)
    cells, planes = nx * ny, 64 * (4 if kernel == "linear" else 1)
    limit = cells * planes * (8 if prec == "fp64" else 4) // 2   # half of the planes (of 4 ordinates)
    R._default_allocator()
    give, back = R._allocator
    refused = []

    def alloc(nbytes, ctx):
        if nbytes > limit:
            refused.append(nbytes)
            return None
        return give(nbytes, ctx)

    def free(p, ctx):
        back(p, ctx)

    cbs = (R._ALLOC_FN(alloc), R._FREE_FN(free))
    W = None if kernel == "iso" else orc.build_W(d, w, orc.SCAT_LINEAR, 0.6, fold=1)
    ref = orc.source_iterate(orc.Problem(nx, ny, *f), d, w, W, tol=-1, max_iter=3)["phi"]
    o = R.si_opts(tol=-1, max_iter=3, precision=R.ROM_PREC_FP64 if prec == "fp64" else R.ROM_PREC_FP32)

    def solve():
        h = R.Handle(nx, ny, *f)
        h.set_ordinates(d, w)
        if kernel != "iso":
            h.set_scattering(R.ROM_SCAT_LINEAR, 0.6)
        phi, s, _ = h.source_iterate(o)
        h.close()
        return phi, s

    bar = 1e-11 if prec == "fp64" else 1e-5
    assert R.lib().rom_set_allocator(cbs[0], cbs[1], None) == R.ROM_OK
    try:
        phi, s = solve()
    finally:
        R.use_torch_allocator()
    assert refused and s.lanes != 1
    parity.check(phi, ref, bar)
    torch.cuda.synchronize()
    phi, s = solve()
    assert s.lanes == 1
    parity.check(phi, ref, bar)


def test_reported_shapes(R, monkeypatch):
    """Each problem of a batch reports the shape of its own width: lanes per row in tile_y, ordinates per group in tile_x."""
    monkeypatch.setenv("ROM_SWEEP_SCAN", "2")   # the first width beyond 128: the form for full GPUs
    hs = []
    for nx in (700, 40, 100, 200, 350, 512):
        st = np.ones(nx * 8)
        h = R.Handle(nx, 8, st, 0.5 * st, st)
        h.set_ordinates(*R.generate_ordinates(R.ROM_ORD_IID_SPHERE, 12, seed=1))
        hs.append(h)
    o = R.si_opts(tol=-1, max_iter=2)
    stats = R.solve_batch(hs, o)[1]
    assert all(s.lanes == 1 and s.band == 8 for s in stats)
    assert [(s.tile_y, s.tile_x) for s in stats] == [(64, 2), (16, 4), (16, 2), (32, 2), (64, 2), (64, 2)]
    s = hs[3].source_iterate(o)[1]
    assert (s.lanes, s.band, s.tile_y, s.tile_x) == (1, 8, 32, 2)
