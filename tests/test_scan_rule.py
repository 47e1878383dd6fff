"""The rule that takes the row-scan sweep, asked about sizes on the host: the limits of its kernels and its lines."""
import ctypes as C

import numpy as np
import pytest

ISO, LINEAR, DENSE, SINGLE = 0, 1, 2, -1


@pytest.fixture(scope="module")
def R():
    from paper_2407_12527_amd import rom
    rom.lib()
    return rom


def choice(R, systems, prec="fp32", mode=ISO, dd=False):
    """(wavefronts, lanes per row, cells per lane), or None where the other kernels are left the choice.
    systems: (nx, ny, ordinates[, rows whose sigma_t differs from the row below])."""
    f = R.lib().rom_scan_rule
    a = np.array([s if len(s) == 4 else (*s, 0) for s in systems], dtype=np.int64)
    out = (C.c_int32 * 3)()
    got = f(C.c_void_p(a.ctypes.data), len(a), R.ROM_PREC_FP64 if prec == "fp64" else R.ROM_PREC_FP32,
            R.ROM_SCHEME_DD if dd else R.ROM_SCHEME_STEP, mode, out)
    return tuple(out) if got else None


def test_offsets_within_a_system_are_32_bit(R):
    # (cells * 4 planes + 33 rows of look-ahead) * bytes per value below 4 GiB
    for prec, esz in (("fp32", 4), ("fp64", 8)):
        most = (2**32 // esz - 1 - 33 * 512) // (4 * 512)   # rows of 512 cells
        assert choice(R, [(512, most, 4)], prec) is not None
        assert choice(R, [(512, most + 1, 4)], prec) is None


def test_partial_planes_fit_32_gib(R):
    # a plane per four ordinates and quadrant remainder: 64 + 4 of 512 x 512 cells in FP64 a system
    most = 2**35 // (512 * 512 * 68 * 8)
    assert choice(R, [(512, 512, 256)] * most, "fp64") is not None
    assert choice(R, [(512, 512, 256)] * (most + 1), "fp64") is None
    # four times that with the linear kernel's moments
    most = 2**35 // (512 * 512 * 68 * 8 * 4)
    assert choice(R, [(512, 512, 256)] * most, "fp64", LINEAR) is not None
    assert choice(R, [(512, 512, 256)] * (most + 1), "fp64", LINEAR) is None


def test_widths(R):
    assert choice(R, [(512, 64, 16)], mode=DENSE) == (4, 64, 8)
    for mode, dd in ((LINEAR, False), (LINEAR, True), (ISO, True), (DENSE, False)):
        assert choice(R, [(512, 200, 16)], mode=mode, dd=dd) is not None
        assert choice(R, [(513, 200, 16)], mode=mode, dd=dd) is None
    assert choice(R, [(64, 64, 16)], mode=DENSE, dd=True) is None
    assert choice(R, [(1024, 100, 16)]) is not None
    assert choice(R, [(1025, 100, 16)]) is None


# One system of the linear kernel: the row scan where it is the faster one (step times in the rule's comment).
@pytest.mark.parametrize("prec,nx,ny,n,taken", [
    ("fp32", 8, 8, 256, False), ("fp32", 16, 16, 512, False), ("fp32", 16, 16, 4096, False), ("fp32", 32, 32, 512, True),
    ("fp32", 32, 32, 1024, False), ("fp32", 32, 32, 4096, False), ("fp32", 64, 64, 1024, True), ("fp32", 64, 64, 2048, False),
    ("fp32", 64, 64, 4096, True), ("fp32", 100, 100, 2048, True), ("fp64", 8, 8, 256, True), ("fp64", 8, 8, 1024, False),
    ("fp64", 8, 8, 4096, False), ("fp64", 16, 16, 512, True), ("fp64", 16, 16, 2048, False), ("fp64", 32, 32, 2048, True)])
def test_linear_kernel_with_many_ordinates(R, prec, nx, ny, n, taken):
    assert (choice(R, [(nx, ny, n)], prec, LINEAR) is not None) == taken
    assert choice(R, [(nx, ny, n)], prec, ISO, dd=True) is not None


# Ensembles that fill the GPU in FP32, diamond difference and the linear kernel: the strip kernel where it is the faster one.
@pytest.mark.parametrize("mode,dd,nx,n,t,taken", [
    (LINEAR, False, 256, 128, 16, True), (LINEAR, False, 256, 128, 64, False), (LINEAR, False, 128, 128, 32, True),
    (LINEAR, False, 128, 128, 64, False), (LINEAR, False, 300, 128, 16, True), (LINEAR, False, 300, 128, 32, False),
    (LINEAR, True, 512, 128, 8, True), (LINEAR, True, 512, 128, 16, False), (LINEAR, False, 64, 128, 128, True),
    (LINEAR, False, 128, 32, 256, True), (ISO, True, 256, 128, 32, True), (ISO, True, 256, 128, 64, False),
    (ISO, True, 300, 128, 16, True), (ISO, True, 300, 128, 32, False), (ISO, True, 300, 32, 128, True),
    (ISO, True, 512, 128, 16, True), (ISO, True, 512, 512, 8, False), (ISO, True, 64, 128, 128, True)])
def test_ensembles_that_fill_the_gpu(R, mode, dd, nx, n, t, taken):
    assert (choice(R, [(nx, nx, n)] * t, "fp32", mode, dd) is not None) == taken
    assert choice(R, [(nx, nx, n)] * t, "fp64", mode, dd) is not None


# Hundreds of small samples with few ordinates: the measured choice (step times in the rule's comment).
@pytest.mark.parametrize("nx,n,t,taken", [
    (32, 16, 1024, False), (64, 64, 256, False), (64, 32, 512, False), (64, 32, 256, True), (64, 128, 128, True), (100, 8, 512, False),
    (100, 32, 256, True), (128, 48, 341, False), (128, 32, 256, True), (128, 128, 512, True), (200, 16, 512, True)])
def test_many_small_samples(R, nx, n, t, taken):
    assert (choice(R, [(nx, nx, n)] * t) is not None) == taken
    assert choice(R, [(nx, nx, n)] * t, "fp64") is not None


# Media that change from row to row: the row-lane kernel where it is the faster one (step times in the rule's comment).
@pytest.mark.parametrize("prec,nx,ny,changes,taken", [
    ("fp32", 8, 64, 63, False), ("fp32", 24, 200, 199, False), ("fp32", 64, 64, 63, False), ("fp32", 64, 300, 299, False),
    ("fp32", 28, 40, 39, False), ("fp32", 60, 20, 19, True), ("fp32", 32, 200, 40, True), ("fp32", 32, 200, 41, False),
    ("fp32", 300, 100, 25, True), ("fp32", 300, 100, 26, False), ("fp64", 64, 64, 63, True), ("fp64", 32, 32, 31, True),
    ("fp64", 8, 64, 63, False), ("fp64", 24, 200, 199, False), ("fp64", 65, 64, 63, False), ("fp64", 65, 64, 16, True)])
def test_media_that_change_from_row_to_row(R, prec, nx, ny, changes, taken):
    assert (choice(R, [(nx, ny, 64, changes)], prec) is not None) == taken
    assert (choice(R, [(nx, ny, 64, changes)] * 3, prec) is not None) == taken
    assert choice(R, [(nx, ny, 64, 0)], prec) is not None
    assert choice(R, [(nx, ny, 64, changes)], prec, dd=True) is not None   # the strip kernel is slower there in any medium
    if nx <= 64:
        assert choice(R, [(nx, ny, 64, changes)], prec, SINGLE) is not None   # and it is the other one for single sweeps


# The samples that an ensemble solves at once fit its 24 GiB with the row scan's partial planes, whose number follows
# from the shape that the rule takes for as many of them.
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("mode", [ISO, LINEAR])
@pytest.mark.parametrize("nx,n,t", [(64, 64, 16), (512, 256, 1000), (512, 128, 64), (256, 128, 1024), (500, 1024, 300), (100, 16, 5000)])
def test_ensemble_batches_fit_their_budget(R, nx, n, t, mode, prec):
    per_sample = nx * nx * 66
    f = R.lib().rom_ensemble_batch_size
    s = np.array([nx, nx, n, 0], dtype=np.int64)
    held = C.c_int64()
    B = f(C.c_void_p(s.ctypes.data), t, C.c_int64(per_sample), R.ROM_PREC_FP64 if prec == "fp64" else R.ROM_PREC_FP32, mode, C.byref(held))
    assert 1 <= B <= min(t, 1024)
    assert held.value <= 24 << 30
    took = choice(R, [(nx, nx, n)] * B, prec, mode)
    if took is not None and took[0] <= 4:   # a plane per workgroup: its wavefronts' ordinates
        planes = n // (took[0] * 64 // took[1])
        assert B * (per_sample + planes * nx * nx * (4 if mode == LINEAR else 1) * (8 if prec == "fp64" else 4)) <= 24 << 30
    if t * per_sample < 1 << 30:   # small ones are not split
        assert B == min(t, 1024)


# Batches of uneven grids on the lanes of the widest: not where a narrow one is so tall that its rows cost more than
# the row-lane kernel's way through it.
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("grids,taken", [([(480, 34), (32, 292)], False), ([(480, 300), (32, 292)], True),
                                         ([(224, 386), (102, 113)], True), ([(480, 34), (300, 292)], True), ([(32, 292)], True)])
def test_batches_of_uneven_grids(R, prec, grids, taken):
    assert (choice(R, [(nx, ny, 64) for nx, ny in grids], prec) is not None) == taken
