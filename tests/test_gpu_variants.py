"""GPU: explicitly chosen stencil variants against the default ones."""
import numpy as np
import pytest

import smpq_inputs as si

pytestmark = pytest.mark.gpu

import paper_1901_02211_amd as smpq  # noqa: E402


def _ctx(dims, prec, tune=None):
    c = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c, si.near_identity_su3(dims, 0.3, 7))
    smpq.smpq_set_zolotarev(c, 14, 0.15, 2.75)
    smpq.smpq_set_solver(c, prec, 1e-12, 5000, 50)
    if tune:
        smpq.smpq_set_tuning(c, *tune)
    return c


@pytest.mark.parametrize("band", [0, -1, 2, 3])
@pytest.mark.parametrize("dims", [(12, 12, 4, 3), (20, 18, 4, 2), (6, 10, 4, 2), (17, 8, 4, 2), (130, 4, 4, 1)])
def test_any_lattice_variant_ignores_the_band(dims, band):
    """One plane per block, rows of one, several planes, no tile: D_W and D_ov equal those of the default
    variant (which has no band) bit for bit."""
    print(f"kind 0 on {dims}, band {band}", flush=True)
    psi = si.random_spinors(dims, 3, 4)
    for prec in (0, 1):
        c, d = _ctx(dims, prec, (0, 4, 1, band)), _ctx(dims, prec)
        for dag in (False, True):
            assert np.array_equal(smpq.smpq_apply_dw(c, psi, dagger=dag, precision=prec),
                                  smpq.smpq_apply_dw(d, psi, dagger=dag, precision=prec))
        assert np.array_equal(smpq.smpq_apply_dov(c, psi), smpq.smpq_apply_dov(d, psi))


@pytest.mark.parametrize("check", [False, True])
@pytest.mark.parametrize("reliable", [50, 20])
@pytest.mark.parametrize("prec", [smpq.SMPQ_MIXED_FP16VEC, smpq.SMPQ_MIXED_BF16VEC])
def test_rounded_vectors_do_not_depend_on_the_block(prec, reliable, check):
    """The block update repeats the rounding of the base direction that the stencil read: q(x) of blocks of 50
    to 1 iterations (by the memory limit), also on a lattice whose solves would fit one workgroup, is equal
    bit for bit."""
    for dims in ((4, 4, 4, 4), (6, 4, 4, 6)):
        print(f"rounded vectors in blocks, precision {prec}, reliable {reliable}, check {check}, {dims}", flush=True)
        c = _ctx(dims, prec)
        smpq.smpq_set_scheme(c, (2, 2, 2, 2), 0)
        smpq.smpq_set_solver(c, prec, 1e-8, 300, reliable)
        if check:
            smpq.smpq_set_shift_check(c, True, 0.0)
        v64 = 192 * (-(-int(np.prod(dims)) // 256) * 256)
        extra = 16 * v64 if check else 0
        want = None
        for k in (50, 20, 10, 5, 2, 1):
            n = k + 1 + 14 + (k > 1)
            slot = n * v64 // 2 + (2 if k >= 5 and not check else 4) * v64 + extra
            smpq.smpq_set_memory_limit(c, 12 * slot)
            try:
                got = smpq.smpq_compute_qx_classes(c, [5])
                got = (got[0].tobytes(), got[2]["total_iters"], got[2]["max_true_resid"])
            except smpq.SmpqError as e:      # BF16's rounding may break the iteration off: alike for every length
                got = (e.status,)
            want = want or got
            assert got == want, k


@pytest.mark.parametrize("dims", [(12, 12, 4, 3), (6, 10, 4, 2), (130, 4, 4, 1), (8, 8, 4, 4), (16, 16, 4, 4)])
def test_reported_and_autotuned_variants_give_the_default_results(dims):
    """The variant that a context reports, and the one that the autotuner picks, set explicitly: mixed D_ov and
    FP32 D_W equal to those of the default variants bit for bit."""
    print(f"reported and autotuned variants on {dims}", flush=True)
    psi = si.random_spinors(dims, 3, 4)
    d = _ctx(dims, 1)
    reported = smpq.smpq_get_tuning(d)
    for pick in (False, True):
        c = _ctx(dims, 1)
        if pick:
            t = smpq.smpq_autotune(c, 12)
            assert t["f32_kind"] in ((0,) if dims[0] in (12, 6, 130) else (0, 1, 2, 3, 4)), t
        else:
            smpq.smpq_set_tuning(c, **reported)
        assert np.array_equal(smpq.smpq_apply_dw(c, psi, precision=1), smpq.smpq_apply_dw(d, psi, precision=1))
        assert np.array_equal(smpq.smpq_apply_dov(c, psi), smpq.smpq_apply_dov(d, psi))


@pytest.mark.parametrize("dims", [(12, 12, 4, 3), (6, 10, 4, 2), (130, 4, 2, 2), (16, 16, 4, 2), (24, 24, 2, 2), (8, 8, 4, 4)])
def test_interleaved_sides_equal_single_ones(dims):
    """Default FP64 launches take two or four right-hand sides of a tile in a row, the last group maybe in part:
    D_W and D_ov of 1 to 7 sides equal those of each side alone bit for bit."""
    print(f"interleaved right-hand sides on {dims}", flush=True)
    psi = si.random_spinors(dims, 7, 4)
    c = _ctx(dims, 0)
    one = [np.concatenate([f(psi[i:i + 1]) for i in range(7)]) for f in
           (lambda p: smpq.smpq_apply_dw(c, p), lambda p: smpq.smpq_apply_dov(c, p))]
    for n in (2, 3, 4, 5, 7):
        assert np.array_equal(smpq.smpq_apply_dw(c, psi[:n]), one[0][:n])
        assert np.array_equal(smpq.smpq_apply_dov(c, psi[:n]), one[1][:n])
