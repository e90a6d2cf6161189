"""GPU: the block update of the shifted systems and the stencil variants that each launch takes by
its size.

Block lengths: a memory limit picks 20, 10, 5, 2 or 1 iterations per block; the arithmetic is that
of an update in every iteration, so q(x) is equal bit for bit, also where reliable updates cut
blocks short.  Stencils: every plane shape of the any-lattice kernel (several planes per block
with a ragged last block, rows of one plane with a shorter last tile, no LDS) against the oracle with
the stencil parity bounds (FP64 1e-13, FP32 2e-6 of the largest entry); results equal bit for bit
whatever number of right-hand sides a launch carries.  Links whose third row is further than
rounding from the product of the other two keep it.
"""
import numpy as np
import pytest

import smpq_inputs as si
from oracle.dirac import apply_dw
from oracle.lattice import Lattice

pytestmark = pytest.mark.gpu

import paper_1901_02211_amd as smpq  # noqa: E402

KAPPA = 0.21


def _slot_bytes(prec, ns, k, volume):
    """Device bytes per right-hand side: k residuals, tmp, the directions (one more with k > 1) and
    y; mixed: those in FP32, y, x0 and, unless the ring holds them, two reliable-update vectors in
    FP64."""
    v64 = 192 * (-(-volume // 256) * 256)
    n = k + 1 + ns + (k > 1)
    return (n + 1) * v64 if prec == smpq.SMPQ_FP64 else n * v64 // 2 + (2 if k >= 5 else 4) * v64


@pytest.mark.parametrize("poles", [3, 14, 32])   # registers for up to 8, 14 and 32 directions
@pytest.mark.parametrize("prec,reliable", [(smpq.SMPQ_FP64, 0), (smpq.SMPQ_MIXED_FP32, 0),
                                           (smpq.SMPQ_MIXED_FP32, 10), (smpq.SMPQ_MIXED_FP32, 50)])
def test_block_lengths_equal(prec, reliable, poles):
    dims = (6, 4, 4, 6)
    print(f"block lengths, precision {prec}, reliable {reliable}, {poles} poles", flush=True)
    c = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c, si.near_identity_su3(dims, 0.3, 7))
    smpq.smpq_set_zolotarev(c, poles, 0.13, 2.7)
    smpq.smpq_set_scheme(c, (2, 2, 2, 2), 0)
    smpq.smpq_set_solver(c, prec, 1e-12, 5000, reliable)
    want = smpq.smpq_compute_qx_classes(c, [5])
    for k in (50, 20, 10, 5, 2, 1):
        smpq.smpq_set_memory_limit(c, 12 * _slot_bytes(prec, poles, k, 576))
        got = smpq.smpq_compute_qx_classes(c, [5])
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), k
        assert got[2]["total_iters"] == want[2]["total_iters"]


@pytest.mark.parametrize("dims", [(3, 3, 3, 3), (5, 3, 4, 7), (6, 10, 6, 2), (12, 12, 2, 3), (17, 17, 3, 2),
                                  (24, 12, 2, 3), (100, 4, 3, 2), (128, 3, 2, 2), (130, 4, 2, 2), (1, 5, 3, 4),
                                  (64, 8, 2, 2)])
def test_stencil_on_any_plane(dims):
    print(f"stencil on {dims}", flush=True)
    lat = Lattice(dims)
    U = si.near_identity_su3(dims, 0.5, 3)
    psi = si.random_spinors(dims, 5, 4)
    c = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c, U)
    for dag in (False, True):
        ref = np.stack([apply_dw(U, lat, KAPPA, p, dagger=dag) for p in psi])
        scale = np.abs(ref).max()
        default = [smpq.smpq_apply_dw(c, psi, dagger=dag, precision=p) for p in (0, 1)]
        one = smpq.smpq_apply_dw(c, psi[4:], dagger=dag, precision=1)
        assert np.array_equal(one[0], default[1][4])
        assert np.abs(default[0] - ref).max() <= 1e-13 * scale
        assert np.abs(default[1] - ref).max() <= 2e-6 * scale
    for nr, lgr in ((2, 0), (4, 1), (8, 2)):     # the last right-hand side without a partner
        c2 = smpq.smpq_create(dims, 0)
        smpq.smpq_load_gauge(c2, U)
        smpq.smpq_set_tuning(c2, 0, nr, lgr)
        for p in (0, 1):
            out = smpq.smpq_apply_dw(c2, psi, dagger=True, precision=p)
            assert np.array_equal(out, default[p]), (nr, p)


def test_default_variants_do_not_change_results():
    """16 x 16 planes: few right-hand sides and many take different kernels by default (2048 tiles x
    sides on); the solver's q(x) and D_W are equal bit for bit."""
    dims = (16, 16, 8, 8)
    print(f"default variants on {dims}", flush=True)
    c = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c, si.near_identity_su3(dims, 0.3, 5))
    psi = si.random_spinors(dims, 66, 6)
    for dag in (False, True):
        many = smpq.smpq_apply_dw(c, psi, dagger=dag, precision=1)
        assert np.array_equal(smpq.smpq_apply_dw(c, psi[:1], dagger=dag, precision=1), many[:1])
    smpq.smpq_set_zolotarev(c, 14, 0.13, 2.7)
    smpq.smpq_set_scheme(c, (2, 2, 2, 2), 0)
    smpq.smpq_set_solver(c, smpq.SMPQ_MIXED_FP32, 1e-12, 5000, 50)
    six = smpq.smpq_compute_qx_classes(c, [0, 3, 5, 9, 11, 14])[0]
    c1 = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c1, si.near_identity_su3(dims, 0.3, 5))
    smpq.smpq_set_zolotarev(c1, 14, 0.13, 2.7)
    smpq.smpq_set_scheme(c1, (2, 2, 2, 2), 0)
    smpq.smpq_set_solver(c1, smpq.SMPQ_MIXED_FP32, 1e-12, 5000, 50)
    one = smpq.smpq_compute_qx_classes(c1, [9])[0]
    on = one != 0
    assert on.sum() == np.prod(dims) // 16 and np.array_equal(one[on], six[on])


@pytest.mark.parametrize("dims", [(8, 8, 4, 4), (6, 4, 4, 6)])
def test_inexact_third_row_is_kept(dims):
    """Links within the accepted 1e-10 of SU(3) whose third rows are 1e-11 off the product of the
    other two: FP64 results follow the links as loaded."""
    print(f"inexact third rows on {dims}", flush=True)
    lat = Lattice(dims)
    U = si.near_identity_su3(dims, 0.5, 9)
    rng = np.random.default_rng(10)
    U[:, :, 2] += 1e-11 * rng.standard_normal(U[:, :, 2].shape)
    psi = si.random_spinors(dims, 3, 11)
    c = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c, U)
    for tune in (None, (2 if dims[0] == 8 else 0, 4, 1, 1, 1 if dims[0] == 8 else 0, 2)):
        if tune:
            smpq.smpq_set_tuning(c, *tune)
        for dag in (False, True):
            ref = np.stack([apply_dw(U, lat, KAPPA, p, dagger=dag) for p in psi])
            out = smpq.smpq_apply_dw(c, psi, dagger=dag)
            assert np.abs(out - ref).max() <= 1e-13 * np.abs(ref).max(), (tune, dag)


@pytest.mark.parametrize("inexact", [False, True])    # FP64 links read as two rows, or in full
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (3, 3, 3, 3), (8, 8, 2, 2), (5, 3, 4, 7), (16, 16, 2, 1), (17, 17, 1, 1)])
def test_small_lattices_equal_separate_kernels(dims, inexact):
    """Up to 512 threads of stencil tiles (one or two tiles of 256, 64-thread tiles, several planes or
    ragged rows per tile) a right-hand side is solved by one workgroup; timed solves keep the separate
    kernels, with results equal bit for bit: D_ov and point densities, in blocks cut short by
    reliable updates and by convergence."""
    print(f"small lattice {dims}, inexact links {inexact}", flush=True)
    V = int(np.prod(dims))
    U = si.near_identity_su3(dims, 0.3, 7)
    if inexact:
        U[:, :, 2] += 1e-11 * np.random.default_rng(8).standard_normal(U[:, :, 2].shape)
    psi = si.random_spinors(dims, 2, 4)
    for prec, reliable in ((0, 0), (1, 30)):
        out = []
        for timing in (False, True):
            c = smpq.smpq_create(dims, 0)
            smpq.smpq_load_gauge(c, U)
            smpq.smpq_set_zolotarev(c, 14, 0.12, 2.75)
            smpq.smpq_set_solver(c, prec, 1e-12, 5000, reliable)
            smpq.smpq_set_timing(c, timing)
            q, st = smpq.smpq_compute_qx_points(c, [0, V // 2, V - 1])
            out.append((q, smpq.smpq_apply_dov(c, psi), st["total_iters"], st["shift_updates"]))
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1]), prec
        assert out[0][2:] == out[1][2:]
    # a solve that breaks off at max_iter leaves the context usable
    smpq.smpq_set_timing(c, False)
    smpq.smpq_set_solver(c, 0, 1e-12, 10, 0)
    with pytest.raises(smpq.SmpqError) as e:
        smpq.smpq_apply_dov(c, psi)
    assert e.value.status == -5
    smpq.smpq_set_solver(c, 1, 1e-12, 5000, 30)
    assert np.array_equal(smpq.smpq_apply_dov(c, psi), out[0][1])


@pytest.mark.parametrize("prec", [smpq.SMPQ_FP64, smpq.SMPQ_MIXED_FP32])
def test_prepared_workspace_serves_smaller_calls(prec):
    """A call with fewer sources between two whole maps changes neither their values nor their batches."""
    dims = (4, 4, 4, 6)
    print(f"small call between maps, precision {prec}", flush=True)
    c = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c, si.near_identity_su3(dims, 0.3, 7))
    smpq.smpq_set_zolotarev(c, 14, 0.13, 2.7)
    smpq.smpq_set_scheme(c, (2, 2, 2, 2), 0)
    smpq.smpq_set_solver(c, prec, 1e-12, 5000, 50)
    for limit in (0, 96 * _slot_bytes(prec, 14, 10, 384)):
        smpq.smpq_set_memory_limit(c, limit)
        q, qi, Q, st = smpq.smpq_compute_qx(c)
        one = smpq.smpq_compute_qx_classes(c, [5])
        q2, qi2, Q2, st2 = smpq.smpq_compute_qx(c)
        assert np.array_equal(q, q2) and np.array_equal(qi, qi2) and st["n_batches"] == st2["n_batches"]
        mask = smpq.smpq_get_coloring(c) == 5
        assert np.array_equal(one[0][mask], q[mask])
