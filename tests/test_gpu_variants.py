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
