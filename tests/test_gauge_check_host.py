"""The SU(3) check of smpq_load_gauge on a host context: what it refuses, it refuses at any size of the
entries.  (Links that pass end in "host-only context".)"""
import numpy as np
import pytest

import paper_1901_02211_amd as smpq
import smpq_inputs as si

DIMS = (2, 2, 2, 2)
ENUMERIC, EDEVICE = -7, -4


def _status(U):
    with pytest.raises(smpq.SmpqError) as e:
        smpq.smpq_load_gauge(smpq.smpq_create(DIMS, -1), U)
    return e.value.status


def test_fields_in_su3_pass():
    assert _status(si.near_identity_su3(DIMS, 0.3, 1)) == EDEVICE


@pytest.mark.parametrize("value", [2.0, 1e150, 1e155, 1e160, 1e200, 1e308])
@pytest.mark.parametrize("phase", [1.0, 1j, 1 + 1j, 1 - 1j, -1 + 0.5j])
@pytest.mark.parametrize("where", ["all", "row", "column", "entry", "diagonal"])
def test_large_entries_are_refused(value, phase, where):
    U = si.near_identity_su3(DIMS, 0.3, 1)
    z = value * phase
    if where == "all":
        U[3, 2] = z
    elif where == "row":
        U[3, 2, 1] = z
    elif where == "column":
        U[3, 2, :, 2] = z
    elif where == "entry":
        U[3, 2, 0, 1] = z
    else:
        U[3, 2] = np.diag([z, z, z])
    assert _status(U) == ENUMERIC


@pytest.mark.parametrize("off,ok", [(0.5e-10, True), (2e-10, False)])
def test_threshold(off, ok):
    U = si.near_identity_su3(DIMS, 0.0, 1)
    U[3, 2, 0, 1] += off          # |U^dag U - 1| = off, det U = 1
    assert _status(U) == (EDEVICE if ok else ENUMERIC)
