"""GPU: the workspace of a context when memory runs short or its options change."""
import ctypes
import re

import numpy as np
import pytest

import smpq_inputs as si

pytestmark = pytest.mark.gpu

import paper_1901_02211_amd as smpq  # noqa: E402

DIMS = (8, 8, 8, 8)


def _ctx(prec=0, dims=DIMS):
    c = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c, si.near_identity_su3(dims, 0.3, 7))
    smpq.smpq_set_zolotarev(c, 14, 0.15, 2.75)
    smpq.smpq_set_scheme(c, (2, 2, 2, 2), 0)
    smpq.smpq_set_solver(c, prec, 1e-12, 5000, 50)
    return c


@pytest.mark.parametrize("prec,limit", [(0, 4 << 40),      # the first vector does not fit the device
                                        (0, 380 << 30),    # the ring does (200 GB), the directions do not
                                        (1, 4 << 40)])
def test_failed_layout_is_not_kept(prec, limit):
    """A workspace larger than the device: every attempt is refused, and the context then works on."""
    print(f"layout beyond the device, precision {prec}, limit {limit >> 30} GiB", flush=True)
    c = _ctx(prec)
    want = smpq.smpq_compute_qx_classes(c, [3])
    smpq.smpq_set_point_scheme(c)                 # 49152 right-hand sides
    smpq.smpq_set_memory_limit(c, limit)
    for _ in range(2):
        with pytest.raises(smpq.SmpqError) as e:
            smpq.smpq_prepare(c)
        assert e.value.status == -3
    smpq.smpq_set_memory_limit(c, 0)
    smpq.smpq_set_scheme(c, (2, 2, 2, 2), 0)
    got = smpq.smpq_compute_qx_classes(c, [3])
    assert np.array_equal(want[0], got[0]) and np.array_equal(want[1], got[1])


@pytest.mark.parametrize("prec", [0, 1])
def test_inverse_after_a_shift_check(prec):
    """The unshifted system's coefficients are there whichever call needs them first."""
    print(f"trace of D_W^-1 after a shift check, precision {prec}", flush=True)
    want = smpq.smpq_compute_trinv(_ctx(prec), [3])[0]
    assert np.abs(want).max() > 1.0
    c = _ctx(prec)
    smpq.smpq_set_shift_check(c, True, 0.0)
    smpq.smpq_compute_qx_classes(c, [5])
    smpq.smpq_set_shift_check(c, False)
    assert np.array_equal(smpq.smpq_compute_trinv(c, [3])[0], want)


class Memory:
    """Free device memory, from the HIP runtime the library is linked to."""

    def __init__(self):
        self.hip = ctypes.CDLL("libamdhip64.so.7")

    def free(self):
        a, b = ctypes.c_size_t(), ctypes.c_size_t()
        assert self.hip.hipMemGetInfo(ctypes.byref(a), ctypes.byref(b)) == 0
        return a.value


def test_locality_after_switching_the_check_on():
    """The twelve solves of the locality need a workspace of twelve when the one at hand has no room for the
    check, not one as large as that with the check's vectors on top (70 GB: more than its limit)."""
    print("locality with the shift check on beside a workspace without it", flush=True)
    want = smpq.smpq_dov_locality(_ctx(), 5)[0]
    c, mem = _ctx(), Memory()
    free = mem.free()
    smpq.smpq_set_point_scheme(c)
    smpq.smpq_set_memory_limit(c, 48 << 30)
    smpq.smpq_prepare(c)
    assert free - mem.free() > 40 << 30
    smpq.smpq_set_shift_check(c, True, 0.0)
    assert np.array_equal(smpq.smpq_dov_locality(c, 5)[0], want)
    assert free - mem.free() < 2 << 30        # 12 x (67 + 18) FP64 vectors of 0.8 MB and small arrays


@pytest.mark.parametrize("vectors", [17, 25, 40])      # K = 1, 5 and 20 of the locality's 14 shifts
def test_locality_and_deflation_keep_to_the_limit(vectors):
    """A memory limit of 12 x (K + 17) FP64 vectors (16 + K with K > 1) or a little more: what the locality
    holds afterwards stays below it, and so does what the inner solves of a deflation hold."""
    dims = (16, 16, 16, 16)
    vec = 192 * 16 ** 4
    print(f"locality and deflation within {vectors} vectors a source", flush=True)
    c, mem = _ctx(0, dims), Memory()
    smpq.smpq_dov_locality(_ctx(0, dims), 5)           # the library's own one-time allocations
    small = 48 << 20                                   # reductions, scalars, scheme arrays, graphs
    free = mem.free()
    smpq.smpq_set_memory_limit(c, 12 * vectors * vec)
    m = smpq.smpq_dov_locality(c, 5)[0]
    assert free - mem.free() <= 12 * vectors * vec + small
    assert np.array_equal(m, smpq.smpq_dov_locality(_ctx(0, dims), 5)[0])
    # deflation: one source and one shift, 4 vectors with K = 1 (54 with K = 50)
    c = _ctx(0, dims)
    free = mem.free()
    smpq.smpq_set_memory_limit(c, 4 * vec)
    with pytest.raises(smpq.SmpqError) as e:
        smpq.smpq_deflate(c, 1, 4)                     # too few steps: refused after the solves
    assert e.value.status == -5
    assert free - mem.free() <= 4 * vec + 4 * vec + small      # and the four vectors of the bounds


@pytest.mark.parametrize("check", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
def test_limits_pick_the_block_lengths(prec, check, monkeypatch, capfd):
    """A limit with room for K residuals a source gives blocks of K iterations, and every length the same
    q(x).  In mixed precision K = 2 needs the check: without it five residuals leave room for the reliable
    updates' two FP64 vectors and take less memory than two with these vectors beside them."""
    monkeypatch.setenv("SMPQ_TRACE", "1")
    c = _ctx(prec, (6, 4, 4, 6))
    if check:
        smpq.smpq_set_shift_check(c, True, 0.0)
    vec, ns, want = 192 * 768, 14, None
    capfd.readouterr()
    for k in (50, 20, 10, 5, 2, 1):
        n = k + 1 + ns + (k > 1)
        if prec == 0:
            slot = (n + 1) * vec + (ns + 4) * vec * check
        else:
            slot = n * vec // 2 + (2 if k >= 5 and not check else 4) * vec + (ns + 2) * vec * check
        smpq.smpq_set_memory_limit(c, 12 * slot)
        got = smpq.smpq_compute_qx_classes(c, [5])
        used = [int(v) for v in re.findall(r"blocks of (\d+)", capfd.readouterr().err)]
        assert used == [5 if k == 2 and prec == 1 and not check else k]
        want = want if want is not None else got[0]
        assert np.array_equal(got[0], want), k


def test_large_workspace_outlives_a_small_call(monkeypatch, capfd):
    """A map's workspace of 90 GB in blocks of 5 (more batches with longer ones) serves a call with one
    source class as it is."""
    print("a small call beside a large workspace", flush=True)
    want = smpq.smpq_compute_qx_points(_ctx(1), [7])[0]
    monkeypatch.setenv("SMPQ_TRACE", "1")
    c, mem = _ctx(1), Memory()
    smpq.smpq_set_point_scheme(c)
    smpq.smpq_set_memory_limit(c, 90 * 10 ** 9)
    smpq.smpq_prepare(c)
    free = mem.free()
    capfd.readouterr()
    got = smpq.smpq_compute_qx_points(c, [7])[0]
    assert re.findall(r"blocks of (\d+)", capfd.readouterr().err) == ["5"]
    assert abs(mem.free() - free) < 1 << 30
    assert np.array_equal(got, want)
