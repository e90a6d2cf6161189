"""GPU: contexts at work at the same time on one device.  A context captures graphs throughout its first
solve; set-up, results and copies of another context must neither fail beside that nor break it."""
import threading

import numpy as np
import pytest

import smpq_inputs as si

pytestmark = pytest.mark.gpu

import paper_1901_02211_amd as smpq  # noqa: E402

SHAPES = [((8, 8, 8, 8), 0, [0, 1, 2]), ((4, 4, 4, 8), 1, [0, 3]), ((12, 12, 12, 12), 1, [1, 2])]


def _ctx(dims, prec):
    c = smpq.smpq_create(dims, 0)
    smpq.smpq_load_gauge(c, si.near_identity_su3(dims, 0.3, 7))
    smpq.smpq_set_zolotarev(c, 14, 0.15, 2.75)
    smpq.smpq_set_scheme(c, (2, 2, 2, 2), 0)
    smpq.smpq_set_solver(c, prec, 1e-12, 10000, 50)
    return c


def test_new_contexts_solve_together():
    """Nothing captured yet: the smallest context copies its results out while the others capture."""
    want = [smpq.smpq_compute_qx_classes(_ctx(d, p), cl)[0] for d, p, cl in SHAPES]
    for i in range(3):
        print(f"new contexts together, pass {i}", flush=True)
        ctxs = [_ctx(d, p) for d, p, _ in SHAPES]
        got = smpq.smpq_compute_qx_multi(ctxs, [cl for _, _, cl in SHAPES])
        for w, g in zip(want, got):
            assert np.array_equal(w, g[0])


def test_set_up_beside_a_first_solve():
    """One thread sets contexts up and solves on a small lattice while another solves on new ones."""
    print("set-up beside a first solve", flush=True)
    dims, prec, cl = SHAPES[0]
    want = smpq.smpq_compute_qx_classes(_ctx(dims, prec), cl)[0]
    errors, done = [], threading.Event()

    def small():
        try:
            for _ in range(200):
                c = _ctx((4, 4, 4, 4), 1)
                smpq.smpq_compute_qx_points(c, [0, 3])
                smpq.smpq_compute_trinv(c, [1])
                if done.is_set():
                    break
        except smpq.SmpqError as e:
            errors.append(e)

    t = threading.Thread(target=small)
    t.start()
    try:
        got = [smpq.smpq_compute_qx_classes(_ctx(dims, prec), cl)[0] for _ in range(6)]
    finally:
        done.set()
        t.join()
    assert not errors
    for g in got:
        assert np.array_equal(g, want)
