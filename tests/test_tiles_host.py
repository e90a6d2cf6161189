"""The block-to-site rules of the stencils (csrc/wilson_site.h), built for the host with g++ and checked over plane
shapes and bands (tests/host/tiles_check.cpp)."""
import os
import shutil
import subprocess

import pytest

import paper_1901_02211_amd as smpq

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_every_site_in_one_block(tmp_path):
    exe = str(tmp_path / "tiles_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w",
                    os.path.join(HERE, "host", "tiles_check.cpp"), "-o", exe], check=True, timeout=300)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr
    assert "0 failures" in out.stdout


@pytest.mark.parametrize("band", [0, -1, 2, 3, 5])
def test_any_lattice_variant_takes_any_band(band):
    """The any-lattice kernels have no band and accept every value; the tile kernels need a divisor of nz."""
    c = smpq.smpq_create((12, 12, 4, 4), -1)
    smpq.smpq_set_tuning(c, 0, 4, 1, band)
    assert smpq.smpq_get_tuning(c)["plane_band"] == band
    c = smpq.smpq_create((8, 8, 4, 4), -1)
    if band in (1, 2, 4):
        smpq.smpq_set_tuning(c, 2, 8, 1, band, 1, 4)
    else:
        for args in ((2, 8, 1, band), (0, 4, 1, band, 1, 4)):
            with pytest.raises(smpq.SmpqError) as e:
                smpq.smpq_set_tuning(c, *args)
            assert e.value.status == -1


@pytest.mark.parametrize("dims", [(12, 12, 12, 12), (6, 10, 6, 14), (130, 4, 2, 2), (3, 3, 3, 3), (1, 5, 3, 4)])
def test_reported_default_is_the_one_in_use_without_a_tile(dims):
    """Without a tile every default launch takes the any-lattice kernel with one right-hand side per block: a
    context reports that, and accepts what it reports."""
    c = smpq.smpq_create(dims, -1)
    t = smpq.smpq_get_tuning(c)
    assert (t["f32_kind"], t["f32_nr"], t["f32_dag_kind"], t["f32_dag_nr"]) == (0, 1, 0, 1)
    assert (t["f64_kind"], t["f64_lgr"]) == (0, 0)
    smpq.smpq_set_tuning(c, **t)
    assert smpq.smpq_get_tuning(c) == t


@pytest.mark.parametrize("dims", [(8, 8, 4, 4), (16, 16, 4, 4), (24, 24, 4, 4), (16, 32, 2, 2)])
def test_reported_default_is_accepted_with_a_tile(dims):
    c = smpq.smpq_create(dims, -1)
    t = smpq.smpq_get_tuning(c)
    smpq.smpq_set_tuning(c, **t)
    assert smpq.smpq_get_tuning(c) == t
