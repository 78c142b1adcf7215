"""Dslash launches that keep the links of the first directions in the memory-side
cache (stages -12, -22, -32, -42, which only the tuner chooses): bit for bit the
results of the streaming launches."""
import pytest
import torch

import oracle
from gpu_util import need_gpu
from paper_2302_09224_amd import inputs
from test_gpu_wave_blocks import load_shape

pytestmark = pytest.mark.gpu


def test_kept_shapes_by_file_only(tmp_path):
    hisq = need_gpu()
    dims = (6, 8, 10, 12)
    load_shape(hisq, tmp_path, "single", 18, dims, 1, [0], (1, 1, -42, 64, 0, 1))
    assert "rhs-block 1: nr 1 rg 1 stage -42 block 64 grid 0 sweep 1" in hisq.hisq_tune_report()
    hisq.hisq_tune_clear()
    for stage in (-12, -42):                # not a shape to pin
        with pytest.raises(hisq.HisqError):
            hisq.hisq_tune_set("single", dims, 1, 1, 1, stage, 128, 0)
    for shape in ((1, 1, -52, 128, 0, 0), (1, 1, -2 - 5, 128, 0, 0), (1, 2, -12, 128, 0, 0), (2, 1, -12, 128, 0, 0)):
        with pytest.raises(hisq.HisqError):
            load_shape(hisq, tmp_path, "single", 18, dims, shape[0] * shape[1], [0], shape)
    hisq.hisq_tune_clear()


@pytest.mark.parametrize("dims", [(4, 6, 6, 4), (6, 10, 8, 12)])
@pytest.mark.parametrize("name,recon", [("single", 18), ("single", 12), ("double", 18), ("double", 12), ("double", 8),
                                        ("int20", 18), ("int20", 12), ("int30", 12), ("int30", 8)])
def test_kept_links(tmp_path, dims, name, recon):
    hisq = need_gpu()
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    f = hisq.fmt(name)
    pg = hisq.pack_gauge(fat, lng, dims, f.gauge, long_recon=recon)
    pin = hisq.pack_spinor(inputs.gaussian_spinor(oracle.volume(dims) // 2, 5, device="cuda"), f.spinor)
    hisq.hisq_tune_clear()
    hisq.hisq_tune_set(name, dims, 1, 1, 1, 2, 256, 0, long_recon=recon)
    ref = [hisq.dslash(pin, pg, p, f) for p in (0, 1)]
    for stage in (-12, -22, -32, -42):
        for block, grid, sweep in ((64, 0, 1), (128, 0, 2), (256, 2048, 0)):
            load_shape(hisq, tmp_path, name, recon, dims, 1, [0], (1, 1, stage, block, grid, sweep))
            for p in (0, 1):
                assert torch.equal(hisq.dslash(pin, pg, p, f), ref[p]), (stage, block, grid, sweep, p)
    hisq.hisq_tune_clear()


@pytest.mark.parametrize("name,recon", [("single", 18), ("int20", 12), ("int30", 12)])
def test_kept_links_cg(tmp_path, monkeypatch, name, recon):
    """the guarded launches with a fused reduction: the same iterates as streaming"""
    hisq = need_gpu()
    monkeypatch.setenv("HISQ_TUNE", "0")    # the FP64 operator in one shape throughout
    dims, mass = (6, 10, 8, 12), 0.1
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    b = inputs.gaussian_spinor(oracle.parity_sites(dims, 0).size, inputs.RHS_SEED, device="cuda")
    g64 = hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_F64)
    gs = hisq.pack_gauge(fat, lng, dims, hisq.fmt(name).gauge, long_recon=recon)
    got = []
    for stage in (-2, -12, -42):
        load_shape(hisq, tmp_path, name, recon, dims, 1, [0], (1, 1, stage, 128, 0, 0))
        x, st = hisq.cg_solve(b, g64, gs, mass, tol=1e-10, sloppy=name)
        assert st["status"] == "HISQ_OK", st
        got.append((x, st["iters"]))
    hisq.hisq_tune_clear()
    for x, n in got[1:]:
        assert n == got[0][1] and torch.equal(x, got[0][0])


# links of 111, 80 and 255 MB: all directions of the first two kept by the solver's rule, three of the last
@pytest.mark.parametrize("dims,name,recon", [((20, 20, 20, 24), "single", 18), ((20, 20, 20, 24), "int30", 8),
                                             ((24, 24, 24, 32), "single", 18)])
def test_solver_rule(tmp_path, monkeypatch, dims, name, recon):
    """a shape that hisq_tune_set fixed streams, the same shape from a file keeps: the same iterates"""
    hisq = need_gpu()
    monkeypatch.setenv("HISQ_TUNE", "0")
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    b = inputs.gaussian_spinor(oracle.volume(dims) // 2, inputs.RHS_SEED, device="cuda")
    g64 = hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_F64)
    gs = hisq.pack_gauge(fat, lng, dims, hisq.fmt(name).gauge, long_recon=recon)
    got = []
    for fixed in (True, False):
        load_shape(hisq, tmp_path, name, recon, dims, 1, [0], (1, 1, -2, 128, 0, 0))
        if fixed:
            hisq.hisq_tune_set(name, dims, 1, 1, 1, -2, 128, 0, long_recon=recon)
        x, st = hisq.cg_solve(b, g64, gs, 0.5, tol=1e-6, sloppy=name)
        assert st["status"] == "HISQ_OK", st
        got.append((x, st["iters"]))
    hisq.hisq_tune_clear()
    assert got[0][1] == got[1][1] and torch.equal(got[0][0], got[1][0])
