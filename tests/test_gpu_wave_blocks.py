"""Dslash launches in blocks of one wave (which the tuner chooses on small
lattices, and which reach the table through a tune cache file) and the two
launch forms of several lattices: bit for bit the results of the other shapes."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import need_gpu
from paper_2302_09224_amd import inputs

pytestmark = pytest.mark.gpu

TID = {"single": (1, 1, 0), "double": (0, 0, 1), "int20": (2, 3, 0), "int30": (3, 4, 1)}


def load_shape(hisq, tmp_path, name, recon, dims, c, red, shape):
    """enter `shape` (nr, rg, stage, block, grid, sweep) through a cache file"""
    hisq.hisq_tune_clear()
    hisq.hisq_tune_set(name, dims, 1, 1, 1, 2, 128, 0, long_recon=recon)
    path = tmp_path / "t.txt"
    hisq.hisq_tune_save(path)
    head = [ln for ln in path.read_text().splitlines() if ln.startswith("hisq-tune")][0].split()
    g, s, r = TID[name]
    tid = g * 10000 + s * 1000 + r * 100 + recon
    path.write_text("\n".join(" ".join(head[:4] + [str(tid), *map(str, dims), str(c), str(k), ":", *map(str, shape),
                                                   "1.0"]) for k in red) + "\n")
    hisq.hisq_tune_clear()
    assert hisq.hisq_tune_load(path) == len(red)


def test_cache_line_layout(tmp_path):
    hisq = need_gpu()
    load_shape(hisq, tmp_path, "single", 18, (6, 8, 10, 12), 1, [0], (1, 1, -2, 64, 0, 1))
    assert "lattice 6x8x10x12 rhs-block 1: nr 1 rg 1 stage -2 block 64 grid 0 sweep 1" in hisq.hisq_tune_report()
    hisq.hisq_tune_clear()
    with pytest.raises(hisq.HisqError):     # more lanes to a site than its partials have room for
        load_shape(hisq, tmp_path, "single", 18, (6, 8, 10, 12), 16, [0], (1, 16, 1, 64, 0, 1))
    with pytest.raises(hisq.HisqError):     # not a shape to pin
        hisq.hisq_tune_set("single", (6, 8, 10, 12), 1, 1, 1, 2, 64, 0)
    hisq.hisq_tune_clear()


# 288 sites per parity: half of the last wave idle; the other has a z-slab order with padded slices
@pytest.mark.parametrize("dims", [(4, 6, 6, 4), (6, 10, 8, 12)])
@pytest.mark.parametrize("name,recon", [("single", 18), ("double", 12), ("int20", 12), ("int30", 8)])
def test_wave_blocks_single(tmp_path, dims, name, recon):
    hisq = need_gpu()
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    f = hisq.fmt(name)
    pg = hisq.pack_gauge(fat, lng, dims, f.gauge, long_recon=recon)
    pin = hisq.pack_spinor(inputs.gaussian_spinor(oracle.volume(dims) // 2, 5, device="cuda"), f.spinor)
    hisq.hisq_tune_clear()
    hisq.hisq_tune_set(name, dims, 1, 1, 1, 2, 256, 0, long_recon=recon)
    ref = [hisq.dslash(pin, pg, p, f) for p in (0, 1)]
    for stage in (1, 8, -2):
        for sweep in (0, 1, 2):
            load_shape(hisq, tmp_path, name, recon, dims, 1, [0], (1, 1, stage, 64, 0, sweep))
            for p in (0, 1):
                assert torch.equal(hisq.dslash(pin, pg, p, f), ref[p]), (stage, sweep, p)
    hisq.hisq_tune_clear()


@pytest.mark.parametrize("nr,rg,stage", [(1, 8, 1), (2, 4, -1), (4, 2, -1), (8, 1, 1)])
@pytest.mark.parametrize("block,sweep", [(64, 0), (64, 2), (128, 1)])
def test_wave_blocks_batched_cg(tmp_path, nr, rg, stage, block, sweep):
    """fused partials of small blocks: the true residual by the oracle's operator"""
    hisq = need_gpu()
    dims, mass = (6, 10, 8, 12), 0.1
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    ev = oracle.parity_sites(dims, 0)
    b = inputs.gaussian_spinor(ev.size, inputs.RHS_SEED, device="cuda", nrhs=7)
    g64 = hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_F64)
    gs = hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_FIX16, long_recon=12)
    load_shape(hisq, tmp_path, "int20", 12, dims, 8, [0, 1], (nr, rg, stage, block, 0, sweep))
    x, st = hisq.cg_solve_batched(b, g64, gs, mass, tol=1e-10, sloppy="int20")
    hisq.hisq_tune_clear()
    assert st["status"] == "HISQ_OK", st
    fat, lng = fat.cpu().numpy(), lng.cpu().numpy()
    for j in range(7):
        xf = np.zeros((oracle.volume(dims), 3), dtype=np.complex128)
        bf = np.zeros_like(xf)
        xf[ev], bf[ev] = x[j].cpu().numpy(), b[j].cpu().numpy()
        assert oracle.true_residual(fat, lng, xf, bf, dims, mass) <= 1e-10 * (1 + 1e-6)


# sites per parity in all: 65536 (the most that go in blocks of one wave), 65664 (the XCD order, the second lattice's
# blocks padded to an eighth), eight lattices of which none fills a block
@pytest.mark.parametrize("lattices", [[(16, 16, 16, 16), (16, 16, 16, 16)], [(16, 16, 16, 32), (4, 4, 4, 4)],
                                      [(4, 4, 4, 4 + 2 * k) for k in range(8)]])
@pytest.mark.parametrize("name,recon", [("int20", 12), ("double", 18)])
def test_lattices_on_both_sides_of_the_line(lattices, name, recon):
    hisq = need_gpu()
    f = hisq.fmt(name)
    gauges, ins = [], []
    for k, d in enumerate(lattices):
        fat, lng = inputs.make_links(d, "near_unit", seed=70 + k, device="cuda")
        gauges.append(hisq.pack_gauge(fat, lng, d, f.gauge, long_recon=recon))
        ins.append(hisq.pack_spinor(inputs.gaussian_spinor(oracle.volume(d) // 2, 80 + k, device="cuda"), f.spinor))
    outs = [torch.zeros_like(v) for v in ins]
    for parity in (0, 1):
        hisq.hisq_dslash_multi(outs, ins, [g.desc for g in gauges], parity, f)
        for o, i, g in zip(outs, ins, gauges):
            assert torch.equal(o, hisq.dslash(i, g, parity, f))
