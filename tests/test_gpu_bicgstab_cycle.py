"""The fused cycle of BiCGStab(l): Gram-Schmidt rows of every register width,
block partials on both sides of the line where a launch of its own adds them up,
both parities in one Dslash; the true residual by the oracle's operator."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import need_gpu
from paper_2302_09224_amd import inputs

pytestmark = pytest.mark.gpu


def solve(dims, sloppy, recon, l, tol=1e-10, **opts):
    hisq = need_gpu()
    mass = 0.1
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    b = inputs.gaussian_spinor(oracle.volume(dims), inputs.SOURCE_SEED, device="cuda")
    g64 = hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_F64, long_recon=12)
    gs = hisq.pack_gauge(fat, lng, dims, hisq.fmt(sloppy).gauge, long_recon=recon)
    x, st = hisq.bicgstab_solve(b, g64, gs, mass, tol=tol, l=l, sloppy=sloppy, **opts)
    b = b.cpu().numpy()
    r = b - oracle.full_op(fat.cpu().numpy(), lng.cpu().numpy(), x.cpu().numpy(), dims, mass)
    return st, np.linalg.norm(r) / np.linalg.norm(b), x


@pytest.mark.parametrize("l", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("sloppy,recon", [("single", 18), ("int30", 8)])
def test_every_row_width(l, sloppy, recon):
    st, res, _ = solve((6, 10, 4, 12), sloppy, recon, l)
    assert st["status"] == "HISQ_OK" and res <= 1e-10 * (1 + 1e-6), (st, res)


# sites of the whole lattice over 256 a block: 1, 405 (the last block ragged), 512 and 576 blocks (either side of the
# Gram-Schmidt's line), 1024 (above every line)
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (12, 12, 24, 30), (16, 16, 16, 32), (16, 16, 24, 24), (16, 16, 32, 32)])
def test_partials_on_both_sides_of_the_line(dims):
    st, res, _ = solve(dims, "int20", 12, 4)
    assert st["status"] == "HISQ_OK" and res <= 1e-10 * (1 + 1e-6), (st, res)


@pytest.mark.parametrize("maxiter", [1, 8, 9, 24])
def test_cap_counts_whole_cycles(maxiter):
    st, res, x = solve((6, 10, 4, 12), "half", 12, 4, tol=1e-12, maxiter=maxiter)
    assert st["status"] == "HISQ_ENOCONV" and st["iters"] == 8 * -(-maxiter // 8)
    assert abs(res - st["true_resid"]) <= 1e-3 * res and bool(torch.isfinite(torch.view_as_real(x)).all())
