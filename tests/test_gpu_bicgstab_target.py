"""BiCGStab(l) meets tol |b|, whatever the size of b: powers of two leave every
rounding of the method as it is, so a scaled source takes the same steps to the
scaled solution."""
import pytest
import torch

import oracle
from gpu_util import need_gpu
from paper_2302_09224_amd import inputs

pytestmark = pytest.mark.gpu


# with delta 0 the residual is checked where the iterated one meets the target and nowhere else
@pytest.mark.parametrize("delta,tol", [(0.1, 1e-9), (1e-3, 1e-9), (0.0, 1e-5)])
@pytest.mark.parametrize("sloppy,l", [("single", 4), ("int20", 1)])
def test_scaled_sources_take_the_same_steps(sloppy, l, delta, tol):
    hisq = need_gpu()
    dims, mass = (6, 10, 4, 12), 0.1
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    g64 = hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_F64, long_recon=12)
    gs = hisq.pack_gauge(fat, lng, dims, hisq.fmt(sloppy).gauge)
    b = inputs.gaussian_spinor(oracle.volume(dims), inputs.SOURCE_SEED, device="cuda")
    got = []
    for k in (0, 20, -20):
        x, st = hisq.bicgstab_solve(b * 2.0 ** k, g64, gs, mass, tol=tol, l=l, sloppy=sloppy, delta=delta,
                                    maxiter=4000)
        assert st["status"] == "HISQ_OK" and st["true_resid"] <= tol, (k, st)
        got.append((x * 2.0 ** -k, st["iters"], st["reliable_updates"]))
    for x, n, rus in got[1:]:
        assert (n, rus) == got[0][1:] and torch.equal(x, got[0][0]), [g[1:] for g in got]
    if delta == 0.0 and sloppy == "single":
        assert got[0][2] == 1
