"""CG and batched CG on an operator that is not positive definite: the status, what
it counts, and the iterate it hands back."""
import pytest
import torch

import oracle
from gpu_util import need_gpu
from paper_2302_09224_amd import inputs

pytestmark = pytest.mark.gpu

DIMS, MASS = (8, 8, 8, 12), 0.05


def solve(hisq, sloppy, shift, nrhs=0, **opts):
    """(status, stats, x0, x)"""
    fat, lng = inputs.make_links(DIMS, "near_unit", device="cuda")
    f, vh = hisq.fmt(sloppy), oracle.volume(DIMS) // 2
    g64, gs = hisq.pack_gauge(fat, lng, DIMS, hisq.GAUGE_F64), hisq.pack_gauge(fat, lng, DIMS, f.gauge)
    b = torch.view_as_real(inputs.gaussian_spinor(vh, inputs.RHS_SEED, nrhs=max(1, nrhs)).cuda())
    x0 = 0.5 * b
    x, p = x0.clone(), hisq.hisq_solver_params_default()
    for k, v in opts.items():
        setattr(p, k, v)
    n = hisq.hisq_cg_batched_workspace_bytes(DIMS, nrhs, f, p) if nrhs else hisq.hisq_cg_workspace_bytes(DIMS, f, p)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    if nrhs:
        status, st = hisq.hisq_cg_solve_batched(x, b, nrhs, g64.desc, gs.desc, MASS, shift, 1e-10, f, p, ws, n)
    else:
        status, st = hisq.hisq_cg_solve(x, b, g64.desc, gs.desc, MASS, shift, 1e-10, f, p, ws, n)
    return status, st.as_dict(), x0, x


# negative definite: <p, A p> < 0 at once; ring lengths at which the first iteration is the last slot, or is not
@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("grad_buffer", [1, 8])
@pytest.mark.parametrize("sloppy", ["single", "half"])
def test_first_step(sloppy, grad_buffer, graph):
    hisq = need_gpu()
    status, st, x0, x = solve(hisq, sloppy, -50.0, grad_buffer=grad_buffer, use_graph=graph)
    assert status == -5 and st["iters"] == 0, st
    assert torch.equal(x, x0)


# indefinite: <p, A p> changes sign after some iterations
@pytest.mark.parametrize("grad_buffer", [1, 3, 8])
def test_later_step(grad_buffer):
    hisq = need_gpu()
    status, st, _, x = solve(hisq, "double", -6.0, grad_buffer=grad_buffer, delta=0.0)
    assert status == -5 and st["iters"] > 0, st
    assert bool(torch.isfinite(x).all())


# a step that no system can take does not count, as in a lone solve
@pytest.mark.parametrize("nrhs", [1, 3, 12])
def test_batched_first_step(nrhs):
    hisq = need_gpu()
    status, st, x0, x = solve(hisq, "half", -50.0, nrhs=nrhs)
    assert status == -5 and st["iters"] == 0 and st["refine_iters"][:nrhs] == [0] * nrhs, st
    assert torch.equal(x, x0)


@pytest.mark.parametrize("solver", ["cg", "batched", "multishift", "bicgstab"])
def test_zero_source(solver):
    """x = 0 whatever the initial guess"""
    hisq = need_gpu()
    fat, lng = inputs.make_links(DIMS, "near_unit", device="cuda")
    g64, gs = hisq.pack_gauge(fat, lng, DIMS, hisq.GAUGE_F64), hisq.pack_gauge(fat, lng, DIMS, hisq.GAUGE_F32)
    n = oracle.volume(DIMS) // (1 if solver == "bicgstab" else 2)
    x0 = inputs.gaussian_spinor(n, inputs.RHS_SEED, device="cuda")
    b = torch.zeros_like(x0)
    if solver == "cg":
        x, st = hisq.cg_solve(b, g64, gs, MASS, x0=x0)
    elif solver == "batched":
        x, st = hisq.cg_solve_batched(torch.stack([b, b]), g64, gs, MASS, sloppy="single", x0=torch.stack([x0, x0]))
    elif solver == "bicgstab":
        x, st = hisq.bicgstab_solve(b, g64, gs, MASS, x0=x0)
    else:
        x, st = hisq.multishift_cg_solve(b, [0.0, 0.1], 1e-10, g64, gs, gs, MASS, ref_fmt="single")
        x = torch.stack(x)
    assert st["status"] == "HISQ_OK" and not bool(x.any()), st
