"""CG and multi-shift CG whose vector kernels form the iteration's scalars
themselves, on both sides of the line where a launch of its own adds the block
partials up first: every solve reaches its true residual (the oracle's FP64
operator), with and without captured graphs, for rings of odd length and for
both reliable-update triggers."""
import pytest
import torch

import oracle
from gpu_util import need_gpu
from paper_2302_09224_amd import inputs

pytestmark = pytest.mark.gpu

MASS, TOL = 0.1, 1e-10
# sites per parity: 128 (half a block), 4320 (a ragged last block), 262144 (as many partials as are added up
# directly), 266240 (the next larger count: the launch of its own)
DIMS = [(4, 4, 4, 4), (6, 10, 12, 12), (32, 32, 32, 16), (32, 32, 20, 26)]


def solve_and_check(dims, sloppy, nshift, **opts):
    hisq = need_gpu()
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    ev = oracle.parity_sites(dims, 0)
    b = inputs.gaussian_spinor(ev.size, inputs.SOURCE_SEED, device="cuda")
    g64 = hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_F64, long_recon=12)
    gs = hisq.pack_gauge(fat, lng, dims, hisq.fmt(sloppy).gauge, long_recon=12)
    if nshift:
        shifts = [0.01 * 4.0 ** i for i in range(nshift)]
        xs, st = hisq.multishift_cg_solve(b, shifts, TOL, g64, gs, gs, MASS, ms_fmt=sloppy, ref_fmt=sloppy, **opts)
    else:
        shifts = [0.0]
        x, st = hisq.cg_solve(b, g64, gs, MASS, tol=TOL, sloppy=sloppy, **opts)
        xs = [x]
    assert st["status"] == "HISQ_OK", st
    fat, lng = fat.cpu().numpy(), lng.cpu().numpy()
    full = lambda v: torch.zeros((oracle.volume(dims), 3), dtype=torch.complex128).index_copy_(  # noqa: E731
        0, torch.from_numpy(ev), v.cpu()).numpy()
    for s, x in zip(shifts, xs):
        res = oracle.true_residual(fat, lng, full(x), full(b), dims, MASS, s)
        assert res <= TOL * (1 + 1e-6), (s, res, st)


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("nshift", [0, 5])
def test_partials_on_both_sides_of_the_line(dims, nshift):
    solve_and_check(dims, "single", nshift)


@pytest.mark.parametrize("opts", [dict(grad_buffer=1), dict(grad_buffer=3, use_graph=0), dict(grad_buffer=5),
                                  dict(grad_buffer=16, ru_estimate=1), dict(grad_buffer=7, ru_estimate=1, use_graph=0)])
@pytest.mark.parametrize("nshift", [0, 12])
def test_rings_and_triggers(opts, nshift):
    solve_and_check((6, 10, 12, 12), "int30", nshift, **opts)


def small_problem():
    hisq = need_gpu()
    dims = (6, 8, 10, 12)
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    b = inputs.gaussian_spinor(dims[0] * dims[1] * dims[2] * dims[3] // 2, inputs.RHS_SEED, device="cuda", nrhs=3)
    return hisq, b, hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_F64), hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_FIX16)


@pytest.mark.parametrize("batched", [False, True])
def test_units_do_not_change_the_solve(batched):
    """units in flight or not, replayed or enqueued directly: the same bits"""
    hisq, b, g64, gs = small_problem()
    ref = None
    for opts in (dict(), dict(poll_every=8), dict(poll_every=100), dict(poll_every=32, use_graph=0),
                 dict(poll_every=8, use_graph=0)):
        if batched:
            x, st = hisq.cg_solve_batched(b, g64, gs, 0.05, tol=TOL, sloppy="int20", **opts)
        else:
            x, st = hisq.cg_solve(b[0], g64, gs, 0.05, tol=TOL, sloppy="int20", **opts)
        got = (x, st["iters"], st["reliable_updates"], st["true_resid"])
        if ref is None:
            ref = got
        assert torch.equal(x, ref[0]) and got[1:] == ref[1:], (opts, got[1:], ref[1:])


@pytest.mark.parametrize("maxiter", [1, 7, 8, 9, 16, 33])
@pytest.mark.parametrize("batched", [False, True])
def test_iteration_cap_at_the_edges_of_a_unit(batched, maxiter):
    hisq, b, g64, gs = small_problem()
    if batched:
        x, st = hisq.cg_solve_batched(b, g64, gs, 0.01, tol=1e-12, sloppy="int20", maxiter=maxiter)
    else:
        x, st = hisq.cg_solve(b[0], g64, gs, 0.01, tol=1e-12, sloppy="int20", maxiter=maxiter)
    assert st["status"] == "HISQ_ENOCONV" and st["iters"] == maxiter
    assert st["true_resid"] > 1e-12 and bool(torch.isfinite(torch.view_as_real(x)).all())


# 128 sites per parity (one block a row); a ragged last block; above the line where a row's partials are
# added up in a launch of their own (one system: its row has over 512 blocks)
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 10, 12, 12), (24, 24, 24, 24)])
@pytest.mark.parametrize("sloppy,nrhs", [("int20", 1), ("half", 2), ("single", 5), ("int20", 11), ("int24", 16)])
def test_batched_rows(dims, sloppy, nrhs):
    hisq = need_gpu()
    fat, lng = inputs.make_links(dims, "near_unit", device="cuda")
    ev = oracle.parity_sites(dims, 0)
    b = inputs.gaussian_spinor(ev.size, inputs.RHS_SEED, device="cuda", nrhs=nrhs)
    if nrhs > 2:
        b[1] = 0.0    # a system that never iterates
    g64 = hisq.pack_gauge(fat, lng, dims, hisq.GAUGE_F64, long_recon=12)
    gs = hisq.pack_gauge(fat, lng, dims, hisq.fmt(sloppy).gauge, long_recon=12)
    x, st = hisq.cg_solve_batched(b, g64, gs, MASS, tol=TOL, sloppy=sloppy)
    assert st["status"] == "HISQ_OK", st
    fat, lng = fat.cpu().numpy(), lng.cpu().numpy()
    full = lambda v: torch.zeros((oracle.volume(dims), 3), dtype=torch.complex128).index_copy_(  # noqa: E731
        0, torch.from_numpy(ev), v.cpu()).numpy()
    for j in range(nrhs):
        if nrhs > 2 and j == 1:
            assert not bool(x[j].abs().any())
            continue
        res = oracle.true_residual(fat, lng, full(x[j]), full(b[j]), dims, MASS)
        assert res <= TOL * (1 + 1e-6), (j, res, st)
