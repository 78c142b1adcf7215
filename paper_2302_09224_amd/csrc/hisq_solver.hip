// hisq_solver.hip -- stabilised mixed-precision CG and multi-shift CG (Sec. 3).
//
// Design (MI355X): every scalar of the recurrences lives on the device in a
// SolverCtrl block and is formed by the vector kernel that needs it first, from
// the per-block partials of the preceding kernel summed in a fixed order.  No
// iteration needs the host: the host enqueues units of iterations (optionally as
// one captured hipGraph replayed per unit), the next one before the running one
// has ended, and reads a status record that each unit leaves in host memory.  A
// kernel that decides to leave the loop (reliable update due, convergence
// candidate, multi-shift phase done, breakdown, iteration cap) lowers ctrl->stop,
// and every later kernel of the block sees its guard fail and returns at once.  The host then performs the
// reliable update (FP64 Dslash on the FP64 solution) and starts a new block.
//
// One CG iteration j of a block (slot jb = j mod N_b of the gradient buffer), four launches:
//   t     = D_oe p[jb]                                       (sloppy Dslash)
//   Ap    = c p[jb] - D_eo t,  partial Re<p,Ap>              (sloppy Dslash, fused xpay + dot)
//   alpha = rho / <p,Ap>;  r -= alpha Ap,  partial |r'|^2, Re<r',r>
//   beta  = (|r'|^2 - Re<r',r>) / |r|^2  (Polak-Ribiere, Sec. 3.1 item 3), RU / stop decisions;
//           p[jb+1] = r' + beta p[jb]; at the last slot x64 += sum_j alpha_j p_j in the same
//           pass (buffered FP64 solution update, Sec. 3.1 item 1)
//   [multi-shift, at the last slot: x_i += alpha_i p_i, p_i = zeta_i r' + beta_i p_i replayed
//    for all shifts, one launch]
// Every block of the two vector kernels adds up the partials of the preceding
// kernel and forms the scalars itself; its first block records them.  On large
// lattices a one-block launch adds the partials up first (SUMS_DIRECT).
// Reliable update (Sec. 3 and its footnote, delta = 0.1): flush the buffered
// gradients into x64, r64 = b - A x64 with the FP64 operator, r = pack(r64),
// re-project p against the new r (Sec. 3.1 item 2), then continue.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <functional>
#include <string>
#include <thread>

#include "hisq_internal.h"

namespace hisq {

namespace {

// one block of 16 waves sums the block partials of a whole-lattice launch
// (tens of thousands at 48^3x96); each thread loads its strided share four
// entries at a time (all four in flight) and adds them in index order
constexpr int FIN_THREADS = 1024;

template <int NV>
__device__ __forceinline__ void fin_sums(const double *partial, int n, double (&v)[NV], double *lds) {
#pragma unroll
    for (int k = 0; k < NV; k++) v[k] = 0.0;
    const int step = blockDim.x;
    int b = threadIdx.x;
    for (; b + 3 * step < n; b += 4 * step) {
        double q[4][NV];
#pragma unroll
        for (int u = 0; u < 4; u++)
#pragma unroll
            for (int k = 0; k < NV; k++) q[u][k] = partial[(size_t)(b + u * step) * NV + k];
#pragma unroll
        for (int u = 0; u < 4; u++)
#pragma unroll
            for (int k = 0; k < NV; k++) v[k] += q[u][k];
    }
    for (; b < n; b += step) {
#pragma unroll
        for (int k = 0; k < NV; k++) v[k] += partial[(size_t)b * NV + k];
    }
    block_sum<NV>(v, lds);
}

__global__ void k_fin_b2(SolverCtrl *c, const double *partial, int n) {
    __shared__ double lds[FIN_THREADS / 64];
    double v[1];
    fin_sums<1>(partial, n, v, lds);
    if (threadIdx.x == 0) c->b2 = v[0];
}

// sums of block partials too many for every block of the consumer to add up
template <int NV> __global__ void k_fin_sum(const double *partial, int n, double *out, Guard gd) {
    __shared__ double lds[NV * (FIN_THREADS / 64)];
    if (!gd.pass()) return;
    double v[NV];
    fin_sums<NV>(partial, n, v, lds);
    if (threadIdx.x) return;
#pragma unroll
    for (int k = 0; k < NV; k++) out[k] = v[k];
}

// |b - A x|^2 from the FP64 operator; done when below tol^2 |b|^2
__global__ void k_fin_ru_check(SolverCtrl *c, const double *partial, int n) {
    __shared__ double lds[FIN_THREADS / 64];
    double v[1];
    fin_sums<1>(partial, n, v, lds);
    if (threadIdx.x) return;
    const double r2 = v[0];
    c->r2_true = r2;
    if (!__builtin_isfinite(r2)) {
        c->breakdown = 1;
        c->done = 0;
        c->stop = -1;
        return;
    }
    const int done = r2 <= c->tol2 * c->b2;
    c->done = done;
    c->stop = done ? -1 : STOP_NEVER;
}

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// ---------------------------------------------------------------------------
// library-owned stream (default priority) and pinned host side of the control block
// ---------------------------------------------------------------------------

struct DevState {
    hipStream_t stream = nullptr;
    hipEvent_t ev = nullptr;
    SolverHost *host = nullptr;
    // the second stream of the multi-shift refinement (shifted systems batched
    // while the base system is refined on `stream`)
    hipStream_t stream2 = nullptr;
    hipEvent_t ev2 = nullptr;
    SolverHost *host2 = nullptr;
    std::mutex mu;
};

DevState g_dev[64];

hisq_status dev_state(DevState **out) {
    int d = 0;
    HISQ_TRY_HIP(hipGetDevice(&d));
    if (d < 0 || d >= 64) return set_error(HISQ_EINVAL, "device index %d out of range", d);
    DevState &s = g_dev[d];
    if (!s.stream) {
        HISQ_TRY_HIP(hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking));
        HISQ_TRY_HIP(hipEventCreateWithFlags(&s.ev, hipEventDisableTiming));
        HISQ_TRY(solver_host_alloc(&s.host));
        HISQ_TRY_HIP(hipStreamCreateWithFlags(&s.stream2, hipStreamNonBlocking));
        HISQ_TRY_HIP(hipEventCreateWithFlags(&s.ev2, hipEventDisableTiming));
        HISQ_TRY(solver_host_alloc(&s.host2));
    }
    *out = &s;
    return HISQ_OK;
}

// ---------------------------------------------------------------------------
// workspace layout
// ---------------------------------------------------------------------------

struct Carver {
    size_t off = 0;
    char *base = nullptr;
    char *take(size_t bytes) {
        char *p = base ? base + off : nullptr;
        off += align256(bytes);
        return p;
    }
};

size_t partial_doubles(const Geom &g, int nrhs) {
    const size_t a = dslash_max_blocks(g) * std::max(1, nrhs);
    const size_t b = (size_t)4096 * 4 * std::max(1, nrhs);
    return std::max(a, b);
}

struct CgBuffers {
    SolverCtrl *ctrl;
    double *partial;
    double *ppart;                     // per-block |p|^2 of the last p update
    char *x64, *b64, *r64, *t64;
    char *rs, *aps, *ts;
    char *p[HISQ_MAX_GRAD_BUFFER];
    char *pconv;                       // multi-shift: base gradient vector in the refinement format
    char *xs[HISQ_MAX_SHIFTS];         // multi-shift: FP64 shifted solutions (index >= 1)
    char *ps[HISQ_MAX_SHIFTS];         // multi-shift: shifted gradient vectors at the block's start (index >= 1)
    char *rr[HISQ_MAX_GRAD_BUFFER];    // multi-shift: the base residuals of the block's iterations
};

// sloppy_bytes: bytes/site of the largest sloppy format used; ms_bytes: of the
// multi-shift gradient vectors (0: not a multi-shift solve)
size_t carve_cg(CgBuffers *b, char *base, const Geom &g, int sloppy_bytes, int nb, int nshift, int ms_bytes,
                int ref_bytes) {
    Carver cv;
    cv.base = base;
    const size_t vh = g.vh;
    CgBuffers tmp;
    CgBuffers &B = b ? *b : tmp;
    B.ctrl = (SolverCtrl *)cv.take(sizeof(SolverCtrl));
    B.partial = (double *)cv.take(partial_doubles(g, 1) * sizeof(double));
    B.ppart = (double *)cv.take((size_t)BLAS_MAX_BLOCKS * sizeof(double));
    B.x64 = cv.take(48 * vh);
    B.b64 = cv.take(48 * vh);
    B.r64 = cv.take(48 * vh);
    B.t64 = cv.take(48 * vh);
    B.rs = cv.take(sloppy_bytes * vh);
    B.aps = cv.take(sloppy_bytes * vh);
    B.ts = cv.take(sloppy_bytes * vh);
    for (int i = 0; i < HISQ_MAX_GRAD_BUFFER; i++) B.p[i] = i < nb ? cv.take(sloppy_bytes * vh) : nullptr;
    B.pconv = nullptr;
    for (int i = 0; i < HISQ_MAX_SHIFTS; i++) B.xs[i] = B.ps[i] = nullptr;
    for (int i = 0; i < HISQ_MAX_GRAD_BUFFER; i++) B.rr[i] = nullptr;
    if (ms_bytes > 0) {
        B.pconv = cv.take(ref_bytes * vh);
        for (int i = 1; i < nshift; i++) {
            B.xs[i] = cv.take(48 * vh);
            B.ps[i] = cv.take((size_t)ms_bytes * vh);
        }
        if (nshift > 1)
            for (int q = 0; q < nb; q++) B.rr[q] = cv.take((size_t)ms_bytes * vh);
    }
    return cv.off;
}

int sloppy_floor_bits(int sf) {
    switch (sf) {
    case SF_F64: return 52;
    case SF_F32: return 24;
    case SF_HALF16: return 15;
    case SF_INT20: return 19;
    case SF_INT30: return 29;
    case SF_INT24: return 23;
    }
    return 24;
}

// ---------------------------------------------------------------------------
// one CG (or multi-shift) run on prepared buffers
// ---------------------------------------------------------------------------

struct Run {
    Geom g;
    size_t vh;
    hisq_fmt fmt;              // sloppy triplet
    const hisq_gauge *g64, *gs;
    double c;                  // 4m^2 + shift of the system being iterated
    int nb;
    int unit;                  // iterations enqueued (and captured) as a whole, a multiple of nb
    int depth;                 // units kept in flight at most
    bool graph;
    bool multishift;
    bool ru_est;
    int nshift;
    CgBuffers *B;
    hipStream_t st;
    SolverHost *h = nullptr;   // pinned host side of the control block
    Status last{};             // the last status record read
    int inflight = 0;          // units enqueued whose records have not been read
    // counters
    long dslash_sloppy = 0, dslash_f64 = 0, rus = 0, iters = 0;
    double alg_bytes = 0.0;
    int maxiter = 0;
    int last_slot = 0;         // slot of the current gradient vector when the run ended
    hipGraphExec_t exec = nullptr;
    DslashPlan plan_s{}, plan_64{};
    int nb_s = 0, nb_64 = 0;

    // launch shapes of the sloppy and FP64 Dslash (autotuned on first use, outside capture)
    void setup_plans() {
        const hisq_fmt f64 = {HISQ_GAUGE_F64, HISQ_SPINOR_F64, 64};
        DslashArgs ps = dargs(gs, B->ts, B->rs, 1);
        plan_s = dslash_plan(fmt, g, 1, &ps, st);
        dslash_keep_links(fmt, g, ps.long_recon, plan_s);
        nb_s = dslash_tile_blocks(g, plan_s.tile[0]);
        DslashArgs p64 = dargs(g64, B->t64, B->x64, 1);
        plan_64 = dslash_plan(f64, g, 1, &p64, st);
        nb_64 = dslash_tile_blocks(g, plan_64.tile[0]);
        // occupancy queries of the capped-grid kernels, before any capture
        (void)flush_x_grid(vh, fmt.spinor, fmt.compute);
        (void)cg_pupdate_grid(vh, fmt.spinor, fmt.compute, true);
        if (multishift) (void)shift_replay_grid(vh, fmt.spinor, fmt.compute);
    }

    DslashArgs dargs(const hisq_gauge *gg, char *out, const char *in, int parity) const {
        DslashArgs a;
        memset(&a, 0, sizeof(a));
        a.out = out;
        a.in = in;
        a.fat = (const char *)gg->fat;
        a.lng = (const char *)gg->lng;
        a.b = 1.0;
        a.g = g;
        a.parity = parity;
        a.red = RED_NONE;
        a.nrhs = 1;
        gauge_args(a, gg);
        return a;
    }

    hisq_status enq_iteration(int j) {
        const int jb = j % nb, jn = (j + 1) % nb;
        SolverCtrl *c = B->ctrl;
        const Guard gns{&c->stop, j, 0};
        DslashArgs A = dargs(gs, B->ts, B->p[jb], 1);
        A.guard = gns;
        HISQ_TRY_HIP(launch_dslash(A, fmt, plan_s, st, nullptr));
        DslashArgs Bk = dargs(gs, B->aps, B->ts, 0);
        Bk.b = -1.0;
        Bk.x = B->p[jb];
        Bk.a = c_;
        Bk.red = RED_DOT_X;
        Bk.partial = B->partial;
        Bk.guard = gns;
        HISQ_TRY_HIP(launch_dslash(Bk, fmt, plan_s, st, nullptr));
        Sums pap, rr, pp{nullptr, 0};
        HISQ_TRY(enq_sums<1>(B->partial, nb_s, SUMS_PAP, gns, &pap));
        HISQ_TRY_HIP(launch_cg_axpy(B->rs, B->aps, c, pap, vh, fmt.spinor, fmt.compute, rpart(), jb, gns, st,
                                    multishift ? B->rr[jb] : nullptr));
        HISQ_TRY(enq_sums<2>(rpart(), blas_blocks(vh), SUMS_RR, gns, &rr));
        // |p_k|^2 is summed before the update that overwrites its partials
        if (ru_est) HISQ_TRY(enq_sums<1>(B->ppart, blas_blocks(vh), SUMS_PP, gns, &pp, true));
        SpinorList pl;
        for (int i = 0; i < HISQ_MAX_SHIFTS; i++) pl.p[i] = i < nb ? B->p[i] : nullptr;
        HISQ_TRY_HIP(launch_cg_pupdate(B->p[jn], B->rs, B->p[jb], c, rr, pp.p, ru_est ? B->ppart : nullptr, B->x64, pl,
                                       jb == nb - 1 ? nb : 0, multishift ? 1 : 0, jb, vh, fmt.spinor, fmt.compute, gns,
                                       st));
        if (multishift && jb == nb - 1) HISQ_TRY(enq_shift_replay(nb, gns));
        return HISQ_OK;
    }
    // partials of the residual update, apart from the Dslash's that its blocks read
    double *rpart() const { return B->partial + 8192; }

    // block partials for the next kernel: as they are when few, else added up in a launch
    template <int NV>
    hisq_status enq_sums(const double *partial, int n, int place, Guard gd, Sums *out, bool always = false) {
        if (!always && n * NV <= SUMS_DIRECT) {
            *out = Sums{partial, n};
            return HISQ_OK;
        }
        double *red = B->ctrl->red + place;
        hipLaunchKernelGGL((k_fin_sum<NV>), dim3(1), dim3(FIN_THREADS), 0, st, partial, n, red, gd);
        HISQ_TRY_HIP(hipGetLastError());
        *out = Sums{red, 1};
        return HISQ_OK;
    }
    double c_ = 0.0;

    // the shifted systems' updates of the block's first `count` iterations
    hisq_status enq_shift_replay(int count, Guard gd) {
        SpinorList xl, pl, rl;
        for (int i = 0; i < HISQ_MAX_SHIFTS; i++) {
            xl.p[i] = B->xs[i];
            pl.p[i] = B->ps[i];
            rl.p[i] = i < HISQ_MAX_GRAD_BUFFER ? B->rr[i] : nullptr;
        }
        HISQ_TRY_HIP(launch_shift_replay(xl, pl, rl, B->ctrl, nshift, vh, count, fmt.spinor, fmt.compute, gd, st));
        return HISQ_OK;
    }

    // a block ended early at slot jb (reliable update, end of the phase): the
    // shifted systems take the block's iterations so far, and like the base
    // restart at slot 0
    hisq_status realign_shifts(int jb) {
        if (!multishift || jb == nb - 1) return HISQ_OK;
        return enq_shift_replay(jb + 1, Guard{nullptr, 0, 0});
    }

    // r64 = b - (c x64 - D_eo D_oe x64), |r64|^2 -> done flag (FP64 operator)
    hisq_status enq_true_residual() {
        const hisq_fmt f64 = {HISQ_GAUGE_F64, HISQ_SPINOR_F64, 64};
        DslashArgs A = dargs(g64, B->t64, B->x64, 1);
        HISQ_TRY_HIP(launch_dslash(A, f64, plan_64, st, nullptr));
        DslashArgs Bk = dargs(g64, B->r64, B->t64, 0);
        Bk.b = 1.0;
        Bk.x = B->x64;
        Bk.a = -c_;
        Bk.y = B->b64;
        Bk.c = 1.0;
        Bk.red = RED_NORM;
        Bk.partial = B->partial;
        HISQ_TRY_HIP(launch_dslash(Bk, f64, plan_64, st, nullptr));
        hipLaunchKernelGGL(k_fin_ru_check, dim3(1), dim3(FIN_THREADS), 0, st, B->ctrl, B->partial,
                           nb_64);
        HISQ_TRY_HIP(hipGetLastError());
        dslash_f64 += 2;
        alg_bytes += 2.0 * vh * (dslash_link_bytes(g64) + 2 * 48) + 2.0 * vh * 48;
        return HISQ_OK;
    }

    // flush `count` buffered gradients, true residual, repack r, re-project p
    // and write the next gradient vector into slot 0.
    hisq_status enq_reliable(int mode, int count, const char *p_src) {
        SolverCtrl *c = B->ctrl;
        if (count > 0) {
            SpinorList pl;
            for (int i = 0; i < HISQ_MAX_SHIFTS; i++) pl.p[i] = i < nb ? B->p[i] : nullptr;
            HISQ_TRY_HIP(launch_flush_x(B->x64, pl, count, c->alpha_buf, vh, fmt.spinor, fmt.compute, Guard{nullptr, 0, 0}, st));
            alg_bytes += vh * (count * (double)spinor_site_bytes(fmt.spinor) + 96.0);
        }
        HISQ_TRY(enq_true_residual());
        const Guard g0{&c->stop, 0, 0};
        HISQ_TRY_HIP(launch_ru_convert(B->rs, B->r64, mode == 1 ? nullptr : p_src, mode == 0 ? B->aps : nullptr,
                                       &c->alpha, vh, fmt.spinor, fmt.compute, B->partial, g0, st));
        Sums ru;
        HISQ_TRY(enq_sums<4>(B->partial, blas_blocks(vh), SUMS_RU, g0, &ru));
        HISQ_TRY_HIP(launch_ru_pupdate(B->p[0], B->rs, mode == 1 ? B->rs : p_src, c, ru, mode,
                                       ru_est ? B->ppart : nullptr, vh, fmt.spinor, fmt.compute, g0, st));
        const double bs = spinor_site_bytes(fmt.spinor);
        alg_bytes += vh * (48.0 + 5 * bs) + vh * 3 * bs;
        return HISQ_OK;
    }

    hisq_status read_ctrl() {
        HISQ_TRY_HIP(hipMemcpyAsync(&h->ctrl, B->ctrl, sizeof(SolverCtrl), hipMemcpyDeviceToHost, st));
        HISQ_TRY_HIP(hipStreamSynchronize(st));
        inflight = 0;
        return HISQ_OK;
    }

    // the control block's state now (every record still outstanding is skipped)
    hisq_status read_status() {
        HISQ_TRY_HIP(launch_status(B->ctrl, h, 0, st));
        h->launched++;
        inflight = 0;
        return wait_status(h, h->launched, st, &last);
    }

    // a unit of iterations and its status record
    hisq_status enq_unit() {
        if (graph) {
            if (!exec) {
                hipGraph_t gr = nullptr;
                HISQ_TRY_HIP(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
                hisq_status s = HISQ_OK;
                for (int j = 0; j < unit && s == HISQ_OK; j++) s = enq_iteration(j);
                hipError_t es = launch_status(B->ctrl, h, 0, st);
                hipError_t e = hipStreamEndCapture(st, &gr);
                if (e == hipSuccess) e = es;
                if (s != HISQ_OK || e != hipSuccess) {
                    if (gr) (void)hipGraphDestroy(gr);
                    if (s != HISQ_OK) return s;
                }
                HISQ_TRY_HIP(e);
                e = hipGraphInstantiate(&exec, gr, nullptr, nullptr, 0);
                (void)hipGraphDestroy(gr);
                HISQ_TRY_HIP(e);
            }
            HISQ_TRY_HIP(hipGraphLaunch(exec, st));
        } else {
            for (int j = 0; j < unit; j++) HISQ_TRY(enq_iteration(j));
            HISQ_TRY_HIP(launch_status(B->ctrl, h, 0, st));
        }
        h->launched++;
        inflight++;
        return HISQ_OK;
    }

    double iter_bytes() const {
        const double bs = spinor_site_bytes(fmt.spinor), bl = dslash_link_bytes(gs);
        double it = 2.0 * (bl + 2.0 * bs) + bs         // two Dslash + xpay operand
                    + 3.0 * bs                           // r update
                    + 3.0 * bs                           // p update
                    + (nb * bs + 96.0) / nb;             // buffered FP64 solution update
        return it * vh;
    }

    // Iterate until the true residual meets tol (returns OK), or the
    // multi-shift phase ends (OK, *ms_done = 1), or an error.  The next unit is
    // enqueued before the running one is read, unless the pace says that the
    // block stops in what is enqueued already: units behind a stop only return
    // from their guards (1.6 us a launch).  After a reliable update the next
    // unit follows at once; its record tells whether the update met tol.
    hisq_status iterate(int *ms_done) {
        if (ms_done) *ms_done = 0;
        long k0 = last.k;
        Pace pace;
        for (;;) {
            while (inflight < depth && (inflight == 0 || pace.left > (double)inflight * unit)) HISQ_TRY(enq_unit());
            const unsigned long long seq = h->launched - (unsigned long long)inflight + 1;
            HISQ_TRY(wait_status(h, seq, st, &last));
            inflight--;
            if (last.done) return HISQ_OK;
            const long dk = last.k - k0;
            k0 = last.k;
            iters += dk;
            dslash_sloppy += 2 * dk;
            alg_bytes += dk * iter_bytes();
            if (multishift) {
                // the base residual written to the ring and read back once per block; per
                // updated shift, once per block of N_b iterations: its gradient vector read
                // and written and its FP64 solution read and written
                const double bs = spinor_site_bytes(fmt.spinor);
                const int ne = __builtin_popcount((unsigned)last.e_mask);
                alg_bytes += dk * (double)vh * (2.0 * bs + ne * (2.0 * bs + 96.0) / nb);
            }
            if (last.breakdown)
                return set_error(HISQ_EBREAKDOWN, "solver breakdown after %d iterations (pAp = %g, |r|^2 = %g)",
                                 last.k, last.pi, last.rho_new);
            pace.update(last);
            if (last.stop == STOP_NEVER) continue;
            if (last.stop < 0 || last.stop >= unit)
                return set_error(HISQ_EBREAKDOWN, "inconsistent solver state (stop %d, reason %d)", last.stop, last.reason);
            inflight = 0;   // the units behind the stop do nothing; their records are skipped
            const int js = last.stop, jb = js % nb;
            last_slot = jb;
            HISQ_TRY(realign_shifts(jb));
            if (last.reason == STOP_MSDONE) {
                SpinorList pl;
                for (int i = 0; i < HISQ_MAX_SHIFTS; i++) pl.p[i] = i < nb ? B->p[i] : nullptr;
                HISQ_TRY_HIP(launch_flush_x(B->x64, pl, jb + 1, B->ctrl->alpha_buf, vh, fmt.spinor, fmt.compute,
                                            Guard{nullptr, 0, 0}, st));
                if (ms_done) *ms_done = 1;
                return HISQ_OK;
            }
            const int reason = last.reason;
            HISQ_TRY(enq_reliable(0, jb + 1, B->p[jb]));
            rus++;
            last_slot = 0;
            pace.reset();
            if (reason == STOP_RU && last.k < maxiter) continue;
            HISQ_TRY(read_status());
            if (last.breakdown) return set_error(HISQ_EBREAKDOWN, "non-finite true residual");
            if (last.done) return HISQ_OK;
            if (reason == STOP_MAXITER || last.k >= maxiter)
                return set_error(HISQ_ENOCONV, "no convergence in %d iterations (true residual %g)", last.k,
                                 std::sqrt(last.r2_true / last.b2));
        }
    }

    ~Run() {
        // a unit behind the last stop may still be running
        if (exec) {
            (void)hipStreamSynchronize(st);
            (void)hipGraphExecDestroy(exec);
        }
    }
};

void init_ctrl(SolverHost *host, const hisq_solver_params &p, double tol, double b2, int sloppy_spinor) {
    SolverCtrl *h = &host->ctrl;
    memset(h, 0, sizeof(*h));
    h->seq = host->launched;
    h->ru_est = p.ru_estimate;
    h->eps_s = std::ldexp(1.0, -sloppy_floor_bits(sloppy_spinor));
    h->stop = STOP_NEVER;
    h->pr = p.pr_beta;
    h->reproject = p.reproject;
    h->maxiter = p.maxiter;
    h->tol2 = tol * tol;
    h->delta2 = p.delta > 0 ? p.delta * p.delta : 0.0;
    h->b2 = b2;
    h->alpha_prev = 1.0;
    h->beta_prev = 0.0;
}

hisq_status check_params(const hisq_solver_params *p, hisq_solver_params *out) {
    hisq_solver_params d;
    hisq_solver_params_default(&d);
    *out = p ? *p : d;
    if (out->maxiter <= 0) out->maxiter = d.maxiter;
    if (out->grad_buffer < 1 || out->grad_buffer > HISQ_MAX_GRAD_BUFFER)
        return set_error(HISQ_EINVAL, "grad_buffer must be in [1,%d]", HISQ_MAX_GRAD_BUFFER);
    if (out->poll_every <= 0) out->poll_every = d.poll_every;
    if (out->batch_refine < 0 || out->batch_refine > 3)
        return set_error(HISQ_EINVAL, "batch_refine must be 0, 1, 2 or 3");
    if (out->ru_estimate != 0 && out->ru_estimate != 1) return set_error(HISQ_EINVAL, "ru_estimate must be 0 or 1");
    return HISQ_OK;
}

// multi-shift workspace: the solver buffers, then (batched refinement) the
// buffers of a block of min(16, nshift-1) shifted systems (min(16, nshift)
// when the base system joins the block)
struct MsLayout {
    size_t solver, batched;
    bool batch;
};
MsLayout ms_layout(const Geom &g, int nshift, const hisq_fmt &ms_fmt, const hisq_fmt &refine_fmt,
                   const hisq_solver_params &q) {
    MsLayout L;
    const int bs = std::max(spinor_site_bytes(ms_fmt.spinor), spinor_site_bytes(refine_fmt.spinor));
    L.solver = (carve_cg(nullptr, nullptr, g, bs, q.grad_buffer, nshift, spinor_site_bytes(ms_fmt.spinor),
                         spinor_site_bytes(refine_fmt.spinor)) + 255) & ~(size_t)255;
    L.batch = q.batch_refine && nshift > 1 && batched_fmt_ok(refine_fmt);
    const int nblock = std::min(16, q.batch_refine == 3 ? nshift : nshift - 1);
    L.batched = L.batch ? batched_ws_bytes(g, nblock, refine_fmt.spinor, q.grad_buffer) : 0;
    return L;
}

hisq_status check_gauge(const hisq_gauge *gg, const int dims[4], const hisq_fmt &f, const char *what) {
    if (!gg || !gg->fat || !gg->lng) return set_error(HISQ_EINVAL, "%s: null gauge field", what);
    for (int k = 0; k < 4; k++)
        if (gg->dims[k] != dims[k]) return set_error(HISQ_EINVAL, "%s: gauge dims differ from the solve", what);
    if (gg->fmt != f.gauge) return set_error(HISQ_EINVAL, "%s: gauge format %d, triplet wants %d", what, gg->fmt, f.gauge);
    if (!aligned16(gg->fat) || !aligned16(gg->lng)) return set_error(HISQ_EALIGN, "%s: gauge not 16-byte aligned", what);
    if (!recon_ok(f, gg->long_recon, false))
        return set_error(HISQ_EINVAL, "%s: eight-parameter long links need FP64 arithmetic on F64 or FIX32 links", what);
    return HISQ_OK;
}

// |b|^2 of the FP64 SoA b64 into ctrl->b2 (device), returned on the host
hisq_status enq_b2(Run &R) {
    int nbk = 0;
    HISQ_TRY_HIP(launch_norm2_f64(R.B->b64, R.vh, R.B->partial, &nbk, R.st));
    hipLaunchKernelGGL(k_fin_b2, dim3(1), dim3(FIN_THREADS), 0, R.st, R.B->ctrl, R.B->partial, nbk);
    HISQ_TRY_HIP(hipGetLastError());
    return HISQ_OK;
}

// Full CG on prepared buffers (x64, b64 filled).  mode 1: fresh start; mode 2:
// continue the gradient vector p_init (refinement format) with rho_prev.
hisq_status cg_core(Run &R, const hisq_solver_params &p, double tol, int mode, const char *p_init, double rho_prev,
                    double *resid0) {
    init_ctrl(R.h, p, tol, 0.0, R.fmt.spinor);
    R.h->ctrl.rho_prev = rho_prev;
    HISQ_TRY_HIP(hipMemcpyAsync(R.B->ctrl, &R.h->ctrl, sizeof(SolverCtrl), hipMemcpyHostToDevice, R.st));
    R.setup_plans();
    HISQ_TRY(enq_b2(R));
    HISQ_TRY(R.enq_reliable(mode, 0, mode == 2 ? p_init : nullptr));
    HISQ_TRY(R.read_status());
    if (resid0) *resid0 = R.last.b2 > 0 ? std::sqrt(R.last.r2_true / R.last.b2) : 0.0;
    if (R.last.breakdown) return set_error(HISQ_EBREAKDOWN, "non-finite initial residual");
    if (R.last.b2 == 0.0 || R.last.done) return HISQ_OK;
    return R.iterate(nullptr);
}

void fill_common_stats(hisq_solver_stats *s, const Run &R) {
    s->iters += (int)R.iters;
    s->reliable_updates += (int)R.rus;
    s->dslash_sloppy += (int)R.dslash_sloppy;
    s->dslash_f64 += (int)R.dslash_f64;
    s->alg_bytes += R.alg_bytes;
}

struct Entry {
    DevState *ds = nullptr;
    hipStream_t user = nullptr;
    std::unique_lock<std::mutex> lock;
    hisq_status begin(void *stream) {
        HISQ_TRY(dev_state(&ds));
        lock = std::unique_lock<std::mutex>(ds->mu);
        user = (hipStream_t)stream;
        HISQ_TRY_HIP(hipEventRecord(ds->ev, user));
        HISQ_TRY_HIP(hipStreamWaitEvent(ds->stream, ds->ev, 0));
        return HISQ_OK;
    }
    hisq_status end() {
        HISQ_TRY_HIP(hipStreamSynchronize(ds->stream));
        return HISQ_OK;
    }
};

}  // namespace

}  // namespace hisq

using namespace hisq;

extern "C" void hisq_solver_params_default(hisq_solver_params *p) {
    if (!p) return;
    memset(p, 0, sizeof(*p));
    p->delta = 0.1;
    p->maxiter = 100000;
    p->grad_buffer = 8;
    p->pr_beta = 1;
    p->reproject = 1;
    p->poll_every = 32;
    p->use_graph = 1;
    p->shift_floor = 0.0;
    p->batch_refine = 3;
    p->ru_estimate = 0;
}

extern "C" size_t hisq_cg_workspace_bytes(const int dims[4], hisq_fmt sloppy, const hisq_solver_params *p) {
    if (!dims || !dims_ok(dims) || !triplet_ok(sloppy)) return 0;
    hisq_solver_params q;
    if (check_params(p, &q) != HISQ_OK) return 0;
    const Geom g = make_geom(dims);
    return carve_cg(nullptr, nullptr, g, spinor_site_bytes(sloppy.spinor), q.grad_buffer, 0, 0, 0);
}

extern "C" hisq_status hisq_cg_solve(double *x, const double *b, const hisq_gauge *g64, const hisq_gauge *gs,
                                     double mass, double shift, double tol, hisq_fmt sloppy,
                                     const hisq_solver_params *p, void *ws, size_t ws_bytes,
                                     hisq_solver_stats *stats, void *stream) {
    auto t0 = std::chrono::steady_clock::now();
    hisq_solver_stats tmp;
    hisq_solver_stats *st = stats ? stats : &tmp;
    memset(st, 0, sizeof(*st));
    st->status = HISQ_EINVAL;
    if (!x || !b || !g64 || !gs || !ws) return set_error(HISQ_EINVAL, "hisq_cg_solve: null argument");
    if (!aligned16(x) || !aligned16(b) || !aligned16(ws)) return set_error(HISQ_EALIGN, "hisq_cg_solve: unaligned pointer");
    if (!triplet_ok(sloppy)) return set_error(HISQ_EINVAL, "hisq_cg_solve: unsupported sloppy triplet");
    if (!(tol > 0.0)) return set_error(HISQ_EINVAL, "hisq_cg_solve: tol must be > 0");
    const int *dims = g64->dims;
    if (!dims_ok(dims)) return set_error(HISQ_EINVAL, "hisq_cg_solve: bad lattice dims");
    HISQ_TRY(check_gauge(g64, dims, hisq_fmt{HISQ_GAUGE_F64, HISQ_SPINOR_F64, 64}, "g64"));
    HISQ_TRY(check_gauge(gs, dims, sloppy, "gs"));
    hisq_solver_params q;
    HISQ_TRY(check_params(p, &q));
    const Geom g = make_geom(dims);
    CgBuffers B;
    const size_t need = carve_cg(&B, (char *)ws, g, spinor_site_bytes(sloppy.spinor), q.grad_buffer, 0, 0, 0);
    if (ws_bytes < need) return set_error(HISQ_EWORKSPACE, "workspace %zu bytes, need %zu", ws_bytes, need);
    Entry E;
    HISQ_TRY(E.begin(stream));
    Run R;
    R.g = g;
    R.vh = g.vh;
    R.fmt = sloppy;
    R.g64 = g64;
    R.gs = gs;
    R.c_ = 4.0 * mass * mass + shift;
    R.nb = q.grad_buffer;
    solver_unit(q, &R.unit, &R.depth);
    R.maxiter = q.maxiter;
    R.graph = q.use_graph != 0;
    R.multishift = false;
    R.ru_est = q.ru_estimate != 0;
    R.nshift = 1;
    R.B = &B;
    R.st = E.ds->stream;
    R.h = E.ds->host;
    HISQ_TRY_HIP(launch_spinor_pack(B.x64, x, g.vh, SF_F64, R.st));
    HISQ_TRY_HIP(launch_spinor_pack(B.b64, b, g.vh, SF_F64, R.st));
    hisq_status s = cg_core(R, q, tol, 1, nullptr, 0.0, nullptr);
    // b = 0: x = 0 whatever the initial guess
    if (s == HISQ_OK && R.last.b2 == 0.0) HISQ_TRY_HIP(hipMemsetAsync(B.x64, 0, spinor_field_bytes(g.vh, SF_F64), R.st));
    if (s == HISQ_OK || s == HISQ_ENOCONV || s == HISQ_EBREAKDOWN) {
        hipError_t e = launch_spinor_unpack(x, B.x64, g.vh, SF_F64, R.st);
        if (e != hipSuccess && s == HISQ_OK) s = set_error(HISQ_EHIP, "unpack: %s", hipGetErrorString(e));
    }
    hisq_status s2 = E.end();
    if (s == HISQ_OK) s = s2;
    fill_common_stats(st, R);
    st->true_resid = R.last.b2 > 0 ? std::sqrt(R.last.r2_true / R.last.b2) : 0.0;
    st->nshift = 1;
    st->shift_resid[0] = st->true_resid;
    st->status = s;
    st->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return s;
}

extern "C" size_t hisq_multishift_workspace_bytes(const int dims[4], int nshift, hisq_fmt ms_fmt, hisq_fmt refine_fmt,
                                                  const hisq_solver_params *p) {
    if (!dims || !dims_ok(dims) || !triplet_ok(ms_fmt) || !triplet_ok(refine_fmt)) return 0;
    if (nshift < 1 || nshift > HISQ_MAX_SHIFTS) return 0;
    hisq_solver_params q;
    if (check_params(p, &q) != HISQ_OK) return 0;
    const MsLayout L = ms_layout(make_geom(dims), nshift, ms_fmt, refine_fmt, q);
    return L.solver + L.batched;
}

extern "C" hisq_status hisq_multishift_cg_solve(double *const *x, const double *b, const double *shifts, int nshift,
                                                const double *tol, const hisq_gauge *g64, const hisq_gauge *g_ms,
                                                const hisq_gauge *g_ref, double mass, hisq_fmt ms_fmt,
                                                hisq_fmt refine_fmt, const hisq_solver_params *p, void *ws,
                                                size_t ws_bytes, hisq_solver_stats *stats, void *stream) {
    auto t0 = std::chrono::steady_clock::now();
    hisq_solver_stats tmp;
    hisq_solver_stats *st = stats ? stats : &tmp;
    memset(st, 0, sizeof(*st));
    st->status = HISQ_EINVAL;
    if (!x || !b || !shifts || !tol || !g64 || !g_ms || !g_ref || !ws)
        return set_error(HISQ_EINVAL, "hisq_multishift_cg_solve: null argument");
    if (nshift < 1 || nshift > HISQ_MAX_SHIFTS)
        return set_error(HISQ_EINVAL, "nshift must be in [1,%d]", HISQ_MAX_SHIFTS);
    for (int i = 0; i < nshift; i++) {
        if (!x[i] || !aligned16(x[i])) return set_error(HISQ_EALIGN, "x[%d] null or unaligned", i);
        if (!(tol[i] > 0.0)) return set_error(HISQ_EINVAL, "tol[%d] must be > 0", i);
        if (i == 0 && !(shifts[0] >= 0.0)) return set_error(HISQ_EINVAL, "shifts[0] must be >= 0");
        if (i > 0 && !(shifts[i] > shifts[i - 1])) return set_error(HISQ_EINVAL, "shifts must be strictly ascending");
    }
    if (!aligned16(b) || !aligned16(ws)) return set_error(HISQ_EALIGN, "unaligned pointer");
    if (!triplet_ok(ms_fmt) || !triplet_ok(refine_fmt)) return set_error(HISQ_EINVAL, "unsupported triplet");
    const int *dims = g64->dims;
    if (!dims_ok(dims)) return set_error(HISQ_EINVAL, "bad lattice dims");
    HISQ_TRY(check_gauge(g64, dims, hisq_fmt{HISQ_GAUGE_F64, HISQ_SPINOR_F64, 64}, "g64"));
    HISQ_TRY(check_gauge(g_ms, dims, ms_fmt, "g_ms"));
    HISQ_TRY(check_gauge(g_ref, dims, refine_fmt, "g_ref"));
    hisq_solver_params q;
    HISQ_TRY(check_params(p, &q));
    const Geom g = make_geom(dims);
    const int bs = std::max(spinor_site_bytes(ms_fmt.spinor), spinor_site_bytes(refine_fmt.spinor));
    MsLayout L = ms_layout(g, nshift, ms_fmt, refine_fmt, q);
    // eight-parameter long links have no batched Dslash: shifts refined one after another
    L.batch = L.batch && g_ref->long_recon != HISQ_RECON_8;
    if (ws_bytes < L.solver + L.batched)
        return set_error(HISQ_EWORKSPACE, "workspace %zu bytes, need %zu", ws_bytes, L.solver + L.batched);
    CgBuffers B;
    carve_cg(&B, (char *)ws, g, bs, q.grad_buffer, nshift, spinor_site_bytes(ms_fmt.spinor),
             spinor_site_bytes(refine_fmt.spinor));
    Entry E;
    HISQ_TRY(E.begin(stream));
    hipStream_t s_ = E.ds->stream;
    SolverCtrl *h = &E.ds->host->ctrl;
    st->nshift = nshift;
    hisq_status status = HISQ_OK;
    const double m2 = 4.0 * mass * mass;

    // ---- multi-shift phase (ms_fmt), base = shift 0 ----
    HISQ_TRY_HIP(launch_spinor_pack(B.b64, b, g.vh, SF_F64, s_));
    HISQ_TRY_HIP(hipMemsetAsync(B.x64, 0, 48 * (size_t)g.vh, s_));
    for (int i = 1; i < nshift; i++) HISQ_TRY_HIP(hipMemsetAsync(B.xs[i], 0, 48 * (size_t)g.vh, s_));
    double rho_ms = 0.0;
    int base_slot = 0;
    {
        Run R;
        R.g = g;
        R.vh = g.vh;
        R.fmt = ms_fmt;
        R.g64 = g64;
        R.gs = g_ms;
        R.c_ = m2 + shifts[0];
        R.nb = q.grad_buffer;
        solver_unit(q, &R.unit, &R.depth);
        R.maxiter = q.maxiter;
        R.graph = q.use_graph != 0;
        R.multishift = nshift > 1;
        R.ru_est = q.ru_estimate != 0;
        R.nshift = nshift;
        R.B = &B;
        R.st = s_;
        R.h = E.ds->host;
        init_ctrl(R.h, q, tol[0], 0.0, ms_fmt.spinor);
        h->nshift = nshift;
        // where a shifted system's iterated residual stops tracking its true
        // residual: with FP32 arithmetic near the storage format's epsilon;
        // with FP64 arithmetic (INT30 or SX24/INT30 storage included) below
        // any tolerance the FP64 reliable updates certify, so only tol_i stops it
        const double fl = q.shift_floor > 0     ? q.shift_floor
                          : ms_fmt.compute == 64 ? 0.0
                                                 : std::ldexp(1.0, -sloppy_floor_bits(ms_fmt.spinor));
        h->floor2 = fl * fl;
        h->active_mask = 0;
        for (int i = 0; i < nshift; i++) {
            h->sh[i] = shifts[i] - shifts[0];
            h->tol2_i[i] = tol[i] * tol[i];
            h->zeta[i] = h->zeta_prev[i] = 1.0;
            h->active_mask |= 1 << i;
        }
        HISQ_TRY_HIP(hipMemcpyAsync(B.ctrl, h, sizeof(SolverCtrl), hipMemcpyHostToDevice, s_));
        R.setup_plans();
        HISQ_TRY(enq_b2(R));
        HISQ_TRY(R.enq_reliable(1, 0, nullptr));  // x = 0: r = b, p_0 = r
        // every shifted gradient vector starts as p_i = b (stored in the sloppy format)
        for (int i = 1; i < nshift; i++)
            HISQ_TRY_HIP(launch_spinor_convert(B.ps[i], ms_fmt.spinor, B.rs, ms_fmt.spinor, g.vh, s_));
        HISQ_TRY(R.read_status());
        if (R.last.b2 == 0.0) {
            for (int i = 0; i < nshift; i++) HISQ_TRY_HIP(hipMemsetAsync(x[i], 0, 48 * (size_t)g.vh, s_));
            HISQ_TRY(E.end());
            st->status = HISQ_OK;
            return HISQ_OK;
        }
        int ms_done = 0;
        if (!R.last.done) {
            // one shift: plain CG with reliable updates in the multi-shift triplet
            status = R.iterate(&ms_done);
            if (status == HISQ_ENOCONV) status = HISQ_OK;  // the refinement continues from here
        }
        const hisq_status sr = R.read_ctrl();   // the shifts' stop iterations and the base's |r|^2
        if (status == HISQ_OK) status = sr;
        fill_common_stats(st, R);
        for (int i = 1; i < nshift; i++) st->shift_iters[i] = h->shift_stop_k[i] ? h->shift_stop_k[i] : h->k;
        st->shift_iters[0] = h->k;
        rho_ms = h->rho_prev;  // |r_k|^2 of the gradient vector p_k carried into the refinement
        st->phase_seconds[0] = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        base_slot = R.last_slot;
        if (status != HISQ_OK) {
            (void)E.end();
            st->status = status;
            return status;
        }
    }

    // ---- refinement (refine_fmt): the base keeps its gradient vector, every shift
    // restarts from its multi-shift solution.  The base first, then the shifts in
    // ascending order or together as a batch; with batch_refine == 2 the batch
    // runs on the second stream while a host thread refines the base on the
    // first (the two are independent once the multi-shift phase is over; every
    // launch shape either uses is planned before they overlap). ----
    auto t1 = std::chrono::steady_clock::now();
    struct Refined {
        hisq_status status = HISQ_OK;
        double r0 = 0.0, r1 = 0.0, seconds = 0.0;
        std::string msg;   // the error message (set in the thread that ran it)
        Run R;
    };
    // refinement run of system i on stream sr with host control block hc
    auto setup_run = [&](Run &R, CgBuffers &Bi, int i, hipStream_t sr, SolverHost *hc) {
        R.g = g;
        R.vh = g.vh;
        R.fmt = refine_fmt;
        R.g64 = g64;
        R.gs = g_ref;
        R.c_ = m2 + shifts[i];
        R.nb = q.grad_buffer;
        solver_unit(q, &R.unit, &R.depth);
        R.maxiter = q.maxiter;
        R.graph = q.use_graph != 0;
        R.multishift = false;
        R.ru_est = q.ru_estimate != 0;
        R.nshift = 1;
        Bi = B;
        if (i > 0) Bi.x64 = B.xs[i];
        R.B = &Bi;
        R.st = sr;
        R.h = hc;
    };
    auto refine_one = [&](int i, Refined &out, SolverHost *hc) {
        auto ts = std::chrono::steady_clock::now();
        CgBuffers Bi;
        setup_run(out.R, Bi, i, s_, hc);
        if (i == 0 && nshift > 1)
            out.status = cg_core(out.R, q, tol[0], 2, B.pconv, rho_ms, &out.r0);
        else
            out.status = cg_core(out.R, q, tol[i], 1, nullptr, 0.0, &out.r0);
        out.r1 = out.R.last.b2 > 0 ? std::sqrt(out.R.last.r2_true / out.R.last.b2) : 0.0;
        hipError_t e = launch_spinor_unpack(x[i], Bi.x64, g.vh, SF_F64, s_);
        if (e == hipSuccess) e = hipStreamSynchronize(s_);
        if (e != hipSuccess && out.status == HISQ_OK)
            out.status = set_error(HISQ_EHIP, "refinement of system %d: %s", i, hipGetErrorString(e));
        if (out.status != HISQ_OK) out.msg = hisq_last_error();
        out.seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - ts).count();
    };
    auto account = [&](int i, const Refined &o) {
        st->shift_resid_ms[i] = o.r0;
        st->refine_iters[i] = (int)o.R.iters;
        st->shift_resid[i] = o.r1;
        st->reliable_updates += (int)o.R.rus;
        st->dslash_sloppy += (int)o.R.dslash_sloppy;
        st->dslash_f64 += (int)o.R.dslash_f64;
        st->alg_bytes += o.R.alg_bytes;
    };
    if (nshift > 1 && status == HISQ_OK)
        HISQ_TRY_HIP(launch_spinor_convert(B.pconv, refine_fmt.spinor, B.p[base_slot], ms_fmt.spinor, g.vh, s_));
    const bool overlap = L.batch && nshift > 1 && q.batch_refine == 2;
    const bool joint = L.batch && nshift > 1 && q.batch_refine == 3;
    // one batched block of the systems [i0, i0 + n): the base (i0 == 0) continues its gradient vector
    auto run_block = [&](int i0, int n, hipStream_t sr, SolverHost *hc, BatchedJob &J) {
        memset(&J, 0, sizeof(J));
        J.nrhs = n;
        for (int j = 0; j < n; j++) {
            J.x[j] = x[i0 + j];
            J.b[j] = b;
            J.c[j] = m2 + shifts[i0 + j];
            J.tol[j] = tol[i0 + j];
        }
        J.g64 = g64;
        J.gs = g_ref;
        J.fmt = refine_fmt;
        J.q = q;
        J.ws = (char *)ws + L.solver;
        J.ws_bytes = L.batched;
        J.st = sr;
        J.h = hc;
        if (i0 == 0) {
            J.p_warm = B.pconv;
            J.rho_warm = rho_ms;
        }
    };
    auto account_block = [&](int i0, const BatchedJob &J) {
        for (int j = 0; j < J.nrhs; j++) {
            st->shift_resid_ms[i0 + j] = J.resid0_j[j];
            st->refine_iters[i0 + j] = J.iters_j[j];
            st->shift_resid[i0 + j] = J.resid_j[j];
        }
        st->reliable_updates += (int)J.rus;
        st->dslash_sloppy += (int)J.dsl;
        st->dslash_f64 += (int)J.d64;
        st->alg_bytes += J.alg;
    };
    if (joint) {
        // the base joins the shifts' batch as system 0 of the first block,
        // continuing its gradient vector; every system converges on its own
        if (status == HISQ_OK) HISQ_TRY_HIP(launch_spinor_unpack(x[0], B.x64, g.vh, SF_F64, s_));
        for (int i = 1; i < nshift && status == HISQ_OK; i++)
            HISQ_TRY_HIP(launch_spinor_unpack(x[i], B.xs[i], g.vh, SF_F64, s_));
        for (int i0 = 0; i0 < nshift && status == HISQ_OK; i0 += 16) {
            BatchedJob J;
            run_block(i0, std::min(16, nshift - i0), s_, E.ds->host, J);
            status = batched_run(J);
            account_block(i0, J);
        }
        st->phase_seconds[1] = 0.0;
    } else if (!overlap) {
        // the base, then the shifts: one after another, or together as a batch
        for (int i = 0; i < (L.batch ? 1 : nshift) && status == HISQ_OK; i++) {
            Refined o;
            refine_one(i, o, E.ds->host);
            status = o.status;
            account(i, o);
            if (i == 0) {
                t1 = std::chrono::steady_clock::now();
                st->phase_seconds[1] = o.seconds;
            }
        }
        if (L.batch && status == HISQ_OK) {
            for (int i = 1; i < nshift; i++) HISQ_TRY_HIP(launch_spinor_unpack(x[i], B.xs[i], g.vh, SF_F64, s_));
            for (int i0 = 1; i0 < nshift && status == HISQ_OK; i0 += 16) {
                BatchedJob J;
                run_block(i0, std::min(16, nshift - i0), s_, E.ds->host, J);
                status = batched_run(J);
                account_block(i0, J);
            }
        }
    } else if (status == HISQ_OK) {
        // the multi-shift solutions are the shifted systems' initial guesses
        for (int i = 1; i < nshift; i++) HISQ_TRY_HIP(launch_spinor_unpack(x[i], B.xs[i], g.vh, SF_F64, s_));
        // the base run's launch shapes, planned before anything overlaps
        {
            Run Rp;
            CgBuffers Bp;
            setup_run(Rp, Bp, 0, s_, E.ds->host);
            Rp.setup_plans();
        }
        HISQ_TRY_HIP(hipEventRecord(E.ds->ev2, s_));
        hipStream_t s2 = E.ds->stream2;
        HISQ_TRY_HIP(hipStreamWaitEvent(s2, E.ds->ev2, 0));
        Refined base;
        std::thread worker;
        struct Start {
            std::thread *w;
            std::function<void()> fn;
        } start{&worker, [&] { refine_one(0, base, E.ds->host); }};
        for (int i0 = 1; i0 < nshift && status == HISQ_OK; i0 += 16) {
            BatchedJob J;
            run_block(i0, std::min(16, nshift - i0), s2, E.ds->host2, J);
            if (!worker.joinable()) {
                // the base starts once the block's launch shapes are planned
                J.after_setup = [](void *c) {
                    Start *sp = static_cast<Start *>(c);
                    try {
                        *sp->w = std::thread(sp->fn);
                    } catch (...) {
                        // no thread: the base is refined after the batch
                    }
                };
                J.after_setup_ctx = &start;
            }
            status = batched_run(J);
            account_block(i0, J);
        }
        if (worker.joinable()) {
            worker.join();
        } else {
            refine_one(0, base, E.ds->host);   // the batched block stopped before it started the base
        }
        account(0, base);
        st->phase_seconds[1] = base.seconds;
        if (status == HISQ_OK && base.status != HISQ_OK)
            status = set_error(base.status, "base refinement: %s", base.msg.c_str());
    }
    hisq_status s2 = E.end();
    if (status == HISQ_OK) status = s2;
    st->phase_seconds[2] = std::chrono::duration<double>(std::chrono::steady_clock::now() - t1).count();
    double worst = 0.0;
    for (int i = 0; i < nshift; i++) worst = std::max(worst, st->shift_resid[i] / tol[i] * tol[0]);
    st->true_resid = worst;
    st->status = status;
    st->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return status;
}
