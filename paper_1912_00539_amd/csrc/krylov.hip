// Restarted flexible GMRES (the Krylov solver of Sections 1 and 6), right-preconditioned by the
// sweep apply, entirely in double precision on the device: Arnoldi basis V and preconditioned
// basis Z in the workspace, classical Gram-Schmidt with a second pass when the norm falls below
// 1/sqrt(2) of its value before orthogonalisation ("twice is enough"), Givens rotations on the
// Hessenberg matrix by the last workgroup of the reduction before them, x update and true residual at each
// cycle end. The host loop reads back a few scalars per iteration to decide when to stop.
//
// All reductions are fixed-order (per-workgroup partials, then one workgroup per column in
// index order), so results do not depend on scheduling. The only atomic is the completion count
// that picks the last workgroup of a reduction; it orders work, not values.
#include <chrono>
#include <cmath>
#include <cstring>

#include "kernels.h"
#include "rules.h"

using namespace abilu;
using namespace abilu_dev;
using namespace abilu_k;

namespace {

template <int VE>
__global__ __launch_bounds__(WG) void k_mdot(int64_t len, Basis V, int q,
                                             const double *__restrict__ w, double *__restrict__ partial, int nb) {
    __shared__ WaveSums sh[MAX_RESTART + 2];
    mdot_body<VE>(blockIdx.x, len, V, q, w, partial, nb, sh);
}

// The updates take the tiles in descending order: the kernel before them runs ascending, so they
// start on the tiles it read last (the partials stay indexed by tile, so sums are unchanged).
template <int VE>
__global__ __launch_bounds__(WG) void k_update(int64_t len, Basis V, int q,
                                               const double *__restrict__ c, double alpha, double *__restrict__ w,
                                               double *__restrict__ partial, const int *guard, bool fresh) {
    update_body<VE>(gridDim.x - 1 - blockIdx.x, len, V, q, c, alpha, w, partial, guard, fresh);
}

template <int QM, int VE>
__global__ __launch_bounds__(WG) void k_update_dot(int64_t len, Basis V, int q,
                                                   const double *__restrict__ c, double *__restrict__ w,
                                                   double *__restrict__ partial, int nb) {
    __shared__ WaveSums sh[MAX_RESTART + 2];
    update_dot_body<QM, VE>(gridDim.x - 1 - blockIdx.x, len, V, q, c, w, partial, nb, sh);
}

// out[col] = sum_b partial[col*nb + b], one workgroup per column, fixed order
__global__ __launch_bounds__(WG) void k_reduce_cols(const double *__restrict__ partial, int nb,
                                                    double *__restrict__ out, const int *guard) {
    reduce_cols_body(blockIdx.x, partial, nb, out, guard);
}

// k_reduce_cols followed by step OP on the column sums in the last workgroup, in one launch.
template <int OP>
__global__ __launch_bounds__(WG) void k_reduce_step(KPtrs P, int nb, const int *guard, int k, int m) {
    reduce_step_body<OP>(blockIdx.x, gridDim.x, P, nb, guard, k, m);
}

// ---- systems of at most FOLD_NB vector workgroups (all of the smaller tile): the dot and update
// kernels reduce their own partials in their last workgroup and run the step there, one launch
// instead of two, with the sums of the two-launch form bit for bit. Beyond FOLD_NB one workgroup
// would add more than four entries per lane and column (at 4 million cells, 31). Solves of triangles to
// 1e-10, FP32, two launches / folded, us: 319 workgroups 433 / 428, 400 534 / 527, 512 576 / 579; with a limit
// of 1,024 instead, 600 638 / 651, 704 (180,000 cells) 684 / 703, 1,024 913 / 922.
constexpr int FOLD_VE = 4;
static_assert((int64_t)FOLD_NB * WG * FOLD_VE < VEC_SMALL, "folded systems have the smaller tile");

template <int OP>
__device__ __forceinline__ void fold_tail(const KPtrs &P, const StepIn &in, int nb, int cols, const int *guard, int k,
                                          int m) {
    __shared__ double sred[MAX_RESTART + 2];
    if (!last_workgroup<true>(P.done, gridDim.x, blockIdx.x)) return;
    if (!skipped(guard)) reduce_cols_fold(P.partials, nb, cols, sred);
    step_tail<OP>(P, in, k, m, sred);
}

template <int OP>
__global__ __launch_bounds__(WG) void k_mdot_step(int64_t len, Basis V, int q,
                                                  const double *__restrict__ w, KPtrs P, int nb, int k, int m) {
    __shared__ WaveSums sh[MAX_RESTART + 2];
    StepIn in;
    in.load<OP>(P, k, m);
    mdot_body<FOLD_VE>(blockIdx.x, len, V, q, w, P.partials, nb, sh);
    fold_tail<OP>(P, in, nb, q + 1, nullptr, k, m);
}

template <int QM>
__global__ __launch_bounds__(WG) void k_update_dot_step(int64_t len, Basis V, int q,
                                                        const double *__restrict__ c, double *__restrict__ w, KPtrs P,
                                                        int nb, int k, int m) {
    __shared__ WaveSums sh[MAX_RESTART + 2];
    StepIn in;
    in.load<RS_GS2>(P, k, m);
    update_dot_body<QM, FOLD_VE>(gridDim.x - 1 - blockIdx.x, len, V, q, c, w, P.partials, nb, sh);
    fold_tail<RS_GS2>(P, in, nb, q + 1, nullptr, k, m);
}

__global__ __launch_bounds__(WG) void k_update_step(int64_t len, Basis V, int q,
                                                    const double *__restrict__ c, double alpha, double *__restrict__ w,
                                                    KPtrs P, int nb, const int *guard, int k, int m) {
    StepIn in;
    in.load<RS_GIVENS>(P, k, m);
    update_body<FOLD_VE>(gridDim.x - 1 - blockIdx.x, len, V, q, c, alpha, w, P.partials, guard);
    fold_tail<RS_GIVENS>(P, in, nb, 1, guard, k, m);
}

__global__ __launch_bounds__(WG) void k_zero(int64_t len, double *v) {
    zero_body(blockIdx.x, len, v);
}

// ---- ILU residual: sums of ||(LU - A)_ij||^2 and ||A_ij||^2 over the pattern (factor layout)
template <typename T>
__global__ __launch_bounds__(WG) void k_ilu_residual(int n, int ZL, const int32_t *__restrict__ rowptr,
                                                     const int32_t *__restrict__ colidx,
                                                     const int32_t *__restrict__ diag_pos,
                                                     const int32_t *__restrict__ lrow, const int32_t *__restrict__ urow,
                                                     const int32_t *__restrict__ pair_ptr,
                                                     const int32_t *__restrict__ sik, const int32_t *__restrict__ skj,
                                                     const double *__restrict__ A, const T *__restrict__ X,
                                                     double *__restrict__ partial, int nb) {
    __shared__ double shn[WG / 64], shd[WG / 64];
    const int r = threadIdx.x & 3;
    double num = 0.0, den = 0.0;
    for (int pass = 0; pass < DIAG_ROWS / ROWS_PER_WG; ++pass) {
        const int i = blockIdx.x * DIAG_ROWS + pass * ROWS_PER_WG + (threadIdx.x >> 2);
        if (i < n) {
            const int b0 = rowptr[i], b1 = rowptr[i + 1], d = diag_pos[i];
            for (int e = b0; e < b1; ++e) {
                const int j = colidx[e];
                double x[4], P[4];
                load_row(X + (int64_t)split_pos(e, i, b0, d, lrow[i], urow[i], ZL, n) * BB, r, x);
                if (i > j) {
                    double u[4];
                    load_row(X + ((int64_t)ZL + j) * BB, r, u);
                    row_times_block(x, u, P);
                } else {
#pragma unroll
                    for (int c = 0; c < 4; ++c) P[c] = x[c];
                }
                for (int q = pair_ptr[e]; q < pair_ptr[e + 1]; ++q) {
                    double l[4], u[4], t[4];
                    load_row(X + (int64_t)sik[q] * BB, r, l);
                    load_row(X + (int64_t)skj[q] * BB, r, u);
                    row_times_block(l, u, t);
#pragma unroll
                    for (int c = 0; c < 4; ++c) P[c] += t[c];
                }
                double a[4];
                load_row(A + (int64_t)e * BB, r, a);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    num += (P[c] - a[c]) * (P[c] - a[c]);
                    den += a[c] * a[c];
                }
            }
        }
    }
    num = wave_sum(num);
    den = wave_sum(den);
    if ((threadIdx.x & 63) == 0) {
        shn[threadIdx.x >> 6] = num;
        shd[threadIdx.x >> 6] = den;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        partial[blockIdx.x] = (shn[0] + shn[1]) + (shn[2] + shn[3]);
        partial[nb + blockIdx.x] = (shd[0] + shd[1]) + (shd[2] + shd[3]);
    }
}

struct Ctx {
    const abilu_pattern *p;
    Workspace W;
    char *work;
    hipStream_t s;
    int64_t nv;
    double *partials, *H, *cs, *sn, *g, *coef, *misc, *status, *vscale, *red, *V, *Zb;
    const double *v0;   // the first basis vector: the right-hand side or V
    int *guard, *done;
    int m;
    double rtol;
    unsigned long long *slot = nullptr, *slot_dev = nullptr;   // where the next status goes, host and device
    unsigned turn = 0;
    bool last = false;
    void ask() {   // the launch that follows publishes a status
        const unsigned at = PIN_BASE + PIN_WORDS * (turn++ % PIN_SLOTS);
        slot = (unsigned long long *)p->pinned + at;
        slot_dev = (unsigned long long *)p->pinned_dev + at;
        for (int w = 0; w < PIN_WORDS; ++w) __atomic_store_n(slot + w, PIN_EMPTY, __ATOMIC_RELAXED);
        __atomic_thread_fence(__ATOMIC_RELEASE);
    }
    Basis basis() const { return Basis{v0, V, nv}; }
    KPtrs ptrs() const { return KPtrs{partials, red, H, cs, sn, g, coef, misc, status, vscale, guard, done, true, slot_dev,
                     (const unsigned *)work, rtol, true, last}; }
};

#define CKL()                                                     \
    do {                                                          \
        if (launch_status() != ABILU_OK) return ABILU_EDEVICE;    \
    } while (0)

// Column sums of the partials into c.red (ncols columns), then step op.
abilu_status reduce_step(Ctx &c, int ncols, const int *guard, int op, int k) {
    const int nb = c.W.nb_vec;
    ProfScope ps("fgmres_reduce", c.s, 8.0 * ncols * nb);
    const KPtrs P = c.ptrs();
    switch (op) {
        case RS_BETA_START_ZERO: k_reduce_step<RS_BETA_START_ZERO><<<ncols, WG, 0, c.s>>>(P, nb, guard, k, c.m); break;
        case RS_BETA_START_X: k_reduce_step<RS_BETA_START_X><<<ncols, WG, 0, c.s>>>(P, nb, guard, k, c.m); break;
        case RS_BETA: k_reduce_step<RS_BETA><<<ncols, WG, 0, c.s>>>(P, nb, guard, k, c.m); break;
        case RS_GS1: k_reduce_step<RS_GS1><<<ncols, WG, 0, c.s>>>(P, nb, guard, k, c.m); break;
        case RS_GS2: k_reduce_step<RS_GS2><<<ncols, WG, 0, c.s>>>(P, nb, guard, k, c.m); break;
        default: k_reduce_step<RS_GIVENS><<<ncols, WG, 0, c.s>>>(P, nb, guard, k, c.m); break;
    }
    CKL();
    return ABILU_OK;
}

// c.red[0..q] <- dots of w with V_0..V_{q-1}, then ||w||^2; then step op
abilu_status mdot_reduce(Ctx &c, int q, const double *w, int op, int k) {
    const int nb = c.W.nb_vec;
    const double n8 = 8.0 * (double)c.nv;
    if (nb <= FOLD_NB) {
        ProfScope ps("fgmres_mdot", c.s, (q + 1) * n8 + 8.0 * (q + 1) * nb);
        const KPtrs P = c.ptrs();
#define ABILU_MDOT_STEP(OP) \
    case OP: k_mdot_step<OP><<<nb, WG, 0, c.s>>>(c.nv, c.basis(), q, w, P, nb, k, c.m); break
        switch (op) {
            ABILU_MDOT_STEP(RS_BETA_START_ZERO);
            ABILU_MDOT_STEP(RS_BETA_START_X);
            ABILU_MDOT_STEP(RS_BETA);
            ABILU_MDOT_STEP(RS_GS1);
        }
#undef ABILU_MDOT_STEP
        CKL();
        return ABILU_OK;
    }
    {
        ProfScope ps("fgmres_mdot", c.s, (q + 1) * n8);
        if (vec_e(c.nv) == 4) k_mdot<4><<<nb, WG, 0, c.s>>>(c.nv, c.basis(), q, w, c.partials, nb);
        else k_mdot<8><<<nb, WG, 0, c.s>>>(c.nv, c.basis(), q, w, c.partials, nb);
    }
    CKL();
    return reduce_step(c, q + 1, nullptr, op, k);
}

// first Gram-Schmidt update of w against V_0..V_{q-1} with the second pass's dots, then the
// decision on that pass
abilu_status update_dot_reduce(Ctx &c, int q, double *w, int k) {
    const int nb = c.W.nb_vec;
    const bool fold = nb <= FOLD_NB;
    const double n8 = 8.0 * (double)c.nv;
    {
        ProfScope ps("fgmres_update_dot", c.s, (q + 2) * n8 + (fold ? 8.0 * (q + 1) * nb : 0.0));
        const KPtrs P = c.ptrs();
#define ABILU_UPDATE_DOT(QM)                                                                                          \
    do {                                                                                                              \
        if (fold) k_update_dot_step<QM><<<nb, WG, 0, c.s>>>(c.nv, c.basis(), q, c.coef, w, P, nb, k, c.m);            \
        else if (vec_e(c.nv) == 4)                                                                                    \
            k_update_dot<QM, 4><<<nb, WG, 0, c.s>>>(c.nv, c.basis(), q, c.coef, w, c.partials, nb);                   \
        else k_update_dot<QM, 8><<<nb, WG, 0, c.s>>>(c.nv, c.basis(), q, c.coef, w, c.partials, nb);                  \
    } while (0)
        switch (update_dot_form(q)) {
            case 4: ABILU_UPDATE_DOT(4); break;
            case 8: ABILU_UPDATE_DOT(8); break;
            case 16: ABILU_UPDATE_DOT(16); break;
            case 32: ABILU_UPDATE_DOT(32); break;
            default: ABILU_UPDATE_DOT(0); break;
        }
#undef ABILU_UPDATE_DOT
    }
    CKL();
    return fold ? ABILU_OK : reduce_step(c, q + 1, nullptr, RS_GS2, k);
}

// w += alpha * sum_k coef[k] Vb_k; with givens: c.red[0] <- ||w||^2 afterwards, then the Givens step
abilu_status update_reduce(Ctx &c, const Basis &Vb, int q, double alpha, double *w, const int *guard, bool givens,
                           int k, bool fresh = false) {
    const int nb = c.W.nb_vec;
    const double n8 = 8.0 * (double)c.nv;
    if (givens && nb <= FOLD_NB) {
        {
            ProfScope ps("fgmres_update", c.s, (q + 2) * n8 + 8.0 * nb);
            k_update_step<<<nb, WG, 0, c.s>>>(c.nv, Vb, q, c.coef, alpha, w, c.ptrs(), nb, guard, k, c.m);
        }
        CKL();
        return ABILU_OK;
    }
    {
        ProfScope ps("fgmres_update", c.s, (q + (fresh ? 1 : 2)) * n8);
        double *part = givens ? c.partials : nullptr;
        if (vec_e(c.nv) == 4) k_update<4><<<nb, WG, 0, c.s>>>(c.nv, Vb, q, c.coef, alpha, w, part, guard, fresh);
        else k_update<8><<<nb, WG, 0, c.s>>>(c.nv, Vb, q, c.coef, alpha, w, part, guard, fresh);
    }
    CKL();
    return givens ? reduce_step(c, 1, guard, RS_GIVENS, k) : ABILU_OK;
}

struct Status {
    double v0, v1;   // est and hn, or beta and ||b||
    uint32_t flags;
    bool guard;
};

// Whether the status asked for in `slot` has arrived.
bool status_here(const unsigned long long *slot) {
    for (int w = 0; w < 3; ++w)
        if (__atomic_load_n(slot + w, __ATOMIC_ACQUIRE) == PIN_EMPTY) return false;
    return true;
}

// Waits for the status asked for in `slot` and reads it. The wait polls the pinned buffer, where the
// status is some 10 us before a stream synchronisation behind a copy would return; every
// millisecond it asks the stream whether it has failed, or has run dry without the status.
abilu_status read_status(Ctx &c, const unsigned long long *slot, Status *out) {
    using clock = std::chrono::steady_clock;
    auto next = clock::now() + std::chrono::milliseconds(1);
    for (unsigned spins = 1; !status_here(slot); ++spins) {
        __builtin_ia32_pause();
        if (spins % 256 != 0 || clock::now() < next) continue;
        const hipError_t e = hipStreamQuery(c.s);
        if (e == hipErrorNotReady) {
            (void)hipGetLastError();
            next = clock::now() + std::chrono::milliseconds(1);
            continue;
        }
        if (!hip_ok(e, "fgmres stream")) return ABILU_EDEVICE;
        if (status_here(slot)) break;
        note_error("fgmres_solve: the stream ended without a status");
        return ABILU_EDEVICE;
    }
    memcpy(&out->v0, slot, sizeof(double));
    memcpy(&out->v1, slot + 1, sizeof(double));
    out->flags = (uint32_t)slot[2];
    out->guard = ((slot[2] >> 32) & 1) != 0;
    return ABILU_OK;
}

// The status asked for last, until it is read: `decide` takes it in and says whether the solve, or the
// cycle, stops. Asked as the gate of an application begun before it, it lets at most `limit` launches pass.
enum { START, CYCLE, STEP };
template <typename Decide>
struct Pending : Gate {
    Ctx &c;
    const Decide &decide;
    Status now{};
    const unsigned long long *slot = nullptr;
    bool open = false, stop = false;
    int kind = START, launched = 0, limit = 0;
    abilu_status st = ABILU_OK;
    Pending(Ctx &ctx, const Decide &d) : c(ctx), decide(d) {}
    void expect(int k) {
        open = true;
        kind = k;
        slot = c.slot;
        launched = 0;
    }
    void read() {
        if (!open) return;
        open = false;
        st = read_status(c, slot, &now);
        stop = st != ABILU_OK || decide(kind, now);
    }
    bool go() override {
        if (open && (status_here(slot) || ++launched >= limit)) read();
        return !stop;
    }
};

// r = b - A x into V_0, beta = ||r|| into g[0] and status[ST_BETA], 1 / beta into vscale[0]. The SpMV runs
// its workgroups descending (measured slightly faster than ascending after either predecessor).
abilu_status true_residual(Ctx &c, const double *A, const double *b, const double *x) {
    abilu_status st = spmv_impl(c.p, A, x, c.V, b, true, c.s);
    if (st != ABILU_OK) return st;
    c.v0 = c.V;
    c.ask();
    return mdot_reduce(c, 0, c.V, RS_BETA, 0);
}

}  // namespace

extern "C" abilu_status fgmres_solve(const abilu_pattern *p, const double *d_A, const double *d_b, double *d_x,
                                     int32_t restart, int32_t maxit, double rtol, const void *d_LU,
                                     const void *d_Dinv, abilu_prec prec, int32_t apply_sweeps, abilu_mode mode,
                                     uint32_t options, void *d_work, size_t work_bytes, void *stream,
                                     abilu_fgmres_result *out) {
    if (!p || !out || !d_work) return ABILU_EINVAL;
    if (restart < 1 || restart > MAX_RESTART || maxit < 0 || !(rtol >= 0.0) || apply_sweeps < 0) return ABILU_EINVAL;
    if (prec != ABILU_F32 && prec != ABILU_F64) return ABILU_EINVAL;
    if (!mode_ok(p, mode)) return ABILU_EINVAL;
    *out = abilu_fgmres_result{0, 0, 0, 0u, 0, 0.0, 0.0};
    Ctx c;
    c.p = p;
    c.W = layout(p, prec, restart);
    if (work_bytes < c.W.total) return ABILU_EINVAL;
    if (p->n == 0) {
        out->converged = 1;
        return ABILU_OK;
    }
    if (!d_A || !d_b || !d_x) return ABILU_EINVAL;
    if (apply_sweeps > 0 && (!d_LU || !d_Dinv)) return ABILU_EINVAL;
    c.work = (char *)d_work;
    c.s = (hipStream_t)stream;
    c.nv = 4 * (int64_t)p->n;
    const int m = restart;
    c.partials = (double *)(c.work + c.W.partials);
    c.H = (double *)(c.work + c.W.hess);
    c.cs = (double *)(c.work + c.W.cs);
    c.sn = (double *)(c.work + c.W.sn);
    c.g = (double *)(c.work + c.W.g);
    c.coef = (double *)(c.work + c.W.coef);
    c.misc = (double *)(c.work + c.W.misc);
    c.status = (double *)(c.work + c.W.status);
    c.vscale = (double *)(c.work + c.W.vscale);
    c.red = (double *)(c.work + c.W.red);
    c.V = (double *)(c.work + c.W.V);
    c.Zb = (double *)(c.work + c.W.Z);
    c.guard = (int *)(c.misc + MI_GUARD);
    c.done = p->done;
    c.m = m;
    c.rtol = rtol;
    // the solve waits for its own launches: it cannot be recorded into a graph
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (!hip_ok(hipStreamIsCapturing(c.s, &capturing), "fgmres capture status")) return ABILU_EDEVICE;
    if (capturing != hipStreamCaptureStatusNone) {
        note_error("fgmres_solve: the stream is being captured");
        return ABILU_EDEVICE;
    }
    abilu_status st;

    // ||b|| and the initial residual: b itself for a zero initial guess, which then also is the
    // first basis vector, and whose x is first written by the first cycle's update
    const bool zero_guess = (options & ABILU_FGMRES_ZERO_GUESS) != 0;
    c.v0 = d_b;
    if (zero_guess) c.ask();
    if ((st = mdot_reduce(c, 0, d_b, zero_guess ? RS_BETA_START_ZERO : RS_BETA_START_X, 0)) != ABILU_OK) return st;
    if (!zero_guess && (st = true_residual(c, d_A, d_b, d_x)) != ABILU_OK) return st;

    double bn = 1.0, tol = 0.0, beta = 0.0, est = 0.0;
    int iters = 0, restarts = 0, reorth = 0;
    bool converged = false, nonfinite = false;
    // The status of the launches so far (the start's, a cycle's or an Arnoldi step's), not yet read.
    // An Arnoldi step's application may begin before: it stops at the first launch after which the
    // status says that it is not needed, and has then written scratch vectors only (or a z_k that
    // nothing reads). Ahead of the status at most `limit` kernels are launched.
    int pass2_begin = 0, pass2_end = 0;
    const auto decide = [&](int kind, const Status &now) {   // takes the status in; true: stop
        if (kind == STEP) {
            if (now.guard)
                ++reorth;
            else
                prof_cancel_bytes(pass2_begin, pass2_end);   // the second pass exited at once
            ++iters;
            est = now.v0;
            nonfinite = !std::isfinite(est) || !std::isfinite(now.v1);
            return nonfinite || est <= tol || now.v1 == 0.0;
        }
        beta = now.v0;
        if (kind == START) {
            const double bnorm = now.v1;
            bn = bnorm > 0 ? bnorm : 1.0;
            tol = rtol * bn;
            est = beta;
            nonfinite = !std::isfinite(bnorm);
        } else {
            ++restarts;
        }
        nonfinite = nonfinite || !std::isfinite(beta);
        converged = beta <= tol;
        return converged || nonfinite || iters >= maxit || !(beta > 0.0);
    };
    Pending<decltype(decide)> pending(c, decide);
    const bool gated = (mode == ABILU_SYNC || mode == ABILU_ASYNC) && apply_sweeps >= 2;   // modes that ask the gate
    pending.limit = gated ? abilu_rules::launches_ahead(p->n, p->nnzb) : 0;
    pending.expect(START);
    if (pending.limit == 0 || maxit == 0) pending.read();

    while (!pending.stop) {
        int k = 0;   // Arnoldi steps launched in this cycle
        while (true) {
            const double *vk = k == 0 ? c.v0 : c.V + (int64_t)k * c.nv;
            double *zk = c.Zb + (int64_t)k * c.nv;
            double *w = c.V + (int64_t)(k + 1) * c.nv;
            const int apply_begin = prof_mark();
            if ((st = apply_impl(p, d_LU, d_Dinv, prec, vk, c.vscale + k, zk, apply_sweeps, mode, c.work, c.W, c.s,
                                 pending.open ? &pending : nullptr)) != ABILU_OK)
                return st;
            pending.read();
            if (pending.st != ABILU_OK) return pending.st;
            if (pending.stop) {
                prof_cancel_bytes(apply_begin, prof_mark());   // begun for nothing
                break;
            }
            if ((st = spmv_impl(p, d_A, zk, w, nullptr, !apply_ends_descending(p, prec, apply_sweeps, mode), c.s)) !=
                ABILU_OK)
                return st;
            // Gram-Schmidt pass 1: dots, H(0:k,k); the update, with the second pass's dots and the
            // decision on that pass
            if ((st = mdot_reduce(c, k + 1, w, RS_GS1, k)) != ABILU_OK) return st;
            if ((st = update_dot_reduce(c, k + 1, w, k)) != ABILU_OK) return st;
            // pass 2's update, executed by the device only when the guard is set; the Givens step
            // after it runs either way and, at the cycle's end, the least-squares solution
            c.ask();
            c.last = k + 1 == m || iters + 1 >= maxit;
            pass2_begin = prof_mark();
            if ((st = update_reduce(c, c.basis(), k + 1, -1.0, w, c.guard, true, k)) != ABILU_OK) return st;
            pass2_end = prof_mark();
            pending.expect(STEP);
            ++k;
            if (c.last || pending.limit == 0) {
                pending.read();
                if (pending.st != ABILU_OK) return pending.st;
                if (pending.stop || c.last) break;
            }
        }
        if (nonfinite || k == 0) break;
        // x += Z y
        if ((st = update_reduce(c, Basis{c.Zb, c.Zb, c.nv}, k, 1.0, d_x, nullptr, false, 0, zero_guess && restarts == 0)) !=
            ABILU_OK)
            return st;
        if ((st = true_residual(c, d_A, d_b, d_x)) != ABILU_OK) return st;
        pending.expect(CYCLE);
        pending.read();
        if (pending.st != ABILU_OK) return pending.st;
    }
    if (zero_guess && restarts == 0) {   // no cycle wrote x
        ProfScope ps("fgmres_zero", c.s, 8.0 * (double)c.nv);
        k_zero<<<c.W.nb_vec, WG, 0, c.s>>>(c.nv, d_x);
        CKL();
    }
    // the last kernel is past its status but may still be ending
    if (!hip_ok(hipStreamSynchronize(c.s), "fgmres end sync")) return ABILU_EDEVICE;
    out->iters = iters;
    out->restarts = restarts;
    out->converged = converged ? 1 : 0;
    out->flags = pending.now.flags;
    out->reorth = reorth;
    out->rel_true_residual = beta / bn;
    out->rel_estimate = est / bn;
    if (nonfinite) return ABILU_ENONFINITE;
    if (!converged) return ABILU_WARN_NOCONV;
    if (pending.now.flags & ABILU_FLAG_MODIFIED) return ABILU_WARN_MODIFIED;
    return ABILU_OK;
}

template <typename T>
static abilu_status ilu_residual_t(const abilu_pattern *p, const double *A, const T *X, char *work,
                                   const Workspace &W, double *h_rel, hipStream_t s) {
    const int nb = W.nb_diag;
    double *partial = (double *)(work + W.partials);
    double *red = (double *)(work + W.red);
    {
        ProfScope ps("ilu_residual", s);
        k_ilu_residual<T><<<nb, WG, 0, s>>>(p->n, (int)p->nnzb_lower, p->rowptr, p->colidx, p->diag_pos, p->lrow,
                                            p->urow, p->pair_ptr, p->sik, p->skj, A, X, partial, nb);
    }
    if (launch_status() != ABILU_OK) return ABILU_EDEVICE;
    k_reduce_cols<<<2, WG, 0, s>>>(partial, nb, red, nullptr);
    if (launch_status() != ABILU_OK) return ABILU_EDEVICE;
    double v[2];
    if (!hip_ok(hipMemcpyAsync(p->pinned, red, 2 * sizeof(double), hipMemcpyDeviceToHost, s), "residual readback"))
        return ABILU_EDEVICE;
    if (!hip_ok(hipStreamSynchronize(s), "residual readback sync")) return ABILU_EDEVICE;
    v[0] = p->pinned[0];
    v[1] = p->pinned[1];
    *h_rel = v[1] > 0 ? std::sqrt(v[0] / v[1]) : std::sqrt(v[0]);
    return ABILU_OK;
}

extern "C" abilu_status abilu_ilu_residual(const abilu_pattern *p, const double *d_A, const void *d_LU,
                                           abilu_prec prec, void *d_work, size_t work_bytes, double *h_rel,
                                           void *stream) {
    if (!p || !h_rel || !d_work) return ABILU_EINVAL;
    if (prec != ABILU_F32 && prec != ABILU_F64) return ABILU_EINVAL;
    const Workspace W = layout(p, prec, 0);
    if (work_bytes < W.total) return ABILU_EINVAL;
    if (p->n == 0) {
        *h_rel = 0.0;
        return ABILU_OK;
    }
    if (!d_A || !d_LU) return ABILU_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    if (prec == ABILU_F32) return ilu_residual_t<float>(p, d_A, (const float *)d_LU, (char *)d_work, W, h_rel, s);
    return ilu_residual_t<double>(p, d_A, (const double *)d_LU, (char *)d_work, W, h_rel, s);
}
