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
#include <cmath>

#include "kernels.h"

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
// would add more than four entries per lane and column (at 4 million cells, 31).
constexpr int FOLD_VE = 4;
static_assert((int64_t)FOLD_NB * WG * FOLD_VE < VEC_SMALL, "folded systems have the smaller tile");

template <int OP>
__device__ __forceinline__ void fold_tail(const KPtrs &P, int nb, int cols, const int *guard, int k, int m) {
    __shared__ double sred[MAX_RESTART + 2];
    if (!last_workgroup<true>(P.done, gridDim.x, blockIdx.x)) return;
    if (!skipped(guard)) reduce_cols_fold(P.partials, nb, cols, sred);
    step_tail<OP>(P, k, m, sred);
}

template <int OP>
__global__ __launch_bounds__(WG) void k_mdot_step(int64_t len, Basis V, int q,
                                                  const double *__restrict__ w, KPtrs P, int nb, int k, int m) {
    __shared__ WaveSums sh[MAX_RESTART + 2];
    mdot_body<FOLD_VE>(blockIdx.x, len, V, q, w, P.partials, nb, sh);
    fold_tail<OP>(P, nb, q + 1, nullptr, k, m);
}

template <int QM>
__global__ __launch_bounds__(WG) void k_update_dot_step(int64_t len, Basis V, int q,
                                                        const double *__restrict__ c, double *__restrict__ w, KPtrs P,
                                                        int nb, int k, int m) {
    __shared__ WaveSums sh[MAX_RESTART + 2];
    update_dot_body<QM, FOLD_VE>(gridDim.x - 1 - blockIdx.x, len, V, q, c, w, P.partials, nb, sh);
    fold_tail<RS_GS2>(P, nb, q + 1, nullptr, k, m);
}

__global__ __launch_bounds__(WG) void k_update_step(int64_t len, Basis V, int q,
                                                    const double *__restrict__ c, double alpha, double *__restrict__ w,
                                                    KPtrs P, int nb, const int *guard, int k, int m) {
    update_body<FOLD_VE>(gridDim.x - 1 - blockIdx.x, len, V, q, c, alpha, w, P.partials, guard);
    fold_tail<RS_GIVENS>(P, nb, 1, guard, k, m);
}

// Back substitution on the k x k upper triangle: coef = y.
__global__ __launch_bounds__(64) void k_solve(int k, int m, const double *__restrict__ H, const double *__restrict__ g,
                                              double *coef) {
    solve_body(k, m, H, g, coef);
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
    Basis basis() const { return Basis{v0, V, nv}; }
    KPtrs ptrs() const { return KPtrs{partials, red, H, cs, sn, g, coef, misc, status, vscale, guard, done, true}; }
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
    if (nb <= FOLD_NB && op != RS_BETA_START_ZERO && op != RS_BETA_START_X) {
        ProfScope ps("fgmres_mdot", c.s, (q + 1) * n8 + 8.0 * (q + 1) * nb);
        const KPtrs P = c.ptrs();
        if (op == RS_BETA) k_mdot_step<RS_BETA><<<nb, WG, 0, c.s>>>(c.nv, c.basis(), q, w, P, nb, k, c.m);
        else k_mdot_step<RS_GS1><<<nb, WG, 0, c.s>>>(c.nv, c.basis(), q, w, P, nb, k, c.m);
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

// copies the flag word and the status scalars to the host
abilu_status readback(Ctx &c, double *h, uint32_t *flags) {
    if (!hip_ok(hipMemcpyAsync(c.p->pinned, c.work, 128, hipMemcpyDeviceToHost, c.s), "fgmres readback"))
        return ABILU_EDEVICE;
    if (!hip_ok(hipStreamSynchronize(c.s), "fgmres readback sync")) return ABILU_EDEVICE;
    *flags = *(const uint32_t *)c.p->pinned;
    for (int q = 0; q < 8; ++q) h[q] = c.p->pinned[8 + q];
    return ABILU_OK;
}

// r = b - A x into V_0, beta = ||r|| into g[0] and status[ST_BETA], 1 / beta into vscale[0]. The SpMV runs
// its workgroups descending (measured slightly faster than ascending after either predecessor).
abilu_status true_residual(Ctx &c, const double *A, const double *b, const double *x) {
    abilu_status st = spmv_impl(c.p, A, x, c.V, b, true, c.s);
    if (st != ABILU_OK) return st;
    c.v0 = c.V;
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
    c.done = (int *)(c.work + c.W.done);
    c.m = m;
    double h[8];
    uint32_t flags = 0;
    abilu_status st;

    // ||b|| and the initial residual: b itself for a zero initial guess, which then also is the
    // first basis vector, and whose x is first written by the first cycle's update
    const bool zero_guess = (options & ABILU_FGMRES_ZERO_GUESS) != 0;
    c.v0 = d_b;
    if ((st = mdot_reduce(c, 0, d_b, zero_guess ? RS_BETA_START_ZERO : RS_BETA_START_X, 0)) != ABILU_OK) return st;
    if (!zero_guess && (st = true_residual(c, d_A, d_b, d_x)) != ABILU_OK) return st;
    if ((st = readback(c, h, &flags)) != ABILU_OK) return st;
    const double bnorm = h[ST_NUM];
    const double bn = bnorm > 0 ? bnorm : 1.0;
    const double tol = rtol * bn;
    double beta = h[ST_BETA], est = beta;
    int iters = 0, restarts = 0, reorth = 0;
    bool converged = beta <= tol;
    bool nonfinite = !std::isfinite(beta) || !std::isfinite(bnorm);

    while (!converged && !nonfinite && iters < maxit && beta > 0.0) {
        int k = 0;
        while (k < m && iters < maxit) {
            const double *vk = k == 0 ? c.v0 : c.V + (int64_t)k * c.nv;
            double *zk = c.Zb + (int64_t)k * c.nv;
            double *w = c.V + (int64_t)(k + 1) * c.nv;
            if ((st = apply_impl(p, d_LU, d_Dinv, prec, vk, c.vscale + k, zk, apply_sweeps, mode, c.work, c.W,
                                 c.s)) != ABILU_OK)
                return st;
            if ((st = spmv_impl(p, d_A, zk, w, nullptr, !apply_ends_descending(apply_sweeps, mode), c.s)) !=
                ABILU_OK)
                return st;
            // Gram-Schmidt pass 1: dots, H(0:k,k); the update, with the second pass's dots and the
            // decision on that pass
            if ((st = mdot_reduce(c, k + 1, w, RS_GS1, k)) != ABILU_OK) return st;
            if ((st = update_dot_reduce(c, k + 1, w, k)) != ABILU_OK) return st;
            // pass 2's update, executed by the device only when the guard is set; the Givens step
            // after it runs either way
            const int pass2_begin = prof_mark();
            if ((st = update_reduce(c, c.basis(), k + 1, -1.0, w, c.guard, true, k)) != ABILU_OK) return st;
            const int pass2_end = prof_mark();
            if ((st = readback(c, h, &flags)) != ABILU_OK) return st;
            if (h[ST_GUARD] != 0.0)
                ++reorth;
            else
                prof_cancel_bytes(pass2_begin, pass2_end);   // the second pass exited at once
            ++iters;
            ++k;
            est = h[ST_EST];
            if (!std::isfinite(est) || !std::isfinite(h[ST_HN])) {
                nonfinite = true;
                break;
            }
            if (est <= tol || h[ST_HN] == 0.0) break;
        }
        if (nonfinite) break;
        // least squares and x += Z y
        {
            ProfScope ps("fgmres_small", c.s);
            k_solve<<<1, 64, 0, c.s>>>(k, m, c.H, c.g, c.coef);
        }
        CKL();
        if ((st = update_reduce(c, Basis{c.Zb, c.Zb, c.nv}, k, 1.0, d_x, nullptr, false, 0, zero_guess && restarts == 0)) !=
            ABILU_OK)
            return st;
        if ((st = true_residual(c, d_A, d_b, d_x)) != ABILU_OK) return st;
        if ((st = readback(c, h, &flags)) != ABILU_OK) return st;
        ++restarts;
        beta = h[ST_BETA];
        if (!std::isfinite(beta)) nonfinite = true;
        converged = beta <= tol;
    }
    if (zero_guess && restarts == 0) {   // no cycle wrote x
        ProfScope ps("fgmres_zero", c.s, 8.0 * (double)c.nv);
        k_zero<<<c.W.nb_vec, WG, 0, c.s>>>(c.nv, d_x);
        CKL();
        if (!hip_ok(hipStreamSynchronize(c.s), "fgmres x sync")) return ABILU_EDEVICE;
    }
    out->iters = iters;
    out->restarts = restarts;
    out->converged = converged ? 1 : 0;
    out->flags = flags;
    out->reorth = reorth;
    out->rel_true_residual = beta / bn;
    out->rel_estimate = est / bn;
    if (nonfinite) return ABILU_ENONFINITE;
    if (!converged) return ABILU_WARN_NOCONV;
    if (flags & ABILU_FLAG_MODIFIED) return ABILU_WARN_MODIFIED;
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
