// The l2 side of a move: change of the squared l2 norm of the residual for every candidate, and the
// arg-min that uses it as second criterion (options.l2_rule).
//
// Paper: section "GPU Acceleration" evaluates the l-infinity and the l2 change of the candidates
// together before the tensor-wide argmin; the quantisation use case checks that the l2 norm does
// not increase (section "Experiment setup and results").  For the move x_j -> D[k] with step delta
// the new residual is r + delta a_j (Appendix A with one basis vector), so
//     dq(j, k) = ||r + delta a_j||^2 - ||r||^2 = 2 delta (a_j . r) + delta^2 ||a_j||^2 .
// Arithmetic contract (what makes the second criterion reproducible bit for bit):
//     g_j = a_j . r   : acc = 0; over the stored entries of column j by ascending row:
//                       acc = fma(A_ij, r_i, acc)
//     c_j = ||a_j||^2 : the same chain with fma(A_ij, A_ij, acc)      (once, at create)
//     dq(j, k)        = delta * fma(delta, c_j, 2 g_j)
// For a batch g is the matrix G = X^T R_mat (n x R), a dense contraction: on fp32 batches it runs on
// the matrix cores in the form that keeps the chain (dmmv_batched_chain.hip), so G carries the same
// bits as the chain on the vector unit.
#include "dmmv_common.h"
#include "dmmv_sparse_common.h"

namespace dmmv {

namespace {

// ---- column sums of squares, once per handle ------------------------------------------------
template <class T>
__global__ void k_l2_colsq_dense(int64_t m, int64_t n, const T* __restrict__ A, int64_t lda, T* __restrict__ csq) {
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= n) return;
    const T* __restrict__ col = A + lda * j;
    T acc = (T)0;
    for (int64_t i = 0; i < m; ++i) acc = dmmv_fma(col[i], col[i], acc);
    csq[j] = acc;
}

// sparse: the segments of a column in ascending partition hold its entries by ascending row; a
// pad has value 0 and adds nothing to either chain
template <class T>
__global__ void k_l2_sums_csc(int64_t m, int64_t n, int32_t mp, int32_t P, const int32_t* __restrict__ segptr,
                              const uint16_t* __restrict__ row16, const T* __restrict__ cval,
                              const T* __restrict__ r, T* __restrict__ g, T* __restrict__ csq) {
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= n) return;
    T acc = (T)0, sq = (T)0;
    for (int32_t p = 0; p < P; ++p) {
        const int32_t e0 = segptr[(int64_t)p * n + j], e1 = segptr[(int64_t)p * n + j + 1];
        for (int32_t e = e0; e < e1; ++e) {
            const uint32_t loc = row16[e];
            if (loc == (uint32_t)mp) continue;
            const T a = cval[e];
            if (g) acc = dmmv_fma(a, r[(int64_t)p * mp + loc], acc);
            if (csq) sq = dmmv_fma(a, a, sq);
        }
    }
    if (g) g[j] = acc;
    if (csq) csq[j] = sq;
}

// ---- g = A^T r -------------------------------------------------------------------------------
template <class T>
__global__ void k_l2_g_dense(int64_t m, int64_t n, const T* __restrict__ A, int64_t lda, const T* __restrict__ r,
                             T* __restrict__ g) {
    const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (j >= n) return;
    const T* __restrict__ col = A + lda * j;
    T acc = (T)0;
    for (int64_t i = 0; i < m; ++i) acc = dmmv_fma(col[i], r[i], acc);
    g[j] = acc;
}

// Batch, vector unit: lane = instance, TJ columns per lane and pass; r is read coalesced over the
// instances, the row of X is the same for every lane (row-major copy, read through the scalar unit).
template <class T, int TJ>
__global__ __launch_bounds__(256) void k_l2_g_batched(int64_t m, int64_t n, int64_t R, const T* __restrict__ Xt,
                                                      const T* __restrict__ r, T* __restrict__ G) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t j0 = blockIdx.y * (int64_t)TJ;
    const int64_t qc = q < R ? q : R - 1;
    T acc[TJ];
#pragma unroll
    for (int u = 0; u < TJ; ++u) acc[u] = (T)0;
    for (int64_t i = 0; i < m; ++i) {
        const T ri = r[i * R + qc];
        const T* __restrict__ xr = Xt + i * n;
#pragma unroll
        for (int u = 0; u < TJ; ++u) {
            const int64_t j = j0 + u < n ? j0 + u : n - 1;
            acc[u] = dmmv_fma(xr[j], ri, acc[u]);
        }
    }
    if (q < R) {
#pragma unroll
        for (int u = 0; u < TJ; ++u)
            if (j0 + u < n) G[(j0 + u) * R + q] = acc[u];
    }
}

// ---- the table dq[q][j*nd + k] -----------------------------------------------------------------
template <class T>
__device__ __forceinline__ T l2_change(T delta, T csq, T g) {
    const T twog = (T)2 * g;
    return delta * dmmv_fma(delta, csq, twog);
}

// A workgroup takes `width` variables x 2^qsh instances (64 x 32, or more variables of fewer instances): g and the current values
// go through LDS, read along the instances ([n][R]) and used along the table's rows, whose width * nd values of an instance are
// contiguous.  The host sizes the tile by its values (table_t).
// (One thread per variable and instance, its nd values written by itself: 242 us for 1376 tables of 4096 x 8, a
// wavefront's stores 64 tables apart; now 47.)
constexpr int LTB_Q = 32, LTB_AREA = 64 * (LTB_Q + 1), LTB_J = 256, LTB_EACH = 8, LTB_D = 256;
static constexpr int ltb_pitch(int32_t qsh) { return (1 << qsh) + (qsh > 0); }
static constexpr int ltb_most(int32_t qsh) {                // variables: what the tile, a thread's registers and sh_c hold
    int v = LTB_AREA / ltb_pitch(qsh);
    v = v < LTB_EACH * (256 >> qsh) ? v : LTB_EACH * (256 >> qsh);
    return v < LTB_J ? v : LTB_J;
}
template <class T>
__global__ __launch_bounds__(256) void k_l2_table(int64_t n, int64_t R, int32_t nd, int32_t width, int32_t qsh, const T* __restrict__ D,
                                                  const T* __restrict__ scale, const int32_t* __restrict__ kidx,
                                                  const T* __restrict__ g, const T* __restrict__ csq, T* __restrict__ dq) {
    __shared__ T sh_g[LTB_AREA], sh_d[LTB_AREA], sh_c[LTB_J], sh_lev[LTB_D];
    const int64_t j0 = blockIdx.x * (int64_t)width, q0 = (blockIdx.y + blockIdx.z * (int64_t)gridDim.y) << qsh;
    if (q0 >= R) return;
    const int32_t nj = (int32_t)(n - j0 < width ? n - j0 : width), nq = (int32_t)(R - q0 < 1 << qsh ? R - q0 : 1 << qsh);
    const int tid = threadIdx.x, lq = tid & ((1 << qsh) - 1), lj0 = tid >> qsh, step = 256 >> qsh;
    const int pitch = (1 << qsh) + (qsh > 0);
    T gv[LTB_EACH];
    int32_t kv[LTB_EACH];
#pragma unroll
    for (int u = 0; u < LTB_EACH; ++u) {
        if (u * step >= width) break;                       // uniform
        const int lj = lj0 + u * step;
        const int64_t at = (j0 + (lj < nj ? lj : nj - 1)) * R + q0 + (lq < nq ? lq : nq - 1);
        gv[u] = g[at];
        kv[u] = kidx[at];
    }
    const bool lev_lds = nd <= LTB_D;
    for (int32_t k = tid; lev_lds && k < nd; k += 256) sh_lev[k] = D[k];
#pragma unroll
    for (int u = 0; u < LTB_EACH; ++u) {
        if (u * step >= width) break;
        const int lj = lj0 + u * step;
        if (lj < width) {
            sh_g[lj * pitch + lq] = gv[u];
            sh_d[lj * pitch + lq] = D[kv[u]];
        }
    }
    for (int32_t lj = tid; lj < width; lj += 256) sh_c[lj] = csq[j0 + (lj < nj ? lj : nj - 1)];
    __syncthreads();
    // a wavefront takes an instance at a time, or with fewer than four several share one; its lanes walk (variable, value) in
    // table order
    const int lane = tid & 63, w = tid >> 6;
    const int share = nq >= 4 ? 1 : nq == 1 ? 4 : 2, jump = 64 * share;
    const int32_t step_j = jump / nd, step_k = jump % nd;
    for (int x = w / share; x < nq; x += 4 / share) {
        const T sc = scale[q0 + x];
        T* __restrict__ out = dq + (q0 + x) * (n * (int64_t)nd) + j0 * nd;
        const int32_t e0 = lane + 64 * (w % share);
        int32_t j = e0 / nd, k = e0 % nd;
        for (int64_t e = e0; j < nj; e += jump) {
            out[e] = l2_change(step_of(lev_lds ? sh_lev[k] : D[k], sh_d[j * pitch + x], sc), sh_c[j], sh_g[j * pitch + x]);
            k += step_k;
            j += step_j;
            if (k >= nd) { k -= nd; ++j; }
        }
    }
}

// ---- arg-min of a score table with dq as second criterion, one workgroup per instance ----------
template <class T>
__device__ __forceinline__ bool rec3_less(T s1, T q1, int64_t c1, T s2, T q2, int64_t c2) {
    if (c1 < 0) return false;
    if (c2 < 0) return true;
    if (s1 != s2) return s1 < s2;
    if (q1 != q2) return q1 < q2;
    return c1 < c2;
}

// The table is read once, eight values of a thread in flight; what the second criterion needs (g, the level and their
// dependent loads) is read for the first eight and then only where a score is not above the best that the wavefront has
// found.  per_xcd > 0: instances to an XCD, which then take neighbouring ones (g and the levels lie along the instances,
// a line of them serves 32).
// Before, every value took a 64-bit division and all loads (or, few instances, a thread took a variable's values one after the
// other).  us before and now, fp32: 1376 tables of 4096 x 8 135 and 46 (181 and 105 where most moves that lower the largest |r|
// raise the l2 norm and the loads cannot be left out: their lines are then what bounds it), 5000 of 600 x 4 85 and 47, 300 of
// 4096 x 16 78 and 31, 100 of 4096 x 8 28 and 17, one of 4096 x 16 34 and 15, one of 16 x 16 3.9 and 3.8.  Slower, by what the second of
// two dependent rounds takes, is one instance of some ten thousand values in fp64: 500 x 31 14.1 and 15.5 (with the next round's
// values requested ahead 16.1, and 5000 x 16 a fifth slower).
template <class T>
__global__ __launch_bounds__(1024) void k_l2_select(int64_t n, int64_t R, int32_t nd, int32_t rule,
                                                    const T* __restrict__ scores, const T* __restrict__ D,
                                                    const T* __restrict__ scale, const int32_t* __restrict__ kidx,
                                                    const T* __restrict__ g, const T* __restrict__ csq,
                                                    InstState<T>* st, int32_t keep_going, dmmv_move* best_out,
                                                    T* best_score_out, int64_t per_xcd) {
    __shared__ T sh_s[16], sh_q[16];
    __shared__ int64_t sh_c[16];
    const int64_t q = per_xcd > 0 ? (int64_t)(blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3) : (int64_t)blockIdx.x;
    if (q >= R) return;
    InstState<T> z = st[q];
    if (z.done && !best_out) return;
    const T sc = scale[q];
    const T* __restrict__ tab = scores + q * (n * (int64_t)nd);
    T bs = (T)0, bq = (T)0;
    int64_t bc = -1;
    constexpr int U = 8;                                   // values of a thread in flight
    const int32_t jump = (int32_t)blockDim.x;
    const uint32_t step_j = (uint32_t)jump / (uint32_t)nd, step_k = (uint32_t)jump % (uint32_t)nd;
    const uint32_t all_j = (uint32_t)(U * jump) / (uint32_t)nd, all_k = (uint32_t)(U * jump) % (uint32_t)nd;
    const int64_t count = n * (int64_t)nd;
    uint32_t j0 = threadIdx.x / (uint32_t)nd, k0 = threadIdx.x % (uint32_t)nd;      // of the first of them
    T most = Limits<T>::inf();                             // smallest score the wavefront has found: above it nothing counts
    auto batch = [&](int64_t e0, bool first) __attribute__((always_inline)) {
        T s[U];
        bool need[U], any = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = e0 + u * jump + threadIdx.x;
            s[u] = tab[e < count ? e : count - 1];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            need[u] = e0 + u * jump + threadIdx.x < count && (first || !(s[u] > most));
            any = any || need[u];
        }
        if (first || __builtin_amdgcn_ballot_w64(any) != 0ull) {
            uint32_t k[U], jn = j0, kn = k0;
            int32_t kc[U];
            T gj[U], cj[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t j = need[u] ? jn : 0;        // (one address for the lanes that need none)
                k[u] = need[u] ? kn : 0;
                kc[u] = kidx[j * R + q];
                gj[u] = g[j * R + q];
                cj[u] = csq[j];
                jn += step_j;
                kn += step_k;
                if (kn >= (uint32_t)nd) { kn -= (uint32_t)nd; ++jn; }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const T dq = l2_change(step_of(D[k[u]], D[kc[u]], sc), cj[u], gj[u]);
                const int64_t e = e0 + u * jump + threadIdx.x;
                if (!need[u] || (rule == 2 && !(dq <= (T)0))) continue;
                if (rec3_less(s[u], dq, e, bs, bq, bc)) { bs = s[u]; bq = dq; bc = e; }
            }
            most = wave_min(bc >= 0 ? bs : Limits<T>::inf());
        }
        j0 += all_j;
        k0 += all_k;
        if (k0 >= (uint32_t)nd) { k0 -= (uint32_t)nd; ++j0; }
    };
    if (count > 0) batch(0, true);
    for (int64_t e0 = U * jump; e0 < count; e0 += U * jump) batch(e0, false);      // whole wavefronts
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T os = __shfl_xor(bs, off, 64), oq = __shfl_xor(bq, off, 64);
        const int64_t oc = (int64_t)__shfl_xor((long long)bc, off, 64);
        if (rec3_less(os, oq, oc, bs, bq, bc)) { bs = os; bq = oq; bc = oc; }
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    if (lane == 0) { sh_s[w] = bs; sh_q[w] = bq; sh_c[w] = bc; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int u = 1; u < nw; ++u)
            if (rec3_less(sh_s[u], sh_q[u], sh_c[u], bs, bq, bc)) { bs = sh_s[u]; bq = sh_q[u]; bc = sh_c[u]; }
        int32_t j = -1, k = -1;
        if (bc >= 0) { j = (int32_t)(bc / nd); k = (int32_t)(bc % nd); }
        const bool improving = bc >= 0 && bs < z.t;
        z.best_s = bs;
        z.apply_j = improving ? j : -1;
        z.apply_k = improving ? k : -1;
        z.delta = improving ? step_of(D[k], D[kidx[(int64_t)j * R + q]], sc) : (T)0;
        if (!improving && !keep_going) z.done = 1;
        st[q] = z;
        if (best_out) { best_out[q].j = j; best_out[q].k = k; }
        if (best_score_out) best_score_out[q] = bc >= 0 ? bs : Limits<T>::inf();
    }
}

// sparse: what the loop's fused select-and-apply kernel does besides the update of r
template <class T>
__global__ void k_l2_after_apply_csc(InstState<T>* st, int32_t applied_before, int32_t iters, dmmv_move* trace,
                                     T* trace_t) {
    InstState<T> z = st[0];
    if (z.apply_j < 0) return;
    (void)applied_before;
    z.t = z.best_s;
    const int32_t slot = z.moves - 1;                     // the apply kernel has counted the move
    if (slot >= 0 && slot < iters) {
        if (trace) { trace[slot].j = z.apply_j; trace[slot].k = z.apply_k; }
        if (trace_t) trace_t[slot] = z.best_s;
    }
    st[0] = z;
}

template <class T>
dmmv_status colsq_t(Ctx* c) {
    const int64_t n = c->p.n;
    if (n == 0) return DMMV_OK;
    const dim3 grid((unsigned)ceil_div(n, 64));
    if (c->kind == KIND_CSC)
        hipLaunchKernelGGL(k_l2_sums_csc<T>, grid, dim3(64), 0, c->stream, c->p.m, n, c->csc_mp, c->csc_P,
                           (const int32_t*)c->segptr, (const uint16_t*)c->row16, (const T*)c->cval, (const T*)nullptr,
                           (T*)nullptr, (T*)c->l2_c);
    else
        hipLaunchKernelGGL(k_l2_colsq_dense<T>, grid, dim3(64), 0, c->stream, c->p.m, n, (const T*)c->p.A_dense,
                           c->p.lda, (T*)c->l2_c);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
dmmv_status update_g_t(Ctx* c) {
    const int64_t m = c->p.m, n = c->p.n, R = c->p.R;
    if (n == 0) return DMMV_OK;
    if (c->kind == KIND_CSC) {
        hipLaunchKernelGGL(k_l2_sums_csc<T>, dim3((unsigned)ceil_div(n, 64)), dim3(64), 0, c->stream, m, n, c->csc_mp,
                           c->csc_P, (const int32_t*)c->segptr, (const uint16_t*)c->row16, (const T*)c->cval,
                           (const T*)c->r, (T*)c->l2_g, (T*)nullptr);
    } else if (c->kind == KIND_DENSE) {
        hipLaunchKernelGGL(k_l2_g_dense<T>, dim3((unsigned)ceil_div(n, 64)), dim3(64), 0, c->stream, m, n,
                           (const T*)c->p.A_dense, c->p.lda, (const T*)c->r, (T*)c->l2_g);
    } else if (batched_chain_l2_applicable(c)) {
        return batched_chain_l2_g(c);
    } else {
        constexpr int TJ = 8;
        const dim3 grid((unsigned)ceil_div(R, 256), (unsigned)ceil_div(n, TJ));
        hipLaunchKernelGGL((k_l2_g_batched<T, TJ>), grid, dim3(256), 0, c->stream, m, n, R, (const T*)c->Xt,
                           (const T*)c->r, (T*)c->l2_g);
    }
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
dmmv_status table_t(Ctx* c, void* dq_out) {
    const int64_t n = c->p.n, R = c->p.R;
    if (n == 0) return DMMV_OK;
    // A workgroup's values: 32768, less where there would be fewer than two workgroups a compute unit (full tiles of 64 x 32
    // left 500 instances of 64 variables and 16 values to 16 workgroups: 20 us, now 6; 100 of 1000 x 64 values 74 and 12), 512 at least.
    int32_t qsh = 0;
    while (1 << qsh < LTB_Q && 1ll << qsh < R) ++qsh;
    int64_t values = n * R * c->p.nd / 512;
    values = values < 512 ? 512 : values > 32768 ? 32768 : values;
    int64_t width = values / ((int64_t)c->p.nd << qsh);
    width = width < 1 ? 1 : width > ltb_most(qsh) ? ltb_most(qsh) : width;
    const int64_t gq = ceil_div(R, 1ll << qsh), gy = gq < 32768 ? gq : 32768;
    hipLaunchKernelGGL(k_l2_table<T>, dim3((unsigned)ceil_div(n, width), (unsigned)gy, (unsigned)ceil_div(gq, gy)), dim3(256), 0, c->stream, n, R, c->p.nd,
                       (int32_t)width, qsh,
                       (const T*)c->D_dev, (const T*)c->scale_dev, (const int32_t*)c->kidx, (const T*)c->l2_g,
                       (const T*)c->l2_c, (T*)dq_out);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
dmmv_status select_t(Ctx* c, const void* scores, int32_t keep_going, dmmv_move* best_out, void* best_score_out) {
    // A thread takes eight values at least, and the more the fewer wavefronts an instance has: 256 threads where the instances fill
    // the chip (with 1024 small tables were slower than before: 5000 of 600 x 4 118 us, now 47), up to 1024 for few.
    const int64_t values = c->p.n * c->p.nd;
    unsigned threads = 64;
    while (threads < (c->p.R > 256 ? 256u : 1024u) && 8 * (int64_t)threads < values) threads *= 2;
    const int64_t per_xcd = c->p.R >= 64 ? ceil_div(c->p.R, 8) : 0;
    hipLaunchKernelGGL(k_l2_select<T>, dim3((unsigned)(per_xcd > 0 ? 8 * per_xcd : c->p.R)), dim3(threads), 0, c->stream, c->p.n, c->p.R, c->p.nd,
                       c->o.l2_rule, (const T*)scores, (const T*)c->D_dev, (const T*)c->scale_dev,
                       (const int32_t*)c->kidx, (const T*)c->l2_g, (const T*)c->l2_c, (InstState<T>*)c->state,
                       keep_going, best_out, (T*)best_score_out, per_xcd);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
dmmv_status after_apply_csc_t(Ctx* c, int32_t iters, dmmv_move* trace, void* trace_t) {
    hipLaunchKernelGGL(k_l2_after_apply_csc<T>, dim3(1), dim3(1), 0, c->stream, (InstState<T>*)c->state, 0, iters, trace,
                       (T*)trace_t);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

}  // namespace

#define L2_DISPATCH(fn, ...) (c->p.dtype == DMMV_F64 ? fn<double>(__VA_ARGS__) : fn<float>(__VA_ARGS__))

dmmv_status l2_build(Ctx* c) { return L2_DISPATCH(colsq_t, c); }
dmmv_status l2_update_g(Ctx* c) { return L2_DISPATCH(update_g_t, c); }
dmmv_status l2_table(Ctx* c, void* dq_out) { return L2_DISPATCH(table_t, c, dq_out); }
dmmv_status l2_select(Ctx* c, const void* scores, int32_t keep_going, dmmv_move* best_out, void* best_score_out) {
    return L2_DISPATCH(select_t, c, scores, keep_going, best_out, best_score_out);
}
dmmv_status l2_after_apply_csc(Ctx* c, int32_t iters, dmmv_move* trace, void* trace_t) {
    return L2_DISPATCH(after_apply_csc_t, c, iters, trace, trace_t);
}

}  // namespace dmmv
