// ALNS outer loop of AMVM (Algorithm 1 of the paper) around the single-move descent:
// destroy (random / worst-remove, Appendix B.1-B.2), repair (random / greedy, B.1, B.3),
// local search, acceptance, adaptive operator weights (Appendix F.2).
//
// Everything is decided on the device; the host only enqueues a fixed sequence of kernels
// per outer iteration.  Whatever a floating-point value decides is decided on integers or by
// a fixed sequence of IEEE operations, so that an independent implementation can follow the
// run move by move:
//   - random numbers are a counter-based chain of SplitMix64 steps addressed by
//     (seed, instance, outer iteration, stream, counter);
//   - the impact score of the worst-remove operator is accumulated in fixed point
//     (a sum of integers does not depend on the order of its terms) and becomes an integer
//     sampling weight; exp is a fixed Horner polynomial after a fixed range reduction;
//   - variables are drawn against integer prefix sums, a repeated draw is skipped.
// This file holds what is independent of the matrix storage plus the dense kernels.
#include <type_traits>

#include "dmmv_alns_common.h"

namespace dmmv {

// ----------------------------------------------------------------------------------------
// loop control.  R instances (R = 1 unless batched): instance q owns S[q], st[q], the slices
// q*n.. of weight / prefix / first, q*count.. of picked; x and r are instance-contiguous
// (kidx[j*R + q], r[i*R + q]) as everywhere in the batched path.
// ----------------------------------------------------------------------------------------
// Squared l2 norm of the residual of every instance, in double precision and in a fixed order:
// rows in blocks of 256, inside a block acc = fma(r_i, r_i, acc) by ascending row, then the
// block sums by ascending block.  Batch: one lane per instance walks all rows (coalesced over
// the instances).
template <class T>
__global__ void k_alns_sumsq_batched(int64_t m, int64_t R, const T* __restrict__ r, double* __restrict__ q2) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= R) return;
    double total = 0.0;
    for (int64_t i0 = 0; i0 < m; i0 += 256) {
        double acc = 0.0;
        const int64_t i1 = i0 + 256 < m ? i0 + 256 : m;
        for (int64_t i = i0; i < i1; ++i) {
            const double v = (double)r[i * R + q];
            acc = __builtin_fma(v, v, acc);
        }
        total += acc;
    }
    q2[q] = total;
}

// Single instance: one thread per block of 256 rows, then one thread adds the block sums.
template <class T>
__global__ __launch_bounds__(1024) void k_alns_sumsq_single(int64_t m, const T* __restrict__ r,
                                                            double* __restrict__ blocks, double* __restrict__ q2) {
    const int64_t nblk = (m + 255) / 256;
    for (int64_t bk = threadIdx.x; bk < nblk; bk += blockDim.x) {
        double acc = 0.0;
        const int64_t i0 = bk * 256, i1 = i0 + 256 < m ? i0 + 256 : m;
        for (int64_t i = i0; i < i1; ++i) {
            const double v = (double)r[i];
            acc = __builtin_fma(v, v, acc);
        }
        blocks[bk] = acc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0;
        for (int64_t bk = 0; bk < nblk; ++bk) total += blocks[bk];
        q2[0] = total;
    }
}

// operators of outer iteration `it` by roulette wheel
__device__ __forceinline__ void alns_begin(AlnsState* S, int64_t q, uint64_t seed, int32_t it) {
    const double ud = alns_unit(alns_rnd(seed, (uint64_t)q, (uint64_t)it, 0, 0));
    const double ur = alns_unit(alns_rnd(seed, (uint64_t)q, (uint64_t)it, 0, 1));
    S[q].it = it;
    S[q].d_op = (ud * (S[q].w[0] + S[q].w[1]) < S[q].w[0]) ? 0 : 1;
    S[q].r_op = (ur * (S[q].w[2] + S[q].w[3]) < S[q].w[2]) ? 0 : 1;
}

template <class T>
__global__ void k_alns_init(AlnsState* S, const InstState<T>* st, int64_t R, const double* q2, uint64_t seed) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= R) return;
    S[q].q2_cur = q2 ? q2[q] : 0.0;
    for (int u = 0; u < 4; ++u) S[q].w[u] = 1.0;
    S[q].t_cur = (double)st[q].t;
    S[q].t_best = (double)st[q].t;
    S[q].accepted = 0; S[q].turn = 0;
    alns_begin(S, q, seed, 0);
}

// Destroy: the prefix sums of the weights where the operator is worst-remove, then the draws.  One workgroup of NT threads
// per instance.
constexpr int SC_E = 8;
constexpr int SC_MARKS = 1024;                 // prefix sums kept in LDS, at every `stride` weights

struct DestroyShared {
    uint64_t mark[SC_MARKS];                   // sum of the weights ahead of weight e * stride
    uint64_t wave[16];
    int32_t cnt[16];
    int32_t have;
};

__device__ __forceinline__ int64_t alns_mark_stride(int64_t n) { return (n + SC_MARKS * SC_E - 1) / (SC_MARKS * SC_E) * SC_E; }

// Inclusive prefix sums of the weights.
// raw_shift >= 0: what is stored are the sums of the impact terms, a weight is 1 + (sum >> raw_shift).
// The weights are integers, so the sums are the same in any order: a thread sums SC_E
// consecutive weights in registers, the wavefronts scan the threads' totals, and the total of a
// tile of NT * SC_E weights is carried into the next.
// clear: the weights are set to 0 for the next iteration, whose terms are added to them.
template <int NT>
__device__ __forceinline__ void alns_scan(int64_t n, uint64_t* weight, uint64_t* prefix, int32_t raw_shift, int32_t clear,
                                          DestroyShared& L) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t stride = alns_mark_stride(n);
    uint64_t carry = 0;                                     // the same in every thread
    for (int64_t base = 0; base < n; base += NT * SC_E) {
        const int64_t j0 = base + (int64_t)threadIdx.x * SC_E;
        uint64_t v[SC_E];
#pragma unroll
        for (int u = 0; u < SC_E; ++u) v[u] = weight[j0 + u < n ? j0 + u : n - 1];   // clamped: the loads go out together
#pragma unroll
        for (int u = 0; u < SC_E; ++u) {
            if (raw_shift >= 0) v[u] = 1 + (v[u] >> raw_shift);
            v[u] = j0 + u < n ? v[u] : 0;
        }
        if (clear) {
#pragma unroll
            for (int u = 0; u < SC_E; ++u)
                if (j0 + u < n) weight[j0 + u] = 0;
        }
#pragma unroll
        for (int u = 1; u < SC_E; ++u) v[u] += v[u - 1];
        const uint64_t tot = v[SC_E - 1];
        uint64_t inc = tot;                                 // inclusive over the wavefront's threads
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t t = (uint64_t)__shfl_up((long long)inc, off, 64);
            if (lane >= off) inc += t;
        }
        if (lane == 63) L.wave[w] = inc;
        __syncthreads();
        uint64_t before = 0, all = 0;
#pragma unroll
        for (int k = 0; k < NT / 64; ++k) {
            const uint64_t x = L.wave[k];
            if (k < w) before += x;
            all += x;
        }
        const uint64_t ex = carry + before + (inc - tot);   // everything ahead of this thread
        if (j0 < n && j0 % stride == 0) L.mark[j0 / stride] = ex;
#pragma unroll
        for (int u = 0; u < SC_E; ++u)
            if (j0 + u < n) prefix[j0 + u] = v[u] + ex;
        carry += all;
        __syncthreads();                                    // L.wave is written again, the sums are read
    }
}

// the first weight whose prefix sum exceeds v (below the total)
__device__ __forceinline__ int64_t alns_find(int64_t n, const uint64_t* prefix, uint64_t v, const DestroyShared& L) {
    const int64_t stride = alns_mark_stride(n);
    int32_t lo = 0, hi = (int32_t)((n - 1) / stride);       // the last mark not above v: the sum ahead of it is not above v
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (L.mark[mid] > v) hi = mid - 1; else lo = mid;
    }
    int64_t j = lo * stride, end = j + stride < n ? j + stride : n;
    while (end - j > SC_E) {
        const int64_t mid = (j + end) / 2;
        if (prefix[mid - 1] > v) end = mid; else j = mid;
    }
    uint64_t x[SC_E];                                       // (the rest at once)
#pragma unroll
    for (int u = 0; u < SC_E; ++u) x[u] = prefix[j + u < n ? j + u : n - 1];
    int32_t more = 0;
#pragma unroll
    for (int u = 0; u < SC_E; ++u) more += j + u < end - 1 && !(x[u] > v) ? 1 : 0;
    return j + more;
}

// Draw `count` distinct variables.  Draw c takes rnd(.., 1, c) mod
// total and the first variable whose prefix sum exceeds it (all weights 1 for the random
// operator); a variable drawn before is skipped.  A few variables are drawn by one wavefront, which compares its lanes' draws;
// otherwise (or if too many of the 64 were alike) NT draws are made at a time: a draw is
// the first of its variable exactly if it holds the largest stamp (iteration, -c) that
// variable has seen.
constexpr int SAMPLE_FEW = 32;
template <int NT>
__device__ __forceinline__ void alns_sample(int64_t n, int32_t count, const uint64_t* prefix, unsigned long long* first,
                                            int32_t* picked, int64_t q, int32_t it, bool weighted, uint64_t seed,
                                            DestroyShared& L) {
    const uint64_t total = weighted ? prefix[n - 1] : (uint64_t)n;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = NT / 64;
    auto draw = [&](uint64_t c) -> int64_t {
        const uint64_t v = alns_rnd(seed, (uint64_t)q, (uint64_t)it, 1, c) % total;
        return weighted ? alns_find(n, prefix, v, L) : (int64_t)v;
    };
    if (threadIdx.x == 0) L.have = 0;
    __syncthreads();
    if (count <= SAMPLE_FEW) {
        if (w == 0) {
            const int32_t j = (int32_t)draw((uint64_t)lane);
            bool is_first = true;
#pragma unroll
            for (int e = 0; e < 63; ++e) is_first = is_first && !(e < lane && __builtin_amdgcn_readlane(j, e) == j);
            const unsigned long long bal = __ballot(is_first);
            if (__popcll(bal) >= count) {
                const int32_t pos = __popcll(bal & ((1ull << lane) - 1ull));
                if (is_first && pos < count) picked[pos] = j;
                if (lane == 0) L.have = count;
            }
        }
        __syncthreads();
    }
    for (uint64_t base = 0;; base += NT) {
        const int32_t have = L.have;
        if (have >= count) break;
        const uint64_t c = base + threadIdx.x;
        const int64_t j = draw(c);
        const unsigned long long stamp = ((unsigned long long)(it + 1) << 32) | (0xFFFFFFFFull - (c & 0xFFFFFFFFull));
        atomicMax(&first[j], stamp);
        // (other wavefronts read it behind the barrier, which by itself waits for no atomic that returns nothing)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const bool is_first = __hip_atomic_load(&first[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == stamp;
        const unsigned long long bal = __ballot(is_first);
        if (lane == 0) L.cnt[w] = __popcll(bal);
        __syncthreads();
        int32_t before = 0, all = 0;
        for (int u = 0; u < nw; ++u) { if (u < w) before += L.cnt[u]; all += L.cnt[u]; }
        const int32_t pos = have + before + __popcll(bal & ((1ull << lane) - 1ull));
        if (is_first && pos < count) picked[pos] = (int32_t)j;
        __syncthreads();
        if (threadIdx.x == 0) L.have = have + all;
        __syncthreads();
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_alns_destroy(int64_t n, int32_t count, uint64_t* weight_all, uint64_t* prefix_all,
                                                     unsigned long long* first_all, int32_t* picked_all, const AlnsState* S,
                                                     uint64_t seed, int32_t raw_shift, int32_t clear) {
    __shared__ DestroyShared L;
    const int64_t q = blockIdx.x;
    const bool weighted = S[q].d_op == 1;
    if (weighted) alns_scan<NT>(n, weight_all + q * n, prefix_all + q * n, raw_shift, clear, L);
    alns_sample<NT>(n, count, prefix_all + q * n, first_all + q * n, picked_all + q * (int64_t)count, q, S[q].it, weighted, seed, L);
}

// Destroy and repair of a dense instance (single or of a batch) in one launch.  A thread keeps its rows tid, tid + NT, .. of r in
// registers for all picks; the picks' levels, steps and random bits are looked up for up to RP_PICKS of them at once, the next
// pick's column is requested before the present one is used, and a greedy choice costs one barrier (two columns' trips to
// memory, a chain of three loads and four barriers a pick before).  Three launches and a fourth that cleared the exchange of
// the one-launch descent: 26 us on 8016 x 251 (2 picks), now 15.5; 25 and 18 on 20 instances of 2048 x 768 (4 picks), 135 and 85 on 1024 of
// 2048 x 4096 (21 picks).  What is left is a chain of latencies.
constexpr int RP_PICKS = 256;
template <class T, int NT, int RPT>
__global__ __launch_bounds__(NT) void k_alns_destroy_repair(int64_t m, int64_t n, int64_t R, int32_t nd, int32_t count,
                                                            uint64_t* weight_all, uint64_t* prefix_all,
                                                            unsigned long long* first_all, int32_t* picked_all,
                                                            const AlnsState* S, uint64_t seed, int32_t raw_shift, int32_t clear,
                                                            const T* __restrict__ A, int64_t lda, const T* __restrict__ D,
                                                            const T* __restrict__ scale_q, T* __restrict__ r, int32_t* kidx,
                                                            InstState<T>* st, uint32_t* zero, int32_t zero_words) {
    __shared__ DestroyShared L;
    __shared__ int32_t sh_j[RP_PICKS];
    __shared__ int32_t sh_k[RP_PICKS];                      // the level to take; with bit 30: this one or the one two below
    __shared__ T sh_up[RP_PICKS], sh_down[RP_PICKS];        // the step to it, or both
    __shared__ T sh_max[2][2][NT / 64];
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int32_t it = S[q].it, m32 = (int32_t)m;
    const bool greedy = S[q].r_op == 1, weighted = S[q].d_op == 1;
    int32_t* picked = picked_all + q * (int64_t)count;
    T rr[RPT], a[RPT], next[RPT];
    if (m32 > 0) {
#pragma unroll
        for (int u = 0; u < RPT; ++u) rr[u] = r[(int64_t)(tid + NT * u < m32 ? tid + NT * u : m32 - 1) * R + q];
    }
    for (int32_t e = tid; e < zero_words; e += NT) zero[e] = 0;       // (the exchange of the descent that follows)
    if (weighted) alns_scan<NT>(n, weight_all + q * n, prefix_all + q * n, raw_shift, clear, L);
    alns_sample<NT>(n, count, prefix_all + q * n, first_all + q * n, picked, q, it, weighted, seed, L);
    const T sc = scale_q[q];
    int turn = 0;                                           // a greedy choice's half of sh_max: the other is read until the next barrier
    for (int32_t p0 = 0; p0 < count; p0 += RP_PICKS) {
        const int32_t here = count - p0 < RP_PICKS ? count - p0 : RP_PICKS;
        if (p0 > 0) __syncthreads();                        // the tables are read no more
        for (int32_t p = tid; p < here; p += NT) {
            const int64_t j = picked[p0 + p];
            const int32_t kc = kidx[j * R + q];
            const bool has_lo = kc > 0, has_hi = kc < nd - 1;
            bool up = !has_lo;
            if (has_lo && has_hi && !greedy) up = (alns_rnd(seed, (uint64_t)q, (uint64_t)it, 2, (uint64_t)(p0 + p)) & 1) != 0;
            const int32_t klo = has_lo ? kc - 1 : kc, khi = has_hi ? kc + 1 : kc;
            sh_j[p] = (int32_t)j;
            sh_k[p] = has_lo && has_hi && greedy ? (khi | (1 << 30)) : up ? khi : klo;
            sh_up[p] = step_of(D[khi], D[kc], sc);
            sh_down[p] = step_of(D[klo], D[kc], sc);
            if (!(has_lo && has_hi && greedy) && !up) sh_up[p] = sh_down[p];
        }
        __syncthreads();
        auto fetch = [&](int32_t p) {
            const T* __restrict__ col = A + lda * sh_j[p < here ? p : here - 1];
#pragma unroll
            for (int u = 0; u < RPT; ++u) next[u] = col[tid + NT * u < m32 ? tid + NT * u : m32 - 1];
        };
        if (m32 > 0) fetch(0);
        for (int32_t p = 0; p < here; ++p) {
#pragma unroll
            for (int u = 0; u < RPT; ++u) a[u] = next[u];
            if (m32 > 0) fetch(p + 1);
            const int32_t kk = sh_k[p];
            T delta = sh_up[p];
            int32_t k = kk & ~(1 << 30);
            if (kk >> 30) {                                 // the same for the whole workgroup
                const T dlo = sh_down[p];
                T elo = (T)0, ehi = (T)0;
                if (m32 > 0) {                              // (rows past the end repeat row m - 1, which changes no maximum)
#pragma unroll
                    for (int u = 0; u < RPT; ++u) {
                        elo = dmmv_max(elo, dmmv_abs(dmmv_fma(dlo, a[u], rr[u])));
                        ehi = dmmv_max(ehi, dmmv_abs(dmmv_fma(delta, a[u], rr[u])));
                    }
                }
                elo = wave_max(elo);
                ehi = wave_max(ehi);
                if (lane == 0) { sh_max[turn][0][w] = elo; sh_max[turn][1][w] = ehi; }
                __syncthreads();
                for (int e = 0; e < NT / 64; ++e) {
                    elo = dmmv_max(elo, sh_max[turn][0][e]);
                    ehi = dmmv_max(ehi, sh_max[turn][1][e]);
                }
                turn ^= 1;
                if (!(ehi < elo)) { delta = dlo; k -= 2; }
            }
#pragma unroll
            for (int u = 0; u < RPT; ++u) rr[u] = dmmv_fma(delta, a[u], rr[u]);
            if (tid == 0) kidx[(int64_t)sh_j[p] * R + q] = k;
        }
    }
    T tmax = (T)0;
#pragma unroll
    for (int u = 0; u < RPT; ++u)
        if (tid + NT * u < m32) {
            tmax = dmmv_max(tmax, dmmv_abs(rr[u]));
            r[(int64_t)(tid + NT * u) * R + q] = rr[u];
        }
    tmax = block_max(tmax, &sh_max[0][0][0]);
    if (tid == 0) { st[q].t = tmax; st[q].done = 0; st[q].moves = 0; }
}

// The end of an outer iteration and the start of the next one (unless it was the last).  Every thread takes the verdict
// for the elements that it copies: accepted: current <- working (and best <- working for a new best); rejected: working
// <- current.  The last workgroup to have done so with a strip of instances (the strip counts them) then updates their state: error,
// operator weights, trace, the next iteration's operators.  One launch instead of three (us): 5.5 instead of 13 on 8016 x 251, 8.4 instead
// of 11 on 20 instances of 2048 x 768, 28 instead of 42 on 1024 of 2048 x 4096, 91 instead of 170 on 11 008 of 2048 x 256, 11 instead of 25
// on 60 000 of 8 x 8.  (With one workgroup that updated the states of all instances: 36, 211 and 696 on the last three.)
template <class T>
__device__ __forceinline__ void alns_verdict(const AlnsState& s, const InstState<T>& z, const double* q2, int64_t q, bool& accepted, bool& best) {
    const double t = (double)z.t;
    // q2 != NULL: the l2 norm of the residual must not increase either
    accepted = t <= s.t_cur && (!q2 || q2[q] <= s.q2_cur);
    best = accepted && t < s.t_best;
}

template <class T>
__device__ __forceinline__ void alns_end(AlnsState* S, InstState<T>* st, int64_t q, int32_t iters, double lambda, double sigma1,
                                         double sigma2, double sigma3, const double* q2, int32_t* trace, T* trace_t) {
    const double t = (double)st[q].t;
    const int32_t it = S[q].it;
    bool accepted, new_best;
    alns_verdict(S[q], st[q], q2, q, accepted, new_best);
    if (accepted) {
        if (q2) S[q].q2_cur = q2[q];
        double psi = sigma3;
        if (t < S[q].t_cur) psi = sigma2;
        if (new_best) { psi = sigma1; S[q].t_best = t; }
        S[q].t_cur = t;
        const double keep = 1.0 - lambda;
        S[q].w[S[q].d_op] = keep * S[q].w[S[q].d_op] + lambda * psi;
        S[q].w[2 + S[q].r_op] = keep * S[q].w[2 + S[q].r_op] + lambda * psi;
    }
    S[q].accepted = accepted;
    const int64_t slot = q * (int64_t)iters + it;
    if (trace) {
        trace[slot * 4 + 0] = S[q].d_op; trace[slot * 4 + 1] = S[q].r_op;
        trace[slot * 4 + 2] = st[q].moves; trace[slot * 4 + 3] = accepted;
    }
    if (trace_t) { trace_t[slot * 2 + 0] = st[q].t; trace_t[slot * 2 + 1] = (T)S[q].t_best; }
    if (!accepted) st[q].t = (T)S[q].t_cur;          // (x and r have been restored)
}

// grid: a strip of 256 instances (or 256 elements of the only one) x some of the rows and variables
template <class T>
__global__ __launch_bounds__(256) void k_alns_turn(int64_t m, int64_t n, int64_t R, AlnsState* S, InstState<T>* st, int32_t* kidx,
                                                   int32_t* kidx_cur, int32_t* kidx_best, T* r, T* r_cur, int32_t iters,
                                                   double lambda, double sigma1, double sigma2, double sigma3, const double* q2,
                                                   int32_t* trace, T* trace_t, uint64_t seed, int32_t next) {
    __shared__ bool last;
    const int64_t at = blockIdx.x * 256ll + threadIdx.x;
    // an instance of its own for every thread, rows over the workgroups; or one instance, rows over the threads too
    const int64_t q = R > 1 ? at : 0, e0 = R > 1 ? blockIdx.y : at, step = R > 1 ? gridDim.y : gridDim.x * 256ll;
    if (q < R) {
        bool accepted, best;
        alns_verdict(S[q], st[q], q2, q, accepted, best);
        // (eight elements in flight in a thread)
        auto copy = [&](int64_t rows, auto* work, auto* cur, auto* most) {
            for (int64_t j0 = e0; j0 < rows; j0 += 8 * step) {
                std::remove_reference_t<decltype(*work)> v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) { const int64_t j = j0 + u * step; v[u] = (accepted ? work : cur)[(j < rows ? j : rows - 1) * R + q]; }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int64_t j = j0 + u * step;
                    if (j >= rows) break;
                    (accepted ? cur : work)[j * R + q] = v[u];
                    if (most && best) most[j * R + q] = v[u];
                }
            }
        };
        copy(n, kidx, kidx_cur, kidx_best);
        copy(m, r, r_cur, (T*)nullptr);
    }
    __syncthreads();                                  // (nobody here reads the state any more)
    int32_t* turn = &S[R > 1 ? blockIdx.x * 256ll : 0].turn;
    if (threadIdx.x == 0)                             // (a count only: no fence, which would write the caches back)
        last = atomicAdd(turn, 1) == (int32_t)(R > 1 ? gridDim.y : gridDim.x) - 1;
    __syncthreads();
    if (!last) return;
    if (R > 1 ? q < R : threadIdx.x == 0) {
        alns_end(S, st, q, iters, lambda, sigma1, sigma2, sigma3, q2, trace, trace_t);
        if (next >= 0) alns_begin(S, q, seed, next);
    }
    if (threadIdx.x == 0) *turn = 0;
}

template <class T>
__global__ void k_alns_snapshot(int64_t m, int64_t n, int64_t R, const int32_t* kidx, int32_t* kidx_cur,
                                int32_t* kidx_best, const T* r, T* r_cur, unsigned long long* first, uint64_t* weight) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t e = t0; e < n * R; e += stride) { kidx_cur[e] = kidx[e]; kidx_best[e] = kidx[e]; first[e] = 0; weight[e] = 0; }
    for (int64_t e = t0; e < m * R; e += stride) r_cur[e] = r[e];
}

template <class T>
__global__ void k_alns_export(const AlnsState* S, int64_t R, T* t_best_out) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q < R && t_best_out) t_best_out[q] = (T)S[q].t_best;
}

// ----------------------------------------------------------------------------------------
// dense matrix: impact weights and repair
// ----------------------------------------------------------------------------------------
// single instance: one workgroup per variable, the rows spread over its threads
template <class T>
__global__ __launch_bounds__(256) void k_alns_impact_dense(int64_t m, int64_t n, const T* __restrict__ A,
                                                           int64_t lda, const T* __restrict__ r,
                                                           const InstState<T>* st, double alpha,
                                                           uint64_t* __restrict__ weight, const AlnsState* S) {
    __shared__ uint64_t sh[4];
    if (S->d_op != 1) return;
    const int64_t j = blockIdx.x;
    const double t = (double)st[0].t;
    const double scale = alns_impact_scale(t);
    uint64_t sum = 0;
    if (scale != 0.0) {
        const T* __restrict__ col = A + lda * j;
        for (int64_t i = threadIdx.x; i < m; i += blockDim.x)
            sum += alns_impact_term(__builtin_fabs((double)col[i]), __builtin_fabs((double)r[i]), t, alpha, scale);
    }
    sum = block_sum_u64(sum, sh);
    if (threadIdx.x == 0) {
        int shift = alns_bits(m) + 24 + alns_bits(n) - 62;
        if (shift < 0) shift = 0;
        weight[j] = 1 + (sum >> shift);
    }
}

// batched: the instances whose destroy operator of this iteration is worst-remove, in ascending
// order (single workgroup); their number goes to flags[FLAG_WORST].  The impact kernel works on
// this list, so that its wavefronts are full of instances that need weights.
__global__ __launch_bounds__(1024) void k_alns_worst_list(int64_t R, const AlnsState* __restrict__ S,
                                                          int32_t* __restrict__ list, int32_t* flags) {
    __shared__ int32_t sh_cnt[16];
    __shared__ int32_t sh_base;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (threadIdx.x == 0) sh_base = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < R; b0 += 1024) {
        const int64_t q = b0 + threadIdx.x;
        const bool on = q < R && S[q].d_op == 1;
        const unsigned long long bal = __ballot(on);
        if (lane == 0) sh_cnt[w] = __popcll(bal);
        __syncthreads();
        int32_t before = 0, all = 0;
        for (int u = 0; u < 16; ++u) { if (u < w) before += sh_cnt[u]; all += sh_cnt[u]; }
        const int32_t base = sh_base;
        if (on) list[base + before + __popcll(bal & ((1ull << lane) - 1ull))] = (int32_t)q;
        __syncthreads();
        if (threadIdx.x == 0) sh_base = base + all;
        __syncthreads();
    }
    if (threadIdx.x == 0) flags[FLAG_WORST] = sh_base;
}

// batched: impact weights of the listed instances, sum over the rows of the fixed-point terms.
//
// Only a few per cent of the terms reach 1; the rest truncate to 0.  A term sk e^(-alpha slack / a)
// scale (sk = |r_i|, slack = t - sk, a = |sc x|) reaches 1 exactly when alpha slack / a <= ln(sk scale),
// i.e. when |x| is at least a limit that depends on the row and the instance alone.  The limits are
// written first (k_alns_impact_limits, lowered by 1 % so that the roundings on both sides are covered: a term the
// test drops is 0, the reverse need not hold), then a term costs one comparison.
//
// fp32 batches of 129 to 8192 variables take k_alns_impact_lists instead (dmmv_alns_impact.hip), which is 3.9 times as fast
// on the layer named below; fp64, fewer and more variables are left to this one.
//
// k_alns_impact_batched: lane = variable, so a row of X is one coalesced load that IM_Q instances share
// (with lane = instance and X through the scalar unit a small batch left most of the chip idle:
// 1.56 ms for the listed half of 20 instances of 2048 x 768, and 5.0 ms for that of 1024 of 2048 x 4096; now 0.056 and
// 1.8 ms, the limits' launch 0.01 and 0.02 more).  A wavefront takes 64 variables x IM_Q instances x IM_ROWS rows at a time: the tests leave one bit
// per row in a mask (two instructions a term), the set bits go to a queue in LDS, a lane's behind those of the lanes before
// it, and the queue is evaluated two entries a lane, for whichever variable and instance they belong to, the integers
// added to the sums with LDS atomics.  About 1050 vector instructions per 64 x 4 x 32 terms, a quarter of them the tests
// and a third the evaluations, the unit 60 % busy.  Where most terms of most variables count (no outlier channels, or a small
// alpha) they are evaluated row by row without the queue: 1000 instances of 700 x 128, normal entries, 239 us with the queue of
// the kernel before, 275 with this one, 145 without; 5000 of 32 x 100 100, 126 and 45.  (One entry a lane: 1.88 ms; the bits
// popped a variable at a time over the wavefront, with an evaluation whenever 64 were waiting and the whole of the term's
// arithmetic in it: 2.25.)  The sums are integers, so neither their order nor the split of the rows over workgroups (small
// batches: one pass each, 0.056 ms against 0.10 with two) changes a weight.
constexpr int IM_Q = 4;                        // instances that share a row of X
constexpr int IM_ROWS = 32;                    // rows per pass: one mask bit each
constexpr int IM_STAGE = IM_ROWS * IM_Q / 64;  // (row, instance) pairs a lane stages per pass
constexpr int IM_MOST = 64 * IM_ROWS;          // terms of an instance a pass can have
constexpr int IM_CAP = IM_MOST + 512;          // queue of a wavefront: evaluated when over 512 are waiting
constexpr int IM_DENSE = 14;                   // more terms than this in half of the variables: no queue
constexpr int IM_FEW = 8;                      // a variable with more terms than this in a pass is queued by rows

// mask = 2 mask + (|x| >= lim): the comparison's bit enters as the carry of one addition
__device__ __forceinline__ uint32_t impact_test(uint32_t mask, float x, float lim) {
    asm("v_cmp_ge_f32 vcc, abs(%1), %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(mask) : "v"(x), "v"(lim) : "vcc");
    return mask;
}
__device__ __forceinline__ uint32_t impact_test(uint32_t mask, double x, double lim) {
    asm("v_cmp_ge_f64 vcc, abs(%1), %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(mask) : "v"(x), "v"(lim) : "vcc");
    return mask;
}

template <class T>
struct ImpactShared {
    double rate[4][IM_ROWS][IM_Q], base[4][IM_ROWS][IM_Q];   // per row and instance: 16 log2(e) alpha (t - sk) / sc, sk scale
    T lim[4][IM_ROWS][IM_Q];
    unsigned long long sum[4][IM_Q][64];
    uint16_t queue[4][IM_CAP];                 // lane | instance << 6 | row << 8
    double rate_q[IM_Q], t[IM_Q], scale[IM_Q]; // per instance: 16 log2(e) alpha / sc, error, fixed-point scale
    double exp2m[16];                          // 2^(-f/16)
};

// inclusive sum over the lanes up to this one
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);      // row_shr 1, 2, 4, 8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);      // row_bcast 15, 31
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
    return v;
}

// lim[i][slot], smallest |x| whose term may reach 1 in row i of the slot's instance; clears the sums
template <class T>
__global__ __launch_bounds__(256) void k_alns_impact_limits(int64_t m, int64_t n, int64_t R, const T* __restrict__ scale_q,
                                                            const T* __restrict__ r, const InstState<T>* st, double alpha,
                                                            T* __restrict__ lim, uint64_t* __restrict__ weight,
                                                            const int32_t* __restrict__ list,
                                                            const int32_t* __restrict__ flags) {
    const int64_t count = flags[FLAG_WORST];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t slot = blockIdx.x * 64ll + lane;
    if (blockIdx.x * 64ll >= count) return;
    const int64_t q = list[slot < count ? slot : count - 1];
    const double t = (double)st[q].t, sc = (double)scale_q[q], scale = alns_impact_scale(t);
    for (int64_t i = blockIdx.y * 4ll + w; i < m; i += 4ll * gridDim.y) {
        const double sk = __builtin_fabs((double)r[i * R + q]), v = sk * scale;
        double l = (double)Limits<T>::inf();
        if (slot < count && v >= 0.999) l = (t - sk) * alpha / (sc * ((log(v) + 0.01) * 1.01));
        if (slot < count) lim[i * R + slot] = (T)l;
    }
    for (int64_t s = blockIdx.x * 64ll + w; s < count && s < (blockIdx.x + 1) * 64ll; s += 4) {
        uint64_t* __restrict__ out = weight + (int64_t)list[s] * n;
        for (int64_t j = blockIdx.y * 64ll + lane; j < n; j += 64ll * gridDim.y) out[j] = 0;
    }
}

// The fixed-point term by a shorter route: y16 = 16 log2(e) alpha (t - sk) / (sc |x|) with the part of row and instance
// given (rate) and a reciprocal with one Newton step instead of a division, 2^(-y16 / 16) from 2^(-f/16) and a polynomial
// of degree 6.  Its relative error stays below 2^-40 (reciprocal 2^-46, rate 2^-50, times y < 20; polynomial 2^-50),
// the term is below 2^24, so the integer part is that of alns_impact_term unless the
// fraction is within 2^-15 of an integer; those (and everything out of the ordinary) are left to it: false.
__device__ __forceinline__ bool alns_impact_term_fast(double x, double rate, double base, const double* exp2m, uint32_t& term) {
    double rc = __builtin_amdgcn_rcp(x);
    rc = __builtin_fma(rc, __builtin_fma(-x, rc, 1.0), rc);
    const double y16 = rate * rc;
    const bool usual = y16 < 20.0 * 16.0 * 0x1.71547652b82fep+0;      // false for NaN
    const double kf = __builtin_rint(usual ? y16 : 0.0);
    const double z = kf - y16;                                        // |z| <= 1/2: powers of (ln 2 / 16) z
    constexpr double C = 0x1.62e42fefa39efp-5;
    double p = __builtin_fma(z, C * C * C * C * C * C / 720.0, C * C * C * C * C / 120.0);
    p = __builtin_fma(p, z, C * C * C * C / 24.0);
    p = __builtin_fma(p, z, C * C * C / 6.0);
    p = __builtin_fma(p, z, C * C / 2.0);
    p = __builtin_fma(p, z, C);
    p = __builtin_fma(p, z, 1.0);
    const int k = (int)kf;
    const double g = __builtin_ldexp(base * (p * exp2m[k & 15]), -(k >> 4));
    const double whole = __builtin_floor(g), frac = g - whole;
    term = (uint32_t)whole;
    return usual && frac > 0x1p-15 && frac < 1.0 - 0x1p-15;
}

// NARROW: at most 128 variables, whose one or two wavefronts' worth of columns leave the others rows of their own (with one of four
// wavefronts busy 500 instances of 4096 x 16 took 188 us, 125 before the queue took its LDS, 98 so).  A form of its own: in the
// other the divisors would cost scalar registers, and 1 % of the time.
template <class T, bool NARROW>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 4 : 3) void k_alns_impact_batched(int64_t m, int64_t n, int64_t R,
                                                             const T* __restrict__ Xt,
                                                             const T* __restrict__ scale_q,
                                                             const T* __restrict__ r, const T* __restrict__ lim,
                                                             const InstState<T>* st, double alpha,
                                                             uint64_t* __restrict__ weight, int64_t chunk_rows,
                                                             const int32_t* __restrict__ list,
                                                             const int32_t* __restrict__ flags) {
    __shared__ ImpactShared<T> L;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t count = flags[FLAG_WORST];                // instances on the list (k_alns_worst_list)
    const int64_t s0 = blockIdx.x * (int64_t)IM_Q;
    if (s0 >= count) return;                                // the same for the whole workgroup
    if (threadIdx.x < 16) L.exp2m[threadIdx.x] = exp2(-(double)threadIdx.x / 16.0);
    if (threadIdx.x < IM_Q) {
        const int64_t q = list[s0 + threadIdx.x < count ? s0 + threadIdx.x : count - 1];
        L.rate_q[threadIdx.x] = 0x1.71547652b82fep+4 * alpha / (double)scale_q[q];
        L.t[threadIdx.x] = (double)st[q].t;
        L.scale[threadIdx.x] = alns_impact_scale((double)st[q].t);
    }
    __syncthreads();
    const int beside = NARROW ? (n > 64 ? 2 : 1) : 4;       // wavefronts side by side
    const int64_t i_begin = (blockIdx.z * (int64_t)(4 / beside) + (NARROW ? w / beside : 0)) * chunk_rows;
    const int64_t i_end = i_begin + chunk_rows < m ? i_begin + chunk_rows : m;
    if (NARROW && i_begin >= m) return;
    // staging of r and of the limits: lane = (row, instance), two passes of 16 rows
    const int sv = lane & (IM_Q - 1), su = lane / IM_Q;
    const int64_t slot = s0 + sv, slot_c = slot < count ? slot : count - 1;
    const int64_t sq = list[slot_c];
    const int wl = threadIdx.x >> 6;                        // (in a vector register: LDS addresses are one register + constants)
    int waiting = 0;                                        // queued terms, the same in every lane
    // all queued terms of the pass at (i_pass, j_pass), 128 at a time, each for the sum it belongs to
    auto evaluate = [&](int64_t i_pass, int64_t j_pass) {
        __builtin_amdgcn_wave_barrier();
        const T* __restrict__ at = Xt + i_pass * n + j_pass;
        // (an entry is column, instance and row from the lowest bit on, which is the order of the tables: its parts are
        // their indices)
        const double* rate = &L.rate[wl][0][0];
        const double* base = &L.base[wl][0][0];
        unsigned long long* sums = &L.sum[wl][0][0];
        // two entries a lane at a time, for one's latencies to hide the other's (past the end: the last, not counted)
        for (int h = 0; h < waiting; h += 128) {
            uint32_t e[2], term[2];
            T x[2];
            bool exact[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int p = h + 64 * u + lane;
                e[u] = L.queue[wl][p < waiting ? p : waiting - 1];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) x[u] = dmmv_abs(at[(int64_t)(e[u] >> 8) * n + (e[u] & 63u)]);
#pragma unroll
            for (int u = 0; u < 2; ++u) exact[u] = alns_impact_term_fast((double)x[u], rate[e[u] >> 6], base[e[u] >> 6], L.exp2m, term[u]);
            if (!(exact[0] && exact[1])) {
#pragma unroll 1
                for (int u = 0; u < 2; ++u) {
                    const uint32_t eu = u ? e[1] : e[0];
                    const int v = (int)(eu >> 6) & (IM_Q - 1);
                    const int64_t q = list[s0 + v < count ? s0 + v : count - 1];
                    const uint32_t whole = (uint32_t)alns_impact_term(__builtin_fabs((double)scale_q[q] * (double)(u ? x[1] : x[0])),
                                                                      __builtin_fabs((double)r[(i_pass + (int)(eu >> 8)) * R + q]), L.t[v], alpha, L.scale[v]);
                    if (u) term[1] = whole; else term[0] = whole;
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (term[u] && h + 64 * u + lane < waiting) atomicAdd(&sums[e[u] & 255u], (unsigned long long)term[u]);
        }
        __builtin_amdgcn_wave_barrier();
        waiting = 0;
    };
    for (int64_t j0 = (blockIdx.y * (int64_t)beside + (NARROW ? w % beside : w)) * 64; j0 < n; j0 += 64ll * beside * gridDim.y) {   // whole wavefronts; no barrier inside
        const int64_t j = j0 + lane;
        const uint32_t lc = (uint32_t)(j < n ? lane : n - 1 - j0);
#pragma unroll
        for (int v = 0; v < IM_Q; ++v) L.sum[wl][v][lane] = 0;
        T x[IM_ROWS], rs[IM_STAGE], ls[IM_STAGE];           // the next pass's operands, in flight
        auto fetch = [&](int64_t i0) {
#pragma unroll
            for (int u = 0; u < IM_STAGE; ++u) {
                const int row = su + u * (64 / IM_Q);
                const int64_t i = i0 + row < i_end ? i0 + row : i_end - 1;
                rs[u] = r[i * R + sq];
                ls[u] = lim[i * R + slot_c];
                if (i0 + row >= i_end || slot != slot_c) ls[u] = Limits<T>::inf();
            }
            // one uniform pointer that walks; the stride is made opaque,
            // or its 32 multiples are kept in scalar registers across the whole loop, which spills them
            const T* __restrict__ row = Xt + i0 * n + j0;
            int64_t stride = n;
            asm volatile("" : "+s"(stride));
            if (i0 + IM_ROWS <= i_end) {
#pragma unroll
                for (int u = 0; u < IM_ROWS; ++u) { x[u] = row[lc]; row += stride; }
            } else {                                        // (rows past the end repeat the last)
#pragma unroll
                for (int u = 0; u < IM_ROWS; ++u) { x[u] = row[lc]; row += i0 + u + 1 < i_end ? stride : 0; }
            }
        };
        fetch(i_begin);
        for (int64_t i0 = i_begin; i0 < i_end; i0 += IM_ROWS) {
#pragma unroll
            for (int u = 0; u < IM_STAGE; ++u) {
                const double sk = __builtin_fabs((double)rs[u]);
                L.rate[wl][su + u * (64 / IM_Q)][sv] = (L.t[sv] - sk) * L.rate_q[sv];
                L.base[wl][su + u * (64 / IM_Q)][sv] = sk * L.scale[sv];
                L.lim[wl][su + u * (64 / IM_Q)][sv] = ls[u];
            }
            __builtin_amdgcn_wave_barrier();
            uint32_t mask[IM_Q];
#pragma unroll
            for (int v = 0; v < IM_Q; ++v) mask[v] = 0;
#pragma unroll
            for (int u = 0; u < IM_ROWS; ++u) {
#pragma unroll
                for (int v = 0; v < IM_Q; ++v) mask[v] = impact_test(mask[v], x[u], L.lim[wl][u][v]);
            }
            if (i0 + IM_ROWS < i_end) fetch(i0 + IM_ROWS);
            // most of the terms, in most of the variables: row by row without the queue, every lane its own
            uint32_t terms = 0;
            const uint32_t live = (uint32_t)(count - s0 < IM_Q ? count - s0 : IM_Q);      // instances of the four
#pragma unroll
            for (int v = 0; v < IM_Q; ++v) terms += __popc(mask[v]);
            if (__builtin_expect(__popcll(__ballot(j < n && terms > live * IM_DENSE)) >= 32, 0)) {
#pragma unroll 1
                for (uint32_t v = 0; v < live; ++v) {
                    const uint32_t mk = mask[0];
#pragma unroll
                    for (int e = 0; e + 1 < IM_Q; ++e) mask[e] = mask[e + 1];
                    int64_t nn = n;                         // (made opaque: nothing of this block is kept in registers for it)
                    asm volatile("" : "+s"(nn));
                    const T* __restrict__ at = Xt + i0 * nn + j0;
                    unsigned long long sum = 0;
#pragma unroll 1
                    for (int row = 0; row < IM_ROWS && i0 + row < i_end; row += 2) {
                        T y[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) y[u] = dmmv_abs(at[(int64_t)(i0 + row + u < i_end ? row + u : row) * nn + lc]);
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const bool on = j < n && ((mk << (row + u)) & 0x80000000u) != 0;
                            uint32_t term;
                            const bool exact = alns_impact_term_fast((double)y[u], L.rate[wl][row + u][v], L.base[wl][row + u][v], L.exp2m, term);
                            const unsigned long long odd = __ballot(on && !exact);      // (rare: by the queue, which knows how)
                            if (odd != 0ull) {
                                if (on && !exact)
                                    L.queue[wl][waiting + __builtin_amdgcn_mbcnt_hi((uint32_t)(odd >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)odd, 0))] = (uint16_t)(lane | (v << 6) | ((row + u) << 8));
                                waiting += __popcll(odd);
                            }
                            if (on && exact) sum += term;
                        }
                    }
                    if (sum) atomicAdd(&L.sum[wl][v][lane], sum);
                    if (waiting > IM_CAP - IM_MOST) evaluate(i0, j0);
                }
                if (waiting > 0) evaluate(i0, j0);
                continue;
            }
            // (the entries of X and r are replaced after the pass: the queue is emptied with its last instance)
#pragma unroll 1
            for (int v = 0;; ++v) {
                if (waiting > IM_CAP - IM_MOST || v == IM_Q) {
                    evaluate(i0, j0);
                    if (v == IM_Q) break;
                }
                uint32_t mk = j < n ? mask[0] : 0;          // highest bit = first row
#pragma unroll
                for (int e = 0; e + 1 < IM_Q; ++e) mask[e] = mask[e + 1];
                unsigned long long many = __ballot(__popc(mk) > IM_FEW);
                // a variable with many terms (an outlier channel): all its rows at once, lane = row
                while (many) {                              // the same for the whole wavefront
                    const int col = __ffsll(many) - 1;
                    many &= many - 1;
                    const uint32_t rows = __brev(__builtin_amdgcn_readlane(mk, col));
                    if (lane == col) mk = 0;
                    if (lane < IM_ROWS && ((rows >> lane) & 1u))
                        L.queue[wl][waiting + __builtin_amdgcn_mbcnt_lo(rows, 0)] = (uint16_t)(col | (v << 6) | (lane << 8));
                    waiting += __popc(rows);
                }
                // the others: a lane's rows one after the other, behind those of the lanes before it
                const uint32_t mine = __popc(mk), upto = wave_scan(mine);
                int at = waiting + (int)(upto - mine);
                waiting += (int)__builtin_amdgcn_readlane(upto, 63);
                while (__ballot(mk != 0) != 0ull) {
                    if (mk) {
                        const int row = __clz(mk);
                        L.queue[wl][at++] = (uint16_t)(lane | (v << 6) | (row << 8));
                        mk ^= 0x80000000u >> row;
                    }
                }
            }
        }
        if (j < n) {
#pragma unroll
            for (int v = 0; v < IM_Q; ++v)
                if (s0 + v < count && L.sum[wl][v][lane] != 0)
                    atomicAdd((unsigned long long*)&weight[(int64_t)list[s0 + v] * n + j], L.sum[wl][v][lane]);
        }
    }
}

// one workgroup per instance; thread i owns the rows i, i + blockDim.x, ...; the picked
// variables are reassigned one after the other, r follows each reassignment.  STAGE: the
// instance's r is copied to LDS first and written back at the end (in a batch its rows lie R
// elements apart in memory, and every picked variable would walk them again).
constexpr int RD_UNROLL = 8;                   // independent global loads a thread issues before it uses them
constexpr size_t RD_STAGE_BYTES = 48 * 1024;   // largest r that is staged

template <class T, bool STAGE>
__global__ __launch_bounds__(1024) void k_alns_repair_dense(int64_t m, int64_t R, int32_t nd,
                                                            const T* __restrict__ A, int64_t lda,
                                                            const T* __restrict__ D,
                                                            const T* __restrict__ scale_q, T* r,
                                                            int32_t* kidx, int32_t count,
                                                            const int32_t* __restrict__ picked_all,
                                                            InstState<T>* st, const AlnsState* S,
                                                            uint64_t seed) {
    extern __shared__ __align__(16) unsigned char repair_smem[];
    T* lr = reinterpret_cast<T*>(repair_smem);
    __shared__ T sh[16];
    const int64_t q = blockIdx.x;
    const int64_t nt = blockDim.x;
    const int32_t* __restrict__ picked = picked_all + q * (int64_t)count;
    const int32_t it = S[q].it;
    const bool greedy = S[q].r_op == 1;
    const T sc = scale_q[q];
    if (STAGE) {
        for (int64_t i0 = threadIdx.x; i0 < m; i0 += nt * RD_UNROLL) {
            T v[RD_UNROLL];
#pragma unroll
            for (int u = 0; u < RD_UNROLL; ++u) {
                const int64_t i = i0 + nt * u;
                v[u] = r[(i < m ? i : m - 1) * R + q];
            }
#pragma unroll
            for (int u = 0; u < RD_UNROLL; ++u) {
                const int64_t i = i0 + nt * u;
                if (i < m) lr[i] = v[u];
            }
        }
        __syncthreads();
    }
    // thread i touches only its own rows of r between barriers, staged or not
    auto rd = [&](int64_t i) -> T { return STAGE ? lr[i] : r[i * R + q]; };
    auto wr = [&](int64_t i, T v) { if (STAGE) lr[i] = v; else r[i * R + q] = v; };
    for (int32_t pos = 0; pos < count; ++pos) {
        const int64_t j = picked[pos];
        const int32_t kc = kidx[j * R + q];
        const bool has_lo = kc > 0, has_hi = kc < nd - 1;
        const T* __restrict__ col = A + lda * j;
        int32_t knew;
        if (has_lo && has_hi) {
            if (greedy) {
                const T dlo = step_of(D[kc - 1], D[kc], sc), dhi = step_of(D[kc + 1], D[kc], sc);
                T elo = (T)0, ehi = (T)0;
                for (int64_t i0 = threadIdx.x; i0 < m; i0 += nt * RD_UNROLL) {
                    T a[RD_UNROLL];
#pragma unroll
                    for (int u = 0; u < RD_UNROLL; ++u) {
                        const int64_t i = i0 + nt * u;
                        a[u] = col[i < m ? i : m - 1];
                    }
#pragma unroll
                    for (int u = 0; u < RD_UNROLL; ++u) {
                        const int64_t i = i0 + nt * u;
                        if (i < m) {
                            const T ri = rd(i);
                            elo = dmmv_max(elo, dmmv_abs(dmmv_fma(dlo, a[u], ri)));
                            ehi = dmmv_max(ehi, dmmv_abs(dmmv_fma(dhi, a[u], ri)));
                        }
                    }
                }
                elo = block_max(elo, sh);
                ehi = block_max(ehi, sh);
                knew = ehi < elo ? kc + 1 : kc - 1;
            } else {
                knew = (alns_rnd(seed, (uint64_t)q, (uint64_t)it, 2, (uint64_t)pos) & 1) ? kc + 1 : kc - 1;
            }
        } else {
            knew = has_lo ? kc - 1 : kc + 1;
        }
        const T delta = step_of(D[knew], D[kc], sc);
        for (int64_t i0 = threadIdx.x; i0 < m; i0 += nt * RD_UNROLL) {
            T a[RD_UNROLL];
#pragma unroll
            for (int u = 0; u < RD_UNROLL; ++u) {
                const int64_t i = i0 + nt * u;
                a[u] = col[i < m ? i : m - 1];
            }
#pragma unroll
            for (int u = 0; u < RD_UNROLL; ++u) {
                const int64_t i = i0 + nt * u;
                if (i < m) wr(i, dmmv_fma(delta, a[u], rd(i)));
            }
        }
        __syncthreads();                      // every thread has read kidx of this step
        if (threadIdx.x == 0) kidx[j * R + q] = knew;
    }
    T tmax = (T)0;
    for (int64_t i = threadIdx.x; i < m; i += nt) {
        const T v = rd(i);
        tmax = dmmv_max(tmax, dmmv_abs(v));
        if (STAGE) r[i * R + q] = v;
    }
    tmax = block_max(tmax, sh);
    if (threadIdx.x == 0) { st[q].t = tmax; st[q].done = 0; st[q].moves = 0; }
}

// ----------------------------------------------------------------------------------------
// host side: one outer iteration's kernels around the local search
// ----------------------------------------------------------------------------------------
static unsigned blocks_for(int64_t items, int per_block) {
    int64_t b = (items + per_block - 1) / per_block;
    return (unsigned)(b < 1 ? 1 : b);
}

template <class T>
static dmmv_status sumsq_t(Ctx* c) {
    const int64_t R = c->p.R;
    if (c->kind == KIND_BATCHED)
        hipLaunchKernelGGL(k_alns_sumsq_batched<T>, dim3(blocks_for(R, 64)), dim3(64), 0, c->stream, c->p.m, R,
                           (const T*)c->r, c->alns_q2);
    else
        hipLaunchKernelGGL(k_alns_sumsq_single<T>, dim3(1), dim3(1024), 0, c->stream, c->p.m, (const T*)c->r,
                           c->alns_q2_blocks, c->alns_q2);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
static dmmv_status start_t(Ctx* c, bool l2_guard, uint64_t seed) {
    const int64_t R = c->p.R;
    if (l2_guard) DMMV_TRY(sumsq_t<T>(c));
    hipLaunchKernelGGL(k_alns_init<T>, dim3(blocks_for(R, 256)), dim3(256), 0, c->stream,
                       (AlnsState*)c->alns_state, (const InstState<T>*)c->state, R,
                       l2_guard ? (const double*)c->alns_q2 : nullptr, seed);
    hipLaunchKernelGGL(k_alns_snapshot<T>, dim3(1024), dim3(256), 0, c->stream, c->p.m, c->p.n, R,
                       (const int32_t*)c->kidx, c->alns_kidx_cur, c->alns_kidx_best, (const T*)c->r,
                       (T*)c->alns_r_cur, (unsigned long long*)c->alns_first, c->alns_weight);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
static dmmv_status destroy_repair_t(Ctx* c, const dmmv_alns_params& prm, int32_t count) {
    AlnsState* S = (AlnsState*)c->alns_state;
    const int64_t R = c->p.R;
    if (c->kind == KIND_DENSE) {
        hipLaunchKernelGGL(k_alns_impact_dense<T>, dim3((unsigned)c->p.n), dim3(256), 0, c->stream, c->p.m,
                           c->p.n, (const T*)c->p.A_dense, c->p.lda, (const T*)c->r,
                           (const InstState<T>*)c->state, prm.alpha, c->alns_weight, (const AlnsState*)S);
    } else if (c->kind == KIND_BATCHED && c->alns_lists) {
        DMMV_TRY(alns_impact_lists(c, prm.alpha));
    } else if (c->kind == KIND_BATCHED) {
        // (the list shares the buffer of the descent's list of running instances, the limits that of its
        // packed residuals: never both at once)
        hipLaunchKernelGGL(k_alns_worst_list, dim3(1), dim3(1024), 0, c->stream, R, (const AlnsState*)S,
                           c->cmp_orig, c->flags);
        int64_t ly = ceil_div(c->p.m, 16);
        if (ly > 64) ly = 64;
        hipLaunchKernelGGL(k_alns_impact_limits<T>, dim3(blocks_for(R, 64), (unsigned)(ly > 0 ? ly : 1)), dim3(256), 0,
                           c->stream, c->p.m, c->p.n, R, (const T*)c->scale_dev, (const T*)c->r,
                           (const InstState<T>*)c->state, prm.alpha, (T*)c->cmp_r, c->alns_weight,
                           (const int32_t*)c->cmp_orig, (const int32_t*)c->flags);
        // about half of the instances are on the list; the rows are split until some 8 wavefronts per SIMD
        // are there to hide the loads of each other, at least one pass of rows each
        const int64_t beside = c->p.n > 128 ? 4 : c->p.n > 64 ? 2 : 1;     // (as in the kernel: the others take rows of their own)
        const int64_t col_groups = ceil_div(c->p.n, 64 * beside);
        const int64_t waves = ceil_div(c->p.n, 64) * ceil_div(ceil_div(R, 2), IM_Q);
        int64_t chunks = ceil_div(8192, waves > 0 ? waves : 1);
        if (chunks > ceil_div(c->p.m, IM_ROWS)) chunks = ceil_div(c->p.m, IM_ROWS);
        if (chunks < 1) chunks = 1;
        const int64_t chunk_rows = ceil_div(ceil_div(c->p.m, chunks), IM_ROWS) * IM_ROWS;
        chunks = ceil_div(c->p.m, chunk_rows > 0 ? chunk_rows : 1);
        if (chunks > 0)
            hipLaunchKernelGGL((beside < 4 ? k_alns_impact_batched<T, true> : k_alns_impact_batched<T, false>), dim3((unsigned)ceil_div(R, IM_Q), (unsigned)(col_groups < 65535 ? col_groups : 65535), (unsigned)ceil_div(chunks, 4 / beside)),
                               dim3(256), 0, c->stream, c->p.m, c->p.n, R, (const T*)c->Xt, (const T*)c->scale_dev,
                               (const T*)c->r, (const T*)c->cmp_r, (const InstState<T>*)c->state, prm.alpha, c->alns_weight,
                               chunk_rows, (const int32_t*)c->cmp_orig, (const int32_t*)c->flags);
    } else {
        DMMV_TRY(csc_alns_impact(c, prm.alpha));
    }
    int32_t raw_shift = -1;
    if (c->kind == KIND_BATCHED) {
        auto bits = [](int64_t v) { int b = 0; while (v > 0) { ++b; v >>= 1; } return b; };
        raw_shift = bits(c->p.m) + 24 + bits(c->p.n) - 62;
        if (raw_shift < 0) raw_shift = 0;
    }
    const int32_t clear = c->kind == KIND_BATCHED && c->alns_lists ? 1 : 0;
    c->exchange_clear = false;
    // One launch for up to 4096 rows, or 8192 where the instances do not fill the chip.  256 threads as long as these hold the rows: more of
    // them wait for each other longer, and keep other instances out.  us of whole calls with 256 and 1024 threads (three launches, in
    // brackets): 400 instances of 64 x 64, 30 iterations 2668 and 3037 (2887), 400 of 1000 x 200, 20, 2523 and 2747 (3567), 20 of 2000 x 768,
    // 20, 1488 and 1527 (1904), 300 of 2500 x 200 in fp64, 10, 2954 and 3114 (2971), one of 2000 x 500, 20, 834 and 871 (1086).
    if (c->kind != KIND_CSC && c->p.m <= (R > 512 ? 256 * 16 : 1024 * 8)) {
        auto both = [&](auto kernel, int threads) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)R), dim3(threads), 0, c->stream, c->p.m, c->p.n, R, c->p.nd, count,
                               c->alns_weight, c->alns_prefix, (unsigned long long*)c->alns_first, c->alns_picked,
                               (const AlnsState*)S, prm.seed, raw_shift, clear, (const T*)c->p.A_dense, c->p.lda,
                               (const T*)c->D_dev, (const T*)c->scale_dev, (T*)c->r, c->kidx, (InstState<T>*)c->state,
                               (uint32_t*)c->persist_exchange, c->kind == KIND_DENSE ? (int32_t)(dense_persistent_exchange_bytes() / 4) : 0);
        };
        if (c->p.m <= 256 * 8) both(k_alns_destroy_repair<T, 256, 8>, 256);
        else if (c->p.m <= 256 * 16) both(k_alns_destroy_repair<T, 256, 16>, 256);
        else both(k_alns_destroy_repair<T, 1024, 8>, 1024);
        DMMV_LAUNCH_CHECK();
        c->exchange_clear = c->kind == KIND_DENSE;
        return DMMV_OK;
    }
    const bool alone = R == 1;
    hipLaunchKernelGGL((alone ? k_alns_destroy<1024> : k_alns_destroy<256>), dim3((unsigned)R), dim3(alone ? 1024 : 256), 0, c->stream, c->p.n,
                       count, c->alns_weight, c->alns_prefix, (unsigned long long*)c->alns_first, c->alns_picked, (const AlnsState*)S, prm.seed, raw_shift, clear);
    if (c->kind == KIND_CSC) {
        DMMV_TRY(csc_alns_repair(c, count, prm.seed));
    } else {
        const size_t rbytes = (size_t)c->p.m * sizeof(T);
        const bool stage = rbytes <= RD_STAGE_BYTES;
        auto repair = stage ? k_alns_repair_dense<T, true> : k_alns_repair_dense<T, false>;
        hipLaunchKernelGGL(repair, dim3((unsigned)R), dim3(R > 1 ? 256 : 1024), stage ? rbytes : 0, c->stream,
                           c->p.m, R, c->p.nd, (const T*)c->p.A_dense, c->p.lda, (const T*)c->D_dev,
                           (const T*)c->scale_dev, (T*)c->r, c->kidx, count, (const int32_t*)c->alns_picked,
                           (InstState<T>*)c->state, (const AlnsState*)S, prm.seed);
    }
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
static dmmv_status finish_iteration_t(Ctx* c, const dmmv_alns_params& prm, int32_t next, int32_t* trace, void* trace_t) {
    const int64_t R = c->p.R, m = c->p.m, n = c->p.n;
    if (prm.l2_guard) DMMV_TRY(sumsq_t<T>(c));
    // some sixteen elements a thread, more where that takes over 1024 workgroups (us with 512, 1024, 2048 of them: 1024 instances of
    // 2048 x 4096 27.6, 27.8, 28.9; 11 008 of 2048 x 256 97.7, 90.7, 91.3)
    constexpr int64_t cap = 1024;
    int64_t strips = ceil_div(R > 1 ? R : ceil_div(m + n, 4), 256), rows = R > 1 ? ceil_div(m + n, 16) : 1;
    if (R == 1 && strips > 1024) strips = 1024;
    if (rows > ceil_div(cap, strips)) rows = ceil_div(cap, strips);
    hipLaunchKernelGGL(k_alns_turn<T>, dim3((unsigned)strips, (unsigned)rows), dim3(256), 0, c->stream, m, n, R,
                       (AlnsState*)c->alns_state, (InstState<T>*)c->state, c->kidx, c->alns_kidx_cur, c->alns_kidx_best, (T*)c->r,
                       (T*)c->alns_r_cur, prm.iters, prm.lambda, prm.sigma1, prm.sigma2, prm.sigma3,
                       prm.l2_guard ? (const double*)c->alns_q2 : nullptr, trace, (T*)trace_t, prm.seed, next);
    DMMV_LAUNCH_CHECK();
    // (before another iteration, its repair gives what it leaves a reservoir of its own)
    if (c->kind == KIND_CSC && next < 0) DMMV_TRY(csc_alns_after_copy(c));
    return DMMV_OK;
}

template <class T>
static dmmv_status export_t(Ctx* c, void* t_best_out) {
    hipLaunchKernelGGL(k_alns_export<T>, dim3(blocks_for(c->p.R, 256)), dim3(256), 0, c->stream,
                       (const AlnsState*)c->alns_state, c->p.R, (T*)t_best_out);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

dmmv_status alns_start(Ctx* c, bool l2_guard, uint64_t seed) {
    return c->p.dtype == DMMV_F64 ? start_t<double>(c, l2_guard, seed) : start_t<float>(c, l2_guard, seed);
}
dmmv_status alns_sumsq(Ctx* c) { return c->p.dtype == DMMV_F64 ? sumsq_t<double>(c) : sumsq_t<float>(c); }
dmmv_status alns_destroy_repair(Ctx* c, const dmmv_alns_params& prm, int32_t count) {
    return c->p.dtype == DMMV_F64 ? destroy_repair_t<double>(c, prm, count) : destroy_repair_t<float>(c, prm, count);
}
dmmv_status alns_finish_iteration(Ctx* c, const dmmv_alns_params& prm, int32_t next, int32_t* trace, void* trace_t) {
    return c->p.dtype == DMMV_F64 ? finish_iteration_t<double>(c, prm, next, trace, trace_t)
                                  : finish_iteration_t<float>(c, prm, next, trace, trace_t);
}
dmmv_status alns_export(Ctx* c, void* t_best_out) {
    return c->p.dtype == DMMV_F64 ? export_t<double>(c, t_best_out) : export_t<float>(c, t_best_out);
}

}  // namespace dmmv
