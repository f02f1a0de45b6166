// Dense single instance, small enough that a launch per step costs more than the step: the
// whole descent (score every move, pick the best, apply it, repeat) in ONE launch.
//
// The moves are cut into units of one variable x DP_KT values of D.  A fixed grid of G
// workgroups shares the units; a workgroup keeps its own copy of r, the columns of A its units
// need and the current indices k_j in LDS for the whole call.  Per iteration it scores its
// units (same arithmetic as the evaluation kernel: |fma(delta, A_ij, r_i)|, maximum over the
// rows), publishes one (score, move) record, reads the records of all workgroups and takes
// their minimum - every workgroup arrives at the same move - and applies it to its own r.  One
// exchange per iteration is the only communication; r is never written to memory before the end.
//
// A record travels as four 64-bit words, each carrying the iteration number in its upper half and
// 32 bits of (score, move index) in its lower half.  Every word is written and read with one
// atomic access and names its own iteration, so the writer needs no ordering between its stores
// and a reader needs no separate arrival flag: it polls the four words until all name the
// iteration it is in (one round trip through the L2 instead of two).  Slots alternate with the
// parity of the iteration; a workgroup can be at most one iteration ahead of the slowest, so a
// slot is never overwritten while somebody still waits for it.
//
// The exchange is a wait on other workgroups, so all G must be resident at once (G never
// exceeds the number of compute units, and each needs at most one unit's LDS).  Should the
// device be shared with a kernel of another process that keeps some of them from starting, the wait ends
// after options.wait_limit polls: the kernel raises an error flag, every workgroup leaves, and
// dmmv_solve returns DMMV_ERR_STATE.
#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <mutex>
#include <type_traits>

#include "dmmv_common.h"

namespace dmmv {

constexpr int DP_KT = 16;                 // values of D per unit
constexpr int DP_MAX_WAVES = 8;            // wavefronts per workgroup: 4 (one per SIMD) or 8, chosen with the grid
constexpr int DP_MAX_THREADS = 64 * DP_MAX_WAVES;
constexpr int DP_SKEW = 65;               // row stride of the per-wavefront transpose scratch
constexpr int DP_MAX_G = 256;
constexpr size_t DP_LDS_LIMIT = 156 * 1024;
constexpr int32_t DP_WAIT_DEFAULT = 1 << 22;
// The loop of launches, for the automatic choice: its two launches take 8.1 us before any work
// is done, and the chip-wide evaluation kernel then needs about 81 ns per million (row, move)
// pairs in fp64 and 40 in fp32 (fitted to the measured iterations of small and large instances).
constexpr double DP_LAUNCH_LOOP_US = 8.1;
constexpr double DP_LAUNCH_LOOP_US_PER_PAIR_F64 = 8.1e-8, DP_LAUNCH_LOOP_US_PER_PAIR_F32 = 4.0e-8;

constexpr int DP_REC_WORDS = 4;
size_t dense_persistent_exchange_bytes() { return (size_t)2 * DP_MAX_G * DP_REC_WORDS * sizeof(uint64_t); }

namespace {

struct Plan {
    int G = 0;            // workgroups (0: not applicable)
    int upw = 0;          // units per workgroup
    int ncols = 0;        // columns of A a workgroup keeps in LDS
    int waves = 0;        // wavefronts per workgroup
    size_t lds = 0;
    double est_us = 0;    // modelled time of one iteration
};

// Picks the grid and the workgroup size: more workgroups shorten the scoring and lengthen the
// exchange; eight wavefronts per workgroup instead of four put two on every SIMD, which share its
// arithmetic but hide each other's latencies (better when a wavefront would otherwise take
// several units in a row, worse for a single short unit).  Measured on MI355X: the exchange
// takes about 2 us + 4 ns per workgroup, the rest of an iteration outside the scoring 1.6 us;
// 64 (row, move) pairs cost a wavefront about 18 cycles in fp64 (the maximum is not a full-rate
// instruction) and 10 in fp32 when it has its SIMD to itself, 32 and 16 when it shares it; the
// reduction of a unit's 16 x 64 lane maxima about 400.
Plan make_plan(const dmmv_problem& p, int cus) {
    Plan best;
    if (p.csr_rowptr || p.R != 1 || p.scale || p.m < 1 || p.n < 1 || p.nd < 1) return best;
    const size_t w = p.dtype == DMMV_F64 ? 8 : 4;
    const int64_t tiles = ceil_div(p.nd, DP_KT);
    const int64_t U = p.n * tiles;
    if (p.m > (int64_t)(DP_LDS_LIMIT / w) || p.n > (1 << 20) || p.nd > (1 << 16)) return best;
    const int gmax = cus < DP_MAX_G ? (cus > 0 ? cus : 1) : DP_MAX_G;
    for (int waves = 4; waves <= DP_MAX_WAVES; waves *= 2) {
        for (int want = 1;; want = want * 2 < gmax ? want * 2 : gmax) {
            const int64_t upw = ceil_div(U, want);
            const int64_t G = ceil_div(U, upw);
            int64_t ncols = 1;
            for (int64_t g = 0; g < G; ++g) {
                const int64_t u0 = g * upw, u1 = (g + 1) * upw < U ? (g + 1) * upw : U;
                const int64_t span = (u1 - 1) / tiles - u0 / tiles + 1;
                if (span > ncols) ncols = span;
            }
            const size_t lds = (size_t)(1 + ncols) * p.m * w + (size_t)waves * DP_KT * DP_SKEW * w + (size_t)p.nd * w +
                               (size_t)p.n * 4;
            if (lds <= DP_LDS_LIMIT) {
                const double per_64 = waves == 4 ? (w == 8 ? 18.0 : 10.0) : (w == 8 ? 32.0 : 16.0);
                const double per_unit = (double)ceil_div(p.m, 64) * DP_KT * per_64 + 400.0;     // cycles
                const double est = 2.0 + 0.004 * (double)G + (double)ceil_div(upw, waves) * per_unit / 2400.0 + 1.6;
                if (best.G == 0 || est < best.est_us) {
                    best.G = (int)G; best.upw = (int)upw; best.ncols = (int)ncols; best.waves = waves; best.lds = lds;
                    best.est_us = est;
                }
            }
            if (want == gmax) break;
        }
    }
    return best;
}

int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cus;
}

__device__ __forceinline__ uint64_t score_bits(double s) { return (uint64_t)__double_as_longlong(s); }
__device__ __forceinline__ uint64_t score_bits(float s) { return (uint64_t)__float_as_uint(s); }
__device__ __forceinline__ void score_from(uint64_t b, double& s) { s = __longlong_as_double((long long)b); }
__device__ __forceinline__ void score_from(uint64_t b, float& s) { s = __uint_as_float((uint32_t)b); }

// ---- the exchange ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ void dp_publish(uint64_t* rec, int G, int g, int32_t it, T bs, int64_t bc) {
    const uint64_t tag = (uint64_t)(uint32_t)(it + 1) << 32;
    uint64_t* slot = rec + ((int64_t)(it & 1) * G + g) * DP_REC_WORDS;
    const uint64_t sb = score_bits(bs), cb = (uint64_t)bc;
    __hip_atomic_store(&slot[0], tag | (sb >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&slot[1], tag | (sb & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&slot[2], tag | (cb >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&slot[3], tag | (cb & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One whole wavefront: the smallest of all workgroups' records of iteration `it`, the same in every
// lane (lane q waits for workgroups q, q + 64, ..).  False when a wait ran into its limit.
template <class T>
__device__ __forceinline__ bool dp_collect(const uint64_t* rec, int G, int32_t it, int lane, int32_t wait_limit,
                                           const int32_t* flags, T& gs, int64_t& gc) {
    const uint64_t tag = (uint64_t)(uint32_t)(it + 1) << 32;
    gs = (T)0;
    gc = -1;
    uint32_t fail = 0;
    for (int q = lane; q < G; q += 64) {
        const uint64_t* slot = rec + ((int64_t)(it & 1) * G + q) * DP_REC_WORDS;
        // Two reads of the record are kept in flight (loads return in order): a read
        // samples memory half a round trip after it was issued, so with one read at a
        // time a record that lands just after the sample costs a whole further round
        // trip; the second read halves that.
        const uint64_t hi = 0xffffffff00000000ull;
        uint64_t a0, a1, a2, a3, b0, b1, b2, b3;
#define DP_READ(x0, x1, x2, x3)                                                              \
    x0 = __hip_atomic_load(&slot[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);             \
    x1 = __hip_atomic_load(&slot[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);             \
    x2 = __hip_atomic_load(&slot[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);             \
    x3 = __hip_atomic_load(&slot[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#define DP_THERE(x0, x1, x2, x3) (((x0) & hi) == tag && ((x1) & hi) == tag && ((x2) & hi) == tag && ((x3) & hi) == tag)
        int32_t polls = 0;
        bool there = false;
        DP_READ(a0, a1, a2, a3)
        do {
            DP_READ(b0, b1, b2, b3)
            there = DP_THERE(a0, a1, a2, a3);
            if (there) break;
            DP_READ(a0, a1, a2, a3)
            there = DP_THERE(b0, b1, b2, b3);
            if (there) { a0 = b0; a1 = b1; a2 = b2; a3 = b3; break; }
            polls += 2;
            // somebody else has given up already: no point in waiting out the limit
            if ((polls & 254) == 254 &&
                __hip_atomic_load(&flags[FLAG_ERROR], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
                polls = wait_limit;
        } while (polls < wait_limit);
#undef DP_READ
#undef DP_THERE
        if (!there) { fail = 1; break; }
        T s;
        score_from((a0 << 32) | (a1 & 0xffffffffull), s);
        const int64_t c = (int64_t)((a2 << 32) | (a3 & 0xffffffffull));
        if (rec_less(s, c, gs, gc)) { gs = s; gc = c; }
    }
    wave_argmin(gs, gc);
    return __ballot(fail != 0) == 0ull;
}

__global__ void k_zero_words(uint32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

template <class T, int NWAVES>
__global__ __launch_bounds__(64 * NWAVES) void k_descent_dense_persistent(
    int64_t m, int64_t n, int32_t nd, const T* __restrict__ A, int64_t lda, const T* __restrict__ D,
    T* r, int32_t* kidx, int32_t radius, const uint8_t* __restrict__ var_mask, InstState<T>* st,
    int32_t keep_going, int32_t steps, int32_t iters, dmmv_move* trace, T* trace_t, int32_t tiles, int32_t upw,
    int32_t ncols, uint64_t* rec /*[2][G][DP_REC_WORDS]*/, int32_t* flags, int32_t wait_limit) {
    constexpr int KT = DP_KT;
    extern __shared__ __align__(16) unsigned char smem[];
    T* sh_r = reinterpret_cast<T*>(smem);                   // [m]
    T* sh_cols = sh_r + m;                                  // [ncols][m]
    constexpr int nthreads = 64 * NWAVES, nwaves = NWAVES;
    T* sh_sc = sh_cols + (int64_t)ncols * m;                // [nwaves][KT * DP_SKEW]
    T* sh_D = sh_sc + nwaves * KT * DP_SKEW;                // [nd]
    int32_t* sh_kidx = reinterpret_cast<int32_t*>(sh_D + nd);   // [n]
    __shared__ T sh_ws[NWAVES];
    __shared__ int64_t sh_wc[NWAVES];
    __shared__ T sh_bs;
    __shared__ int64_t sh_bc;
    __shared__ int32_t sh_fail;

    const int G = gridDim.x, g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t U = n * tiles;
    const int64_t u0 = (int64_t)g * upw, u1 = u0 + upw < U ? u0 + upw : U;
    const int64_t j_lo = u0 / tiles, j_hi = (u1 - 1) / tiles;

    for (int64_t i = tid; i < m; i += nthreads) sh_r[i] = r[i];
    for (int64_t j = j_lo; j <= j_hi; ++j)
        for (int64_t i = tid; i < m; i += nthreads) sh_cols[(j - j_lo) * m + i] = A[lda * j + i];
    for (int64_t j = tid; j < n; j += nthreads) sh_kidx[j] = kidx[j];
    for (int32_t k = tid; k < nd; k += nthreads) sh_D[k] = D[k];
    if (tid == 0) sh_fail = 0;
    T t = st[0].t;
    int32_t moves = st[0].moves;
    T last_s = st[0].best_s;
    bool stopped = st[0].done != 0, failed = false;
    __syncthreads();

    // A wavefront with a single unit keeps that unit's level index and steps in registers; they
    // change only when a move lands on its variable (the chain level index -> levels -> steps is
    // three LDS latencies that nothing hides with one wavefront per SIMD).
    const bool one_unit = upw <= nwaves;
    bool steps_stale = true;
    int32_t kcur_keep = 0;
    T delta_keep[KT];
#pragma unroll
    for (int q = 0; q < KT; ++q) delta_keep[q] = (T)0;

    for (int32_t it = 0; it < steps && !stopped; ++it) {
        // ---- score this wavefront's units ------------------------------------------------
        T ws = (T)0;
        int64_t wc = -1;
        for (int64_t u = u0 + w; u < u1; u += nwaves) {
            const int64_t j = u / tiles;
            const int32_t kbase = (int32_t)(u % tiles) * KT;
            const T* __restrict__ col = sh_cols + (j - j_lo) * m;
            T delta[KT], acc[KT];
            int32_t kcur;
            if (!one_unit || steps_stale) {
                kcur = sh_kidx[j];
                const T dcur = sh_D[kcur];
#pragma unroll
                for (int q = 0; q < KT; ++q) {
                    const int32_t k = kbase + q < nd ? kbase + q : nd - 1;
                    delta[q] = step_of(sh_D[k], dcur, (T)1);
                }
                if (one_unit) {
                    kcur_keep = kcur;
#pragma unroll
                    for (int q = 0; q < KT; ++q) delta_keep[q] = delta[q];
                    steps_stale = false;
                }
            } else {
                kcur = kcur_keep;
#pragma unroll
                for (int q = 0; q < KT; ++q) delta[q] = delta_keep[q];
            }
#pragma unroll
            for (int q = 0; q < KT; ++q) acc[q] = (T)0;
            // two rows per pass, both requested before the first is used (a row past the end
            // is replaced by the pass's first row: a maximum does not mind the repeat)
            for (int64_t i = lane; i < m; i += 128) {
                const int64_t i2 = i + 64 < m ? i + 64 : i;
                const T a = col[i], ri = sh_r[i], a2 = col[i2], ri2 = sh_r[i2];
#pragma unroll
                for (int q = 0; q < KT; ++q) acc[q] = dmmv_max(acc[q], dmmv_abs(dmmv_fma(delta[q], a, ri)));
#pragma unroll
                for (int q = 0; q < KT; ++q) acc[q] = dmmv_max(acc[q], dmmv_abs(dmmv_fma(delta[q], a2, ri2)));
            }
            // 16 x 64 lane maxima -> 16 scores: lane folds a quarter of value lane / 4, two DPP steps join
            T* sc = sh_sc + w * KT * DP_SKEW;
#pragma unroll
            for (int q = 0; q < KT; ++q) sc[q * DP_SKEW + lane] = acc[q];
            __builtin_amdgcn_wave_barrier();
            const int q = lane >> 2, quarter = lane & 3;
            T v = (T)0;
#pragma unroll
            for (int e = 0; e < 16; ++e) v = dmmv_max(v, sc[q * DP_SKEW + quarter * 16 + e]);
            __builtin_amdgcn_wave_barrier();
            v = dmmv_max(v, dpp_mov<DPP_QUAD_XOR1>(v));
            v = dmmv_max(v, dpp_mov<DPP_QUAD_XOR2>(v));
            // the unit's candidates sit in lanes 0, 4, 8, ... in ascending k: the smallest score,
            // then the first lane that holds it
            const int32_t k = kbase + q;
            const bool cand = quarter == 0 && k < nd;
            T cs = Limits<T>::inf();
            if (cand) {
                const bool var_ok = var_mask ? var_mask[j] != 0 : true;
                if (cand_allowed(kcur, k, radius, var_ok)) cs = v;
            }
            const T smin = wave_min(cs);
            const unsigned long long hit = __ballot(cand && cs == smin);
            if (hit) {
                const int64_t cc = j * (int64_t)nd + kbase + (__builtin_ctzll(hit) >> 2);
                if (rec_less(smin, cc, ws, wc)) { ws = smin; wc = cc; }
            }
        }
        if (lane == 0) { sh_ws[w] = ws; sh_wc[w] = wc; }
        __syncthreads();
        // ---- publish this workgroup's record, read every workgroup's ---------------------------
        if (tid == 0) {
            T bs = (T)0;
            int64_t bc = -1;
            T xs[NWAVES];
            int64_t xc[NWAVES];
#pragma unroll
            for (int x = 0; x < NWAVES; ++x) { xs[x] = sh_ws[x]; xc[x] = sh_wc[x]; }
#pragma unroll
            for (int x = 0; x < NWAVES; ++x)
                if (rec_less(xs[x], xc[x], bs, bc)) { bs = xs[x]; bc = xc[x]; }
            dp_publish(rec, G, g, it, bs, bc);
        }
        if (w == 0) {
            T gs;
            int64_t gc;
            const bool fail = !dp_collect(rec, G, it, lane, wait_limit, flags, gs, gc);
            if (lane == 0) {
                sh_bs = gs;
                sh_bc = gc;
                if (fail) { sh_fail = 1; atomicOr(&flags[FLAG_ERROR], ERRBIT_WAIT_LIMIT); }
            }
        }
        __syncthreads();
        if (sh_fail) { failed = true; break; }
        // ---- the same decision in every workgroup ------------------------------------------
        const T s = sh_bs;
        const int64_t c = sh_bc;
        last_s = s;
        if (c >= 0 && s < t) {
            const int32_t j = (int32_t)(c / nd), k = (int32_t)(c % nd);
            const T delta = step_of(sh_D[k], sh_D[sh_kidx[j]], (T)1);
            if (g == 0 && tid == 0 && moves < iters) {
                if (trace) { trace[moves].j = j; trace[moves].k = k; }
                if (trace_t) trace_t[moves] = s;
            }
            const T* __restrict__ colg = A + lda * (int64_t)j;
            for (int64_t i = tid; i < m; i += nthreads) sh_r[i] = dmmv_fma(delta, colg[i], sh_r[i]);
            __syncthreads();                                  // every thread has read sh_kidx[j]
            if (tid == 0) sh_kidx[j] = k;
            if (one_unit && u0 + w < u1 && (u0 + w) / tiles == j) steps_stale = true;
            t = s;
            moves += 1;
        } else if (!keep_going) {
            stopped = true;
        }
        __syncthreads();
    }
    // ---- workgroup 0 hands the state back (after a failed wait the state is not written) ---
    if (g != 0 || failed) return;
    for (int64_t i = tid; i < m; i += nthreads) r[i] = sh_r[i];
    for (int64_t j = tid; j < n; j += nthreads) kidx[j] = sh_kidx[j];
    if (tid == 0) {
        InstState<T> z = st[0];
        z.t = t;
        z.best_s = last_s;
        z.apply_j = -1; z.apply_k = -1; z.delta = (T)0;
        z.moves = moves;
        z.done = stopped ? 1 : 0;
        st[0] = z;
    }
}

// ---- the same loop for the descent itself (not fixed-work mode) ------------------------------
// Only strictly improving moves matter there, and a variable has few of them.  For a row i of
// value r_i the product chain x_i(k) = fma(delta_k, A_ij, r_i) is monotone in k (D ascends, rounding is
// monotone), so the values with |x_i(k)| < t form an interval; a move that lowers the maximum lies in
// the intersection of the intervals of any rows.  Per iteration a workgroup
//   1. keeps one row of largest |r| out of each wavefront's share (the largest of all among them),
//      found while the last move is applied;
//   2. finds each of its variables' intervals by bisection on those rows, one lane per (row, bound);
//   3. scores the values of the interval over all rows, DI_KT at a time.  A longer interval is narrowed first:
//      the score is quasi-convex in k (a maximum of monotone chains' magnitudes, also as computed), so the
//      minimum lies between the neighbours of the lowest of DI_KT spaced samples; if a plateau keeps
//      that from shrinking, every value is scored.
// What is skipped scores at least t, so the record of an iteration is that of the full table whenever
// there is an improving move, and the loop stops just the same when there is none.
// On 4096 x 32 with 1024 levels (fp64) an iteration takes 9.1 us instead of 17.7 (all 1024 levels scored),
// of which the exchange is about 2 and the rest a chain of reductions; a local search of 8 moves to
// neighbouring levels on 8016 x 251 (256 levels, fp64) takes 59 us in this launch instead of 320 with
// two launches per move that score all levels.  On 256 x 64 with 16 levels there is too little to skip
// (5.3 us against 4.3): the host's model keeps the kernel above there.
// COOP: all wavefronts score one variable, its rows shared out (tall matrices, few variables);
// otherwise a wavefront scores a variable by itself.
constexpr int DI_KT = 8;                  // values scored together
constexpr int DI_PF = 8;                  // loads of a thread in flight where rows come from memory
constexpr double DI_COOP_US = 0.6;        // more for rounds that all wavefronts share (a barrier each), not near levels only

struct PlanI {
    int G = 0, vpw = 0, waves = 0;
    bool coop = false, cols = false;
    size_t lds = 0;
    double est_us = 0;
    double more_us = 0;   // what the choice between the two kernels counts on top
};

// Modelled like the plan above: exchange 2 us + 4 ns per workgroup, 1.6 us for the rest of an
// iteration, per variable its interval (0.3 us up to 64 levels, then 0.14 us per step of the bisection) and 1.5
// rounds of scoring DI_KT values (one round of one value where only the neighbouring levels are
// allowed).  Rows that come from memory instead of LDS count three times.
PlanI make_plan_interval(const dmmv_problem& p, int32_t radius, int cus) {
    PlanI best;
    if (p.csr_rowptr || p.R != 1 || p.scale || p.m < 1 || p.n < 1 || p.nd < 1) return best;
    const size_t w = p.dtype == DMMV_F64 ? 8 : 4;
    if (p.m > (int64_t)(DP_LDS_LIMIT / w) || p.n > (1 << 20) || p.nd > (1 << 16)) return best;
    const int gmax = cus < DP_MAX_G ? (cus > 0 ? cus : 1) : DP_MAX_G;
    for (int waves = 4; waves <= DP_MAX_WAVES; waves *= 2)
        for (int coop = 0; coop < 2; ++coop) {
            const int64_t want = coop ? p.n : ceil_div(p.n, waves);
            const int64_t g0 = want < gmax ? want : gmax;
            const int64_t vpw = ceil_div(p.n, g0), G = ceil_div(p.n, vpw);
            const size_t base = (size_t)p.m * w + (size_t)waves * DI_KT * DP_SKEW * w + (size_t)p.nd * w + (size_t)p.n * 4;
            if (base > DP_LDS_LIMIT) continue;
            const bool cols = base + (size_t)vpw * p.m * w <= DP_LDS_LIMIT;
            const double per_64 = waves == 4 ? (w == 8 ? 18.0 : 10.0) : (w == 8 ? 32.0 : 16.0);
            const double rows = (double)ceil_div(p.m, coop ? 64 * waves : 64);
            const bool near = radius == 1 || p.nd <= 3;
            double interval = 0.3;
            for (int32_t k = radius > 0 && radius < p.nd / 2 ? 2 * radius : p.nd; p.nd > 64 && k > 0; k >>= 1) interval += 0.14;
            const double round = (coop ? 0.6 : 0.4) * (near ? 1.0 : 1.5) + rows * (near ? 1.0 : 1.5 * DI_KT) * per_64 / 2400.0 * (cols ? 1.0 : 3.0);
            const double est = 3.6 + 0.004 * (double)G + (double)(coop ? vpw : ceil_div(vpw, waves)) * (interval + round) + 0.0002 * (double)p.m;
            if (best.G == 0 || est < best.est_us) {
                best.G = (int)G; best.vpw = (int)vpw; best.waves = waves; best.coop = coop != 0; best.cols = cols;
                best.lds = base + (cols ? (size_t)vpw * p.m * w : 0);
                best.est_us = est;
                best.more_us = coop && !near ? DI_COOP_US : 0.0;
            }
        }
    return best;
}

template <int CTRL>
__device__ __forceinline__ int32_t dpp_int(int32_t v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }

template <class T, int NWAVES, bool COOP, bool COLS>
__global__ __launch_bounds__(64 * NWAVES) void k_descent_dense_interval(
    int64_t m, int64_t n, int32_t nd, const T* __restrict__ A, int64_t lda, const T* __restrict__ D,
    T* r, int32_t* kidx, int32_t radius, const uint8_t* __restrict__ var_mask, InstState<T>* st,
    int32_t steps, int32_t iters, dmmv_move* trace, T* trace_t, int32_t vpw, uint64_t* rec, int32_t* flags,
    int32_t wait_limit) {
    constexpr int KT = DI_KT, NT = 64 * NWAVES, ROWS = 2 * NWAVES < 16 ? NWAVES : 8;   // rows the intervals are cut on
    extern __shared__ __align__(16) unsigned char smem[];
    T* sh_r = reinterpret_cast<T*>(smem);                   // [m]
    T* sh_cols = sh_r + m;                                  // [vpw][m] (COLS)
    T* sh_sc = sh_cols + (COLS ? (int64_t)vpw * m : 0);     // [NWAVES][KT * DP_SKEW]
    T* sh_D = sh_sc + NWAVES * KT * DP_SKEW;                // [nd]
    int32_t* sh_kidx = reinterpret_cast<int32_t*>(sh_D + nd);   // [n]
    __shared__ T sh_ws[NWAVES], sh_red[2][NWAVES][KT], sh_top_r[NWAVES];
    __shared__ int64_t sh_wc[NWAVES];
    __shared__ int32_t sh_top[NWAVES];
    __shared__ T sh_bs;
    __shared__ int64_t sh_bc;
    __shared__ int32_t sh_fail;

    const int G = gridDim.x, g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t j_lo = (int64_t)g * vpw, j_end = j_lo + vpw < n ? j_lo + vpw : n;

    // every pass over the rows of an array in memory keeps DI_PF loads of a thread in flight
    auto rows_of = [&](const T* src, auto use) {
        for (int64_t i0 = tid; i0 < m; i0 += DI_PF * NT) {
            T v[DI_PF];
#pragma unroll
            for (int u = 0; u < DI_PF; ++u) v[u] = src[i0 + u * NT < m ? i0 + u * NT : m - 1];
#pragma unroll
            for (int u = 0; u < DI_PF; ++u)
                if (i0 + u * NT < m) use(i0 + u * NT, v[u]);
        }
    };
    if (COLS)
        for (int64_t j = j_lo; j < j_end; ++j) {
            T* const dst = sh_cols + (j - j_lo) * m;
            rows_of(A + lda * j, [&](int64_t i, T v) { dst[i] = v; });
        }
    for (int64_t j = tid; j < n; j += NT) sh_kidx[j] = kidx[j];
    for (int32_t k = tid; k < nd; k += NT) sh_D[k] = D[k];
    if (tid == 0) sh_fail = 0;
    T t = st[0].t;
    int32_t moves = st[0].moves;
    T last_s = st[0].best_s;
    bool stopped = st[0].done != 0, failed = false;
    // the wavefront's row of largest |r| among those its threads hold
    auto top_row = [&](T bv, int32_t bi) {
        const T top = wave_max(bv);
        const unsigned long long has = __ballot(bi >= 0 && bv == top);
        if (has == 0) { if (lane == 0) { sh_top[w] = -1; sh_top_r[w] = (T)0; } }
        else if (lane == __builtin_ctzll(has)) { sh_top[w] = bi; sh_top_r[w] = sh_r[bi]; }
    };
    {
        T bv = (T)-1;
        int32_t bi = -1;
        rows_of(r, [&](int64_t i, T v) {
            sh_r[i] = v;
            if (dmmv_abs(v) > bv) { bv = dmmv_abs(v); bi = (int32_t)i; }
        });
        top_row(bv, bi);
    }
    __syncthreads();

    int parity = 0;
    for (int32_t it = 0; it < steps && !stopped; ++it) {
        T ws = (T)0;
        int64_t wc = -1;
        for (int64_t j = j_lo + (COOP ? 0 : w); j < j_end; j += COOP ? 1 : NWAVES) {
            const int32_t kcur = sh_kidx[j];
            const T dcur = sh_D[kcur];
            const T* __restrict__ col = COLS ? sh_cols + (j - j_lo) * m : A + lda * j;
            int32_t klo = radius > 0 && kcur - radius > 0 ? kcur - radius : 0;
            int32_t khi = radius > 0 && kcur < nd - 1 - radius ? kcur + radius : nd - 1;
            if (var_mask && var_mask[j] == 0) continue;      // the same for everyone who scores this variable
            // ---- the values that bring the top rows below t
            if (nd <= 64) {                                   // lane = value, no chain of dependent reads
                const int32_t k = lane;
                const T delta = step_of(sh_D[k < nd ? k : nd - 1], dcur, (T)1);
                bool good = k >= klo && k <= khi;
#pragma unroll
                for (int u = 0; u < ROWS; ++u) {
                    const int32_t row = sh_top[u];
                    const T a = col[row >= 0 ? row : 0], ri = sh_top_r[u];
                    good = good && (row < 0 || dmmv_abs(dmmv_fma(delta, a, ri)) < t);
                }
                const unsigned long long b = __ballot(good);
                if (b == 0) continue;                         // the same for everyone who scores this variable
                klo = __builtin_ctzll(b);
                khi = 63 - __builtin_clzll(b);
            } else {                                          // lane = (row, bound): bisection
                const int u = (lane >> 1) % ROWS;
                const bool upper = (lane & 1) == 0;           // x < t, else x > -t
                const int32_t row = sh_top[u];
                const T a = row >= 0 ? col[row] : (T)0, ri = sh_top_r[u];
                const bool prefix = upper == (a >= (T)0);     // the values that satisfy the bound are the first ones
                int32_t x = klo, y = khi + 1;                 // first value that breaks (prefix) or satisfies it
                const int32_t span = khi - klo + 1;
                for (int32_t s = span; s > 0; s >>= 1) {      // the same number of steps in every lane
                    if (x < y) {
                        const int32_t mid = (x + y) >> 1;
                        const T v = dmmv_fma(step_of(sh_D[mid], dcur, (T)1), a, ri);
                        const bool good = upper ? v < t : v > -t;
                        if (good != prefix) y = mid; else x = mid + 1;
                    }
                }
                int32_t lo = !prefix && row >= 0 ? y : klo, hi = prefix && row >= 0 ? y - 1 : khi;
                int32_t o;
                o = dpp_int<DPP_QUAD_XOR1>(lo); lo = o > lo ? o : lo;
                o = dpp_int<DPP_QUAD_XOR2>(lo); lo = o > lo ? o : lo;
                o = dpp_int<DPP_ROW_HALF_MIRROR>(lo); lo = o > lo ? o : lo;
                o = dpp_int<DPP_ROW_MIRROR>(lo); lo = o > lo ? o : lo;
                o = dpp_int<DPP_QUAD_XOR1>(hi); hi = o < hi ? o : hi;
                o = dpp_int<DPP_QUAD_XOR2>(hi); hi = o < hi ? o : hi;
                o = dpp_int<DPP_ROW_HALF_MIRROR>(hi); hi = o < hi ? o : hi;
                o = dpp_int<DPP_ROW_MIRROR>(hi); hi = o < hi ? o : hi;
                klo = __builtin_amdgcn_readlane(lo, 0);
                khi = __builtin_amdgcn_readlane(hi, 0);
            }
            // scores of the first KE of the values k0, k0 + stride, .. (clamped to khi): lane 8 q + x holds that of
            // value q (the others infinity)
            auto score = [&](auto ke, int32_t k0, int32_t stride) -> T {
                constexpr int KE = decltype(ke)::value;
                T delta[KE], acc[KE];
#pragma unroll
                for (int e = 0; e < KE; ++e) {
                    const int64_t k = k0 + (int64_t)e * stride;
                    delta[e] = step_of(sh_D[k < khi ? k : khi], dcur, (T)1);
                    acc[e] = (T)0;
                }
                constexpr int STEP = COOP ? NT : 64, RB = KE == KT ? 2 : 4;
                for (int64_t i0 = COOP ? tid : lane; i0 < m; i0 += RB * STEP) {
                    T a[RB], ri[RB];
#pragma unroll
                    for (int u = 0; u < RB; ++u) {                      // past the end: a maximum does not mind the repeat
                        const int64_t i = i0 + u * STEP < m ? i0 + u * STEP : i0;
                        a[u] = col[i];
                        ri[u] = sh_r[i];
                    }
#pragma unroll
                    for (int u = 0; u < RB; ++u)
#pragma unroll
                        for (int e = 0; e < KE; ++e) acc[e] = dmmv_max(acc[e], dmmv_abs(dmmv_fma(delta[e], a[u], ri[u])));
                }
                const int q = lane >> 3, part = lane & 7;
                T v;
                if (KE == KT) {
                    T* sc = sh_sc + w * KT * DP_SKEW;
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int e = 0; e < KE; ++e) sc[e * DP_SKEW + lane] = acc[e];
                    __builtin_amdgcn_wave_barrier();
                    v = (T)0;
#pragma unroll
                    for (int e = 0; e < 8; ++e) v = dmmv_max(v, sc[q * DP_SKEW + part * 8 + e]);
                    __builtin_amdgcn_wave_barrier();
                    v = dmmv_max(v, dpp_mov<DPP_QUAD_XOR1>(v));
                    v = dmmv_max(v, dpp_mov<DPP_QUAD_XOR2>(v));
                    v = dmmv_max(v, dpp_mov<DPP_ROW_HALF_MIRROR>(v));
                } else {
                    v = Limits<T>::inf();
#pragma unroll
                    for (int e = 0; e < KE; ++e) { const T x = wave_max(acc[e]); if (q == e) v = x; }
                }
                if (COOP) {
                    // (two buffers in turn: nobody writes one again before everyone has passed the next barrier)
                    if (part == 0) sh_red[parity][w][q] = v;
                    __syncthreads();
#pragma unroll
                    for (int x = 0; x < NWAVES; ++x) v = dmmv_max(v, sh_red[parity][x][q]);
                    parity ^= 1;
                }
                return v;
            };
            constexpr std::integral_constant<int, KT> all{};
            while (klo <= khi) {                              // uniform
                const int32_t len = khi - klo + 1;
                if (len <= KT) {
                    const T v = len == 1 ? score(std::integral_constant<int, 1>{}, klo, 1)
                                         : len == 2 ? score(std::integral_constant<int, 2>{}, klo, 1) : score(all, klo, 1);
                    const T cs = (lane >> 3) < len ? v : Limits<T>::inf();
                    const T smin = wave_min(cs);
                    const int64_t c = j * (int64_t)nd + klo + (__builtin_ctzll(__ballot(cs == smin)) >> 3);
                    if (rec_less(smin, c, ws, wc)) { ws = smin; wc = c; }
                    break;
                }
                const int32_t stride = (len + KT - 3) / (KT - 1);     // the last sample is khi, or clamped to it
                const T v = score(all, klo, stride);
                const T smin = wave_min(v);
                const unsigned long long hit = __ballot(v == smin);
                const int e1 = __builtin_ctzll(hit) >> 3, e2 = (63 - __builtin_clzll(hit)) >> 3;
                const int64_t after = klo + (int64_t)(e2 + 1) * stride;
                const int32_t nlo = e1 > 0 ? klo + (e1 - 1) * stride + 1 : klo;
                const int32_t nhi = e2 + 1 < KT && after <= khi ? (int32_t)after - 1 : khi;
                if ((nhi - nlo + 1) * 2 > len + stride) {             // a plateau: score every value
                    const int32_t kend = khi;
                    for (int32_t k0 = klo; k0 <= kend; k0 += KT) {
                        const T f = score(all, k0, 1);
                        const T cs = k0 + (lane >> 3) <= kend ? f : Limits<T>::inf();
                        const T fmin = wave_min(cs);
                        const int64_t c = j * (int64_t)nd + k0 + (__builtin_ctzll(__ballot(cs == fmin)) >> 3);
                        if (rec_less(fmin, c, ws, wc)) { ws = fmin; wc = c; }
                    }
                    break;
                }
                klo = nlo;
                khi = nhi;
            }
        }
        if (lane == 0) { sh_ws[w] = ws; sh_wc[w] = wc; }
        __syncthreads();
        // ---- one record per workgroup, the smallest of all -----------------------------------
        if (w == 0) {
            T bs = lane < NWAVES ? sh_ws[lane] : (T)0;
            int64_t bc = lane < NWAVES ? sh_wc[lane] : (int64_t)-1;
            wave_argmin(bs, bc);
            if (lane == 0) dp_publish(rec, G, g, it, bs, bc);
            T gs;
            int64_t gc;
            const bool fail = !dp_collect(rec, G, it, lane, wait_limit, flags, gs, gc);
            if (lane == 0) {
                sh_bs = gs;
                sh_bc = gc;
                if (fail) { sh_fail = 1; atomicOr(&flags[FLAG_ERROR], ERRBIT_WAIT_LIMIT); }
            }
        }
        __syncthreads();
        if (sh_fail) { failed = true; break; }
        // ---- the same decision in every workgroup ------------------------------------------
        const T s = sh_bs;
        const int64_t c = sh_bc;
        if (c >= 0 && s < t) {
            last_s = s;
            const int32_t j = (int32_t)(c / nd), k = (int32_t)(c % nd);
            const T delta = step_of(sh_D[k], sh_D[sh_kidx[j]], (T)1);
            if (g == 0 && tid == 0 && moves < iters) {
                if (trace) { trace[moves].j = j; trace[moves].k = k; }
                if (trace_t) trace_t[moves] = s;
            }
            const T* __restrict__ colg = A + lda * (int64_t)j;
            T bv = (T)-1;
            int32_t bi = -1;
            rows_of(colg, [&](int64_t i, T a) {
                const T v = dmmv_fma(delta, a, sh_r[i]);
                sh_r[i] = v;
                if (dmmv_abs(v) > bv) { bv = dmmv_abs(v); bi = (int32_t)i; }
            });
            top_row(bv, bi);
            __syncthreads();                                  // every thread has read sh_kidx[j]
            if (tid == 0) sh_kidx[j] = k;
            t = s;
            moves += 1;
        } else {
            stopped = true;
        }
        __syncthreads();
    }
    // ---- workgroup 0 hands the state back (after a failed wait the state is not written) ---
    if (g != 0 || failed) return;
    for (int64_t i = tid; i < m; i += NT) r[i] = sh_r[i];
    for (int64_t j = tid; j < n; j += NT) kidx[j] = sh_kidx[j];
    if (tid == 0) {
        InstState<T> z = st[0];
        z.t = t;
        z.best_s = last_s;
        z.apply_j = -1; z.apply_k = -1; z.delta = (T)0;
        z.moves = moves;
        z.done = stopped ? 1 : 0;
        st[0] = z;
    }
}

template <class T>
dmmv_status run_t(Ctx* c, const Plan& pl, int32_t steps, int32_t iters, dmmv_move* trace, void* trace_t) {
    // iteration numbers start at 1: cleared records name no iteration
    uint64_t* rec = (uint64_t*)c->persist_exchange;
    const int words = 2 * DP_MAX_G * DP_REC_WORDS * 2;       // as 32-bit words
    if (!c->exchange_clear)
        hipLaunchKernelGGL(k_zero_words, dim3((unsigned)ceil_div(words, 256)), dim3(256), 0, c->stream, (uint32_t*)rec, words);
    c->exchange_clear = false;
    const int32_t wait_limit = c->o.wait_limit > 0 ? c->o.wait_limit : DP_WAIT_DEFAULT;
    auto kernel = pl.waves == 8 ? k_descent_dense_persistent<T, 8> : k_descent_dense_persistent<T, 4>;
    DMMV_TRY(ensure_dynamic_lds((const void*)kernel, (int)DP_LDS_LIMIT));
    hipLaunchKernelGGL(kernel, dim3((unsigned)pl.G), dim3(64 * pl.waves), pl.lds, c->stream,
                       c->p.m, c->p.n, c->p.nd, (const T*)c->p.A_dense, c->p.lda, (const T*)c->D_dev, (T*)c->r,
                       c->kidx, c->o.radius, c->o.var_mask, (InstState<T>*)c->state, c->o.keep_going, steps, iters, trace,
                       (T*)trace_t, (int32_t)ceil_div(c->p.nd, DP_KT), (int32_t)pl.upw, (int32_t)pl.ncols, rec,
                       c->flags, wait_limit);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
dmmv_status run_interval_t(Ctx* c, const PlanI& pl, int32_t steps, int32_t iters, dmmv_move* trace, void* trace_t) {
    uint64_t* rec = (uint64_t*)c->persist_exchange;
    const int words = 2 * DP_MAX_G * DP_REC_WORDS * 2;
    if (!c->exchange_clear)
        hipLaunchKernelGGL(k_zero_words, dim3((unsigned)ceil_div(words, 256)), dim3(256), 0, c->stream, (uint32_t*)rec, words);
    c->exchange_clear = false;
    const int32_t wait_limit = c->o.wait_limit > 0 ? c->o.wait_limit : DP_WAIT_DEFAULT;
    auto launch = [&](auto kernel) -> dmmv_status {
        DMMV_TRY(ensure_dynamic_lds((const void*)kernel, (int)DP_LDS_LIMIT));
        hipLaunchKernelGGL(kernel, dim3((unsigned)pl.G), dim3(64 * pl.waves), pl.lds, c->stream, c->p.m, c->p.n, c->p.nd,
                           (const T*)c->p.A_dense, c->p.lda, (const T*)c->D_dev, (T*)c->r, c->kidx, c->o.radius,
                           c->o.var_mask, (InstState<T>*)c->state, steps, iters, trace, (T*)trace_t, (int32_t)pl.vpw, rec,
                           c->flags, wait_limit);
        DMMV_LAUNCH_CHECK();
        return DMMV_OK;
    };
    auto by_mode = [&](auto waves) -> dmmv_status {
        constexpr int W = decltype(waves)::value;
        if (pl.coop) return pl.cols ? launch(k_descent_dense_interval<T, W, true, true>) : launch(k_descent_dense_interval<T, W, true, false>);
        return pl.cols ? launch(k_descent_dense_interval<T, W, false, true>) : launch(k_descent_dense_interval<T, W, false, false>);
    };
    return pl.waves == 8 ? by_mode(std::integral_constant<int, 8>{}) : by_mode(std::integral_constant<int, 4>{});
}

}  // namespace

// Two of these kernels that are each resident in part would wait for one another until their limits end.  Every launch
// therefore claims as many of the device's compute units as it has workgroups, from before the launch until the stream has
// been waited for, and the claims of the process together do not exceed the compute units: a workgroup that is not resident
// then always finds one that has none of them.  Workgroups are dealt to the 8 XCDs in turn, and what holds for the device
// has to hold for each XCD, so a claim is rounded up to the same number in all of them.  Kernels that do not wait only
// delay a start.  With dense_loop = 2 a call waits for its turn, in the order of the calls; an automatic choice waits for as
// long as the loop of launches would take, at most CLAIM_WAIT_US, and then takes that loop.
// (Four threads with an instance of 8016 x 251 each, whose grid is 251: 40 moves took 1.1 s a call without the claims and
// take 4.0 ms with them; one thread, 0.98 ms.)
namespace {
constexpr int CLAIM_MAX_DEVICES = 64;
constexpr int CLAIM_XCDS = 8;
constexpr double CLAIM_WAIT_US = 5000.0;
struct Claims {
    int units = 0;                         // compute units claimed
    uint64_t next = 0, served = 0;         // the queue of claims that wait
};
std::mutex g_claim_mu;
std::condition_variable g_claim_cv;
Claims g_claims[CLAIM_MAX_DEVICES];
}  // namespace

static double launch_loop_us(const Ctx* c) {               // an iteration of the loop of launches, by its model
    const double pairs = (double)c->p.m * (double)c->p.n * (double)c->p.nd;
    return DP_LAUNCH_LOOP_US + pairs * (c->p.dtype == DMMV_F64 ? DP_LAUNCH_LOOP_US_PER_PAIR_F64
                                                               : DP_LAUNCH_LOOP_US_PER_PAIR_F32);
}

bool OneLaunchClaim::take(const Ctx* c, int32_t workgroups, int64_t moves) {
    release();
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= CLAIM_MAX_DEVICES) return true;    // not counted
    const int cus = device_cus();
    const int need = (int)ceil_div(workgroups, CLAIM_XCDS) * CLAIM_XCDS;
    std::unique_lock<std::mutex> lock(g_claim_mu);
    Claims& k = g_claims[dev];
    auto room = [&] { return k.units == 0 || k.units + need <= cus; };
    if (c->o.dense_loop == 2) {
        const uint64_t turn = k.next++;
        g_claim_cv.wait(lock, [&] { return k.served == turn && room(); });
        ++k.served;
        g_claim_cv.notify_all();           // the next one in the queue may fit too
    } else {
        const std::chrono::duration<double, std::micro> most(std::min((double)moves * launch_loop_us(c), CLAIM_WAIT_US));
        if (!g_claim_cv.wait_for(lock, most, [&] { return k.served == k.next && room(); })) return false;
    }
    k.units += need;
    dev_ = dev;
    units_ = need;
    return true;
}

void OneLaunchClaim::release() {
    if (units_ == 0) return;
    {
        std::lock_guard<std::mutex> lock(g_claim_mu);
        g_claims[dev_].units -= units_;
    }
    units_ = 0;
    g_claim_cv.notify_all();
}

// options.dense_loop: 0 = one launch when the model says its iteration is shorter than that of
// the loop of launches, 1 = always a launch per step, 2 = one launch whenever the instance fits
// (dmmv_create refuses the option otherwise).
bool dense_persistent_fits(const dmmv_problem& p) { return make_plan(p, DP_MAX_G).G > 0; }

// The descent itself takes the kernel with the shorter modelled iteration: scoring every value (few
// levels and rows: 256 x 64 with 16 levels 4.3 us against 5.3) or only the intervals that can improve.  Where the two come
// close, the barriers of rounds that the wavefronts share decide: 1024 x 64 with 16 levels in fp64 takes 7.3 us by
// intervals and 6.0 with every value scored, 5.6 and 5.8 by the model alone.  Of 378 measured choices (66 shapes, both types,
// random and filter matrices, radius 0, 1 and 2) one is by then the slower one, 2048 x 512 with 64 levels in fp32, 10.8 against
// 10.5.
static bool take_interval(const Ctx* c, const Plan& all, const PlanI& some) {
    return !c->o.keep_going && some.G > 0 && (all.G == 0 || some.est_us + some.more_us < all.est_us);
}

int32_t dense_persistent_workgroups(const Ctx* c) {
    if (c->kind != KIND_DENSE || c->o.dense_loop == 1 || !c->persist_exchange) return 0;
    if (c->o.l2_rule == 1 || c->o.l2_rule == 2) return 0;
    if (!c->o.keep_going && (c->o.value_search || c->o.prune)) return 0;      // those have loops of their own
    const Plan all = make_plan(c->p, device_cus());
    const PlanI some = make_plan_interval(c->p, c->o.radius, device_cus());
    const bool interval = take_interval(c, all, some);
    const int32_t workgroups = interval ? some.G : all.G;
    const double est_us = interval ? some.est_us : all.est_us;
    return workgroups > 0 && (c->o.dense_loop == 2 || est_us < launch_loop_us(c)) ? workgroups : 0;
}

int32_t dense_interval_in_use(const Ctx* c) {
    if (!dense_persistent_applicable(c)) return 0;
    const PlanI some = make_plan_interval(c->p, c->o.radius, device_cus());
    if (!take_interval(c, make_plan(c->p, device_cus()), some)) return 0;
    return 4 | (some.coop ? 8 : 0) | (some.cols ? 16 : 0) | (some.waves == 8 ? 32 : 0);
}

dmmv_status dense_descent_persistent(Ctx* c, int32_t steps, int32_t iters, dmmv_move* trace, void* trace_t) {
    const Plan pl = make_plan(c->p, device_cus());
    const PlanI some = make_plan_interval(c->p, c->o.radius, device_cus());
    if (take_interval(c, pl, some))
        return c->p.dtype == DMMV_F64 ? run_interval_t<double>(c, some, steps, iters, trace, trace_t)
                                      : run_interval_t<float>(c, some, steps, iters, trace, trace_t);
    if (pl.G == 0) return fail(DMMV_ERR_STATE, "one-launch dense descent: the instance does not fit");
    return c->p.dtype == DMMV_F64 ? run_t<double>(c, pl, steps, iters, trace, trace_t)
                                  : run_t<float>(c, pl, steps, iters, trace, trace_t);
}

}  // namespace dmmv
