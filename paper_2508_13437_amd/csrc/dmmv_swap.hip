// Swap move of the local search (paper: section "Search Operators", Proposition 1 and
// Corollary 1; Appendix B "Swap Move", Algorithm 2) for dense matrices and batches.
//
// A swap exchanges the values of two variables x_i > x_j.  With Delta = s * (D[k_i] - D[k_j])
// the new residual is r'_k = fma(Delta, A_kj - A_ki, r_k) and the swap kept is the one with
// the smallest t' = max_k |r'_k| (lowest pair number c = i*n + j on a tie), if t' < t.
//
// The filter of Corollary 1 tests a necessary condition on the k_eps rows of largest |r_k|.
// Here the condition is the evaluation itself restricted to those rows: a pair whose new
// residual reaches t on one of them cannot improve.  The rows are tried in order of
// decreasing |r_k| and a pair is dropped at the first row that reaches t, or that exceeds the
// best t' found so far; what survives is evaluated on every row.  Dropping only such pairs
// leaves the result that of the full enumeration, whatever the order in which wavefronts
// find their candidates.
//
// Work split: one workgroup handles one instance; each of its wavefronts takes variables u and
// a lane one partner v > u, so every unordered pair is met once.  The first rows of the filter
// are staged in LDS (as many as fit beside the instance's values D[k_j]), the others are read
// from memory; pairs that pass all of them are finished by the whole wavefront, one lane per
// row, so that A is read along its columns.  A batch's workgroups share the best t' of their
// instance through memory, so that a pair one of them has found prunes the others' (512 instances of
// 2048 x 4096: 18.6 -> 11.9 ms at a rounded start, where good swaps are plenty, 15.8 -> 15.4 at a
// local optimum; 20 instances 10.7 -> 3.0; the kernel alone).
#include "dmmv_common.h"

namespace dmmv {

namespace {

constexpr int SW_BLOCK = 256;
constexpr int SW_WAVES = SW_BLOCK / 64;
constexpr int SWE_BLOCK = 1024;                // evaluation: many wavefronts share one instance's LDS tile
constexpr int SWE_WAVES = SWE_BLOCK / 64;
constexpr int SWE_QCAP = 128;                  // queue of a wavefront: under 64 waiting plus at most 64 new
constexpr size_t SW_LDS_BUDGET = 68 * 1024;    // dynamic LDS of the evaluation kernel (8 KiB more are static):
                                               // two workgroups share a compute unit's 160 KiB

__device__ __forceinline__ unsigned long long order_bits(float v) { return (unsigned long long)__float_as_uint(v); }
__device__ __forceinline__ unsigned long long order_bits(double v) { return (unsigned long long)__double_as_longlong(v); }
// best t' of an instance found by any of its workgroups: the bit pattern orders like the value (t' >= 0)
__device__ __forceinline__ void share_best(float* g, float v) { atomicMin(reinterpret_cast<unsigned int*>(g), __float_as_uint(v)); }
__device__ __forceinline__ void share_best(double* g, double v) {
    atomicMin(reinterpret_cast<unsigned long long*>(g), (unsigned long long)__double_as_longlong(v));
}
__device__ __forceinline__ void from_order_bits(unsigned long long b, float& v) { v = __uint_as_float((uint32_t)b); }
__device__ __forceinline__ void from_order_bits(unsigned long long b, double& v) { v = __longlong_as_double((long long)b); }
// the largest value below t >= 0 (finite); -1 for t = 0, which no magnitude is at or below
__device__ __forceinline__ float value_below(float t) { return t > 0.0f ? __uint_as_float(__float_as_uint(t) - 1u) : -1.0f; }
__device__ __forceinline__ double value_below(double t) {
    return t > 0.0 ? __longlong_as_double(__double_as_longlong(t) - 1ll) : -1.0;
}

// ---- K rows of large |r| per instance for the filter, in decreasing order.  Which rows the
// filter tries first changes the time a search takes, never its result, so an exact top-K
// selection is not needed: every thread takes the largest |r| among its rows i = thread,
// thread + 256, ... and the 256 maxima are ranked (larger first, lower row first among equal
// values).  The row of largest |r| always comes first; of the next largest most are there.
// One workgroup per instance, bound by the latency of its reads of memory and of LDS: eight of either are in flight in a thread
// (one at a time 24 us on 256 rows and 74 on 100 000, now 13 and 30).
template <class T>
__global__ __launch_bounds__(SW_BLOCK) void k_swap_top(int64_t m, int64_t R, int32_t K,
                                                        const T* __restrict__ r,
                                                        const int32_t* __restrict__ skip,
                                                        int32_t* __restrict__ rows_all, T* __restrict__ gbest) {
    __shared__ T sh_a[SW_BLOCK];
    __shared__ int32_t sh_row[SW_BLOCK];
    const int64_t q = blockIdx.x;
    if (skip && skip[q]) return;
    if (gbest && threadIdx.x == 0) gbest[q] = Limits<T>::inf();
    T a = (T)-1;                                           // no row: ranks after every real one
    int32_t row = INT32_MAX;
    for (int64_t i0 = threadIdx.x; i0 < m; i0 += 8 * SW_BLOCK) {
        T v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = dmmv_abs(r[(i0 + e * SW_BLOCK < m ? i0 + e * SW_BLOCK : m - 1) * R + q]);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (i0 + e * SW_BLOCK < m && v[e] > a) { a = v[e]; row = (int32_t)(i0 + e * SW_BLOCK); }
    }
    sh_a[threadIdx.x] = a;
    sh_row[threadIdx.x] = row;
    __syncthreads();
    int32_t rank = 0;
    for (int x = 0; x < SW_BLOCK; x += 8) {
        T oa[8];
        int32_t orow[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) { oa[e] = sh_a[x + e]; orow[e] = sh_row[x + e]; }
#pragma unroll
        for (int e = 0; e < 8; ++e) rank += (oa[e] > a || (oa[e] == a && orow[e] < row)) ? 1 : 0;
    }
    if (row != INT32_MAX && rank < K) rows_all[q * K + rank] = row;
}

// ---- evaluation: grid (R, nb).  Writes one record (t', c) per workgroup; c = -1 if the
// workgroup found no pair with t' < t.
//
// A wavefront owns a variable u and walks its partners v > u, 64 at a time, through the filter
// rows held in LDS.  Every such row drops about half of the pairs still alive when many rows
// are close to t (the state a descent leaves), so the survivors are packed into a queue of the
// wavefront and taken through the remaining filter rows (read from memory) 64 at a time, all
// lanes busy.  What passes every filter row is evaluated on all m rows by the whole wavefront,
// one lane per row.
template <class T, bool DVL>
__global__ __launch_bounds__(SWE_BLOCK) void k_swap_eval(
    int64_t m, int64_t n, int64_t R, int32_t nb, int32_t K, int32_t L, const T* __restrict__ A,
    int64_t lda, const T* __restrict__ At, const T* __restrict__ D, const T* __restrict__ scale,
    const int32_t* __restrict__ kidx, const T* __restrict__ r, const InstState<T>* __restrict__ st,
    const uint8_t* __restrict__ var_mask, const int32_t* __restrict__ rows_all,
    const int32_t* __restrict__ skip, T* gbest, Partial<T>* __restrict__ part) {
    extern __shared__ __align__(16) unsigned char sw_smem[];
    // carve: rtop[K] | dv[n] (DVL) | atop[L][n] | rows[K]
    T* rtop = reinterpret_cast<T*>(sw_smem);
    T* sh_dv = rtop + K;
    T* atop = sh_dv + (DVL ? n : 0);
    int32_t* sh_rows = reinterpret_cast<int32_t*>(atop + (int64_t)L * n);
    __shared__ int32_t sh_queue[SWE_WAVES][SWE_QCAP];      // partners v waiting for the later rows
    __shared__ unsigned long long sh_best;                 // order bits of the best t' of the workgroup
    __shared__ T sh_s[SWE_WAVES];
    __shared__ int64_t sh_c[SWE_WAVES];

    const int64_t q = blockIdx.x;
    const int blk = blockIdx.y;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    Partial<T>* out = part + q * nb + blk;
    if (skip && skip[q]) {
        if (threadIdx.x == 0) { Partial<T> e; e.s = (T)0; e.c = -1; *out = e; }
        return;
    }
    const int32_t* __restrict__ rows_g = rows_all + q * K;
    const uint8_t* __restrict__ vm = var_mask ? var_mask + q * n : nullptr;
    for (int l = threadIdx.x; l < K; l += SWE_BLOCK) {
        const int32_t row = rows_g[l];
        sh_rows[l] = row;
        rtop[l] = r[(int64_t)row * R + q];
    }
    if (DVL)
        for (int64_t j = threadIdx.x; j < n; j += SWE_BLOCK) sh_dv[j] = D[kidx[j * R + q]];
    for (int64_t e = threadIdx.x; e < (int64_t)L * n; e += SWE_BLOCK) {
        const int64_t l = e / n, j = e % n;
        atop[e] = A[(int64_t)rows_g[l] + j * lda];
    }
    if (threadIdx.x == 0) sh_best = order_bits(Limits<T>::inf());
    __syncthreads();
    int32_t* queue = sh_queue[w];                          // written and read by this wavefront only

    auto dv = [&](int64_t j) -> T { return DVL ? sh_dv[j] : D[kidx[j * R + q]]; };
    // Unordered pairs {u, v}, u < v, each taken in the orientation its values give: with
    // Ds = +Delta when x_u > x_v (pair (u, v)) and -Delta when x_v > x_u (pair (v, u)) the new
    // residual of either is fma(Ds, A_kv - A_ku, r_k), bit for bit (a - b = -(b - a) and
    // fma(-x, y, z) = fma(x, -y, z) exactly).
    const T sc = scale[q];
    auto step_of = [&](T dvu, T dvv) -> T {
        if (dvu > dvv) { const T diff = dvu - dvv; return sc * diff; }
        const T diff = dvv - dvu;
        return -(sc * diff);
    };

    const T t = st[q].t;
    T best_t = Limits<T>::inf();
    int64_t best_c = -1;                                   // the wavefront's record (uniform)
    T others = Limits<T>::inf();                           // what the instance's other workgroups had found
    auto bound = [&]() -> T {
        T shared_t;
        from_order_bits(__hip_atomic_load(&sh_best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP), shared_t);
        return dmmv_min(dmmv_min(best_t, others), shared_t);
    };

    // the first `cnt` queued partners of u: remaining filter rows, then the full evaluation
    auto drain = [&](int64_t u, T dvu, const T* __restrict__ Au, int cnt) {
        bool alive = lane < cnt;
        const int64_t v = alive ? (int64_t)queue[lane] : u;
        const T Ds = alive ? step_of(dvu, dv(v)) : (T)0;
        T bnd = bound();
        const T thr = dmmv_min(bnd, value_below(t));       // val < t and val <= bound in one test
        for (int l = L; l < K && __any(alive); ++l) {
            if (alive) {
                const int64_t row = sh_rows[l];
                const T au = At ? At[row * n + u] : Au[row];
                const T av = At ? At[row * n + v] : A[row + v * lda];
                const T val = dmmv_abs(dmmv_fma(Ds, av - au, rtop[l]));
                alive = val <= thr;
            }
        }
        unsigned long long todo = __ballot(alive);
        while (todo) {
            const int src = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int64_t sv = (int64_t)queue[src];
            const T dvv = dv(sv);
            const T Dl = step_of(dvu, dvv);
            const T* __restrict__ Av = A + sv * lda;
            bnd = bound();
            T val = (T)0, wm = (T)0;
            bool ok = true;
            for (int64_t base = 0; base < m && ok; base += 256) {
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int64_t row = base + x * 64 + lane;
                    if (row < m) val = dmmv_max(val, dmmv_abs(dmmv_fma(Dl, Av[row] - Au[row], r[row * R + q])));
                }
                wm = wave_max(val);
                ok = wm < t && !(wm > bnd);
            }
            if (ok && wm < t) {
                const int64_t c = dvu > dvv ? u * n + sv : sv * n + u;
                if (rec_less(wm, c, best_t, best_c)) {
                    best_t = wm;
                    best_c = c;
                    if (lane == 0) {
                        atomicMin(&sh_best, order_bits(wm));
                        if (gbest) share_best(gbest + q, wm);
                    }
                }
            }
        }
    };

    // n < 2^31 (the variables are numbered with int32 throughout the library), and L * n
    // elements fit in LDS, so 32-bit indices do below.
    const int32_t n32 = (int32_t)n;
    const unsigned long long below = (1ull << lane) - 1ull;
    const T t_below = value_below(t);
    for (int32_t u = blk * SWE_WAVES + w; u < n32; u += nb * SWE_WAVES) {
        if (vm && !vm[u]) continue;
        if (gbest) others = __hip_atomic_load(gbest + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const T dvu = dv(u);
        const T* __restrict__ Au = A + (int64_t)u * lda;
        int qn = 0;                                        // queued partners (uniform)
        for (int32_t v0 = (u + 1) & ~63; v0 < n32; v0 += 64) {
            const int32_t v = v0 + lane;
            bool alive = false;
            T Ds = (T)0;
            if (v > u && v < n32) {
                const T dvv = dv(v);
                alive = dvu != dvv;
                if (vm) alive = alive && vm[v];
                Ds = step_of(dvu, dvv);
            }
            // One threshold for both tests: val < t and val <= bound  <=>  val <= min(bound, t-),
            // t- the largest value below t.  After the first row (which, far from a local
            // optimum, often leaves no pair of the 64) the rows are taken without a branch: a
            // wavefront instruction costs the same however many lanes still need it.
            const T thr = dmmv_min(bound(), t_below);
            const int32_t vv = alive ? v : u;              // a lane without a pair reads in bounds
            const T* __restrict__ row_l = atop;
            if (L > 0) {
                const T val = dmmv_abs(dmmv_fma(Ds, row_l[vv] - row_l[u], rtop[0]));
                alive = alive & (val <= thr);
                if (!__any(alive)) continue;
                row_l += n32;
            }
            for (int l = 1; l < L; ++l, row_l += n32) {
                const T val = dmmv_abs(dmmv_fma(Ds, row_l[vv] - row_l[u], rtop[l]));
                alive = alive & (val <= thr);
            }
            const unsigned long long bal = __ballot(alive);
            if (!bal) continue;
            if (alive) queue[qn + __popcll(bal & below)] = v;
            qn += __popcll(bal);
            __builtin_amdgcn_wave_barrier();
            if (qn >= 64) {
                drain(u, dvu, Au, 64);
                const int32_t carry = 64 + lane < qn ? queue[64 + lane] : 0;
                __builtin_amdgcn_wave_barrier();
                if (64 + lane < qn) queue[lane] = carry;
                __builtin_amdgcn_wave_barrier();
                qn -= 64;
            }
        }
        if (qn > 0) drain(u, dvu, Au, qn);
    }
    if (lane == 0) { sh_s[w] = best_t; sh_c[w] = best_c; }
    __syncthreads();
    if (threadIdx.x == 0) {
        T bs = sh_s[0];
        int64_t bc = sh_c[0];
        for (int x = 1; x < SWE_WAVES; ++x)
            if (rec_less(sh_s[x], sh_c[x], bs, bc)) { bs = sh_s[x]; bc = sh_c[x]; }
        Partial<T> p;
        p.s = bc < 0 ? (T)0 : bs;
        p.c = bc;
        *out = p;
    }
}

// ---- evaluation over sorted variables: grid (R, nb), the same records.
//
// The variables are sorted by (level, entry in the row of largest |r|).  For a variable u and a lower level b the
// step Delta is fixed, so the new residual of that row, fma(Delta, A_v - A_u, r), ascends with A_v also as computed
// (every rounding is monotone): the partners that keep it within a threshold are a contiguous range of the level's
// variables, found by bisection on the evaluation itself.  Only pairs of such ranges are looked at.
// The threshold grows in stages towards t, each of which leaves out the pairs that the one before has looked at (a pair is tested
// against the best t' found so far, not against its stage: what a stage meets is settled), and ends at the best t' found so far: at a rounded start the best swap lowers
// t by a tenth or a third, which one variable of large entries is needed for, and the ranges hold some hundredth of the
// pairs (50 000 of 7 million on 2048 x 4096); at a local optimum two thirds, of which the next rows drop most.
// A unit of work is (64 consecutive variables, level), or with `slices` (a power of two) every slices-th of the 64; the wavefronts of a workgroup take units from a counter
// per stage.  A wavefront is through when a stage it has finished reached the bound: the units of that stage
// are all taken, and whoever holds one covers it up to the smaller of stage and bound.  A few units hold most
// pairs (outlier channels sort to the ends of their levels), so what is over SWI_PART is shared.
// Bound by the latency of its gathers in the slowest instances (three times the pairs of the average one) and, at
// local optima, by instruction issue; one workgroup of 16 wavefronts a compute unit (67 registers, 89 in fp64).
// A whole search in ms, rounded start / local optimum, by the evaluation of all pairs and by this one:
//     512 instances of 2048 x 4096, 16 levels  22.6 / 16.6    0.67 / 11.2      one of 2048 x 512, 16 levels      0.36 / 0.089    0.055 / 0.054
//     20 of them                               9.0 / 1.28     0.19 / 0.91      2048 x 8192, 2 levels             1.98 / 0.54     0.31 / 0.26
//     64 of 4096 x 4096, 8 levels              29.1 / 2.52    0.33 / 1.51      100 000 x 512, 8 levels           11.9 / 0.122    0.69 / 0.068
//     200 of 700 x 1000, 8 levels              2.12 / 0.90    0.20 / 0.49      256 x 64, 16 levels               0.070 / 0.041   0.040 / 0.037
// Slower at a local optimum are most fp64 instances, whose tests cost twice and whose keys are 16 bytes (all pairs, this one; the same at a
// rounded start): one of 2048 x 8192, 16 levels, 0.50 and 0.79 (1.42, 0.35), four 1.83 and 2.38 (1.92, 0.45); 16 000 x 300, 8 levels,
// 0.060 and 0.090 (2.00, 0.16); 700 x 1000, 8 levels, 0.066 and 0.092 (0.40, 0.079); 2048 x 512, 2 levels, 0.054 and 0.065 (0.61, 0.067).
template <class T> struct SwapKey;
template <> struct SwapKey<float> {                        // level 8 bits | entry, as ordered bits, 32 | variable 16
    uint64_t k;
    __device__ __forceinline__ void set(uint32_t lev, float y, uint32_t j) {
        uint32_t b = __float_as_uint(y);
        b = (b & 0x80000000u) ? ~b : b | 0x80000000u;
        k = ((uint64_t)lev << 48) | ((uint64_t)b << 16) | j;
    }
    __device__ __forceinline__ bool less(const SwapKey& o) const { return k < o.k; }
    __device__ __forceinline__ uint32_t level() const { return (uint32_t)(k >> 48); }
    __device__ __forceinline__ uint32_t var() const { return (uint32_t)k & 0xFFFFu; }
    __device__ __forceinline__ float entry() const {
        const uint32_t b = (uint32_t)(k >> 16);
        return __uint_as_float((b & 0x80000000u) ? b ^ 0x80000000u : ~b);
    }
};
template <> struct SwapKey<double> {
    double y;
    uint32_t lev, j;
    __device__ __forceinline__ void set(uint32_t l, double v, uint32_t var) { lev = l; y = v; j = var; }
    __device__ __forceinline__ bool less(const SwapKey& o) const {
        return lev != o.lev ? lev < o.lev : y != o.y ? y < o.y : j < o.j;
    }
    __device__ __forceinline__ uint32_t level() const { return lev; }
    __device__ __forceinline__ uint32_t var() const { return j; }
    __device__ __forceinline__ double entry() const { return y; }
};

constexpr int SWI_LEVELS = 64;                 // most levels (one byte each, and a lane to look each up)
constexpr int SWI_NMIN = 64;                   // fewest variables
constexpr int SWI_NMAX = 8192;                 // most variables
constexpr int SWI_EACH = SWI_NMAX / SWE_BLOCK; // of them a thread holds
constexpr int SWI_LROWS = 3;                   // filter rows in LDS at most
constexpr int SWI_STAGES = 5;
constexpr int64_t SWI_FEW = 1 << 17;           // pairs of an instance up to which two stages are enough
constexpr int SWI_ROWS = 8;                    // of the others, those tried a lane a pair, and one more for every 1024 rows that a
                                               // pair left over is evaluated on
constexpr int SWI_SEEN = 8;                    // rows that pairs have failed at, remembered by a workgroup
constexpr int SWI_HOT = 4;                     // rows of large |entry| looked up per variable, where they are known
constexpr int SWI_PART = 1024;                 // pairs of a unit one wavefront takes at a time
constexpr int SWI_SHARED = 128;                // larger units a workgroup can have on its list
constexpr size_t SWI_LDS = 152 * 1024;          // dynamic LDS at most: the registers leave room for one workgroup a compute unit

// what lies in the dynamic LDS of a workgroup (the sort's keys overlap everything)
struct SwapLds {
    size_t y, lr, queue, rtop, rows, perm, lev, bytes;
    int32_t L;
    bool stage_r;
};
static SwapLds swap_lds(int64_t m, int64_t n, int32_t K, size_t esz, size_t key) {
    SwapLds s;
    int64_t n2 = 64;
    while (n2 < n) n2 *= 2;
    auto up = [](size_t v) { return (v + 15) / 16 * 16; };
    size_t at = 0;
    s.queue = at; at = up(at + (size_t)SWE_WAVES * SWE_QCAP * sizeof(uint32_t));
    s.rtop = at; at = up(at + (size_t)K * esz);
    s.rows = at; at = up(at + (size_t)K * sizeof(int32_t));
    s.perm = at; at = up(at + (size_t)n * 2);
    s.lev = at; at = up(at + (size_t)n);
    const size_t row = up((size_t)n * esz), rr = up((size_t)m * esz);
    s.stage_r = at + row + rr <= SWI_LDS;
    s.lr = at;
    if (s.stage_r) at += rr;
    s.y = at;
    s.L = 0;
    while (s.L < SWI_LROWS && s.L < K && at + row <= SWI_LDS) { at += row; ++s.L; }
    s.bytes = at > key * (size_t)n2 ? at : key * (size_t)n2;
    if (s.bytes > SWI_LDS) s.L = 0;
    return s;
}

template <class T>
__global__ __launch_bounds__(SWE_BLOCK) void k_swap_intervals(
    int64_t m, int32_t n, int64_t R, int32_t nd, int32_t nb, int32_t slices, bool few, int32_t K, SwapLds lds, const T* __restrict__ A,
    int64_t lda, const T* __restrict__ At, const T* __restrict__ D, const T* __restrict__ scale,
    const int32_t* __restrict__ kidx, const T* __restrict__ r, const InstState<T>* __restrict__ st,
    const uint8_t* __restrict__ var_mask, const int32_t* __restrict__ rows_all,
    const uint16_t* __restrict__ hot, int32_t n_hot,
    const int32_t* __restrict__ skip, T* gbest, Partial<T>* __restrict__ part) {
    extern __shared__ __align__(16) unsigned char sw_smem[];
    SwapKey<T>* keys = reinterpret_cast<SwapKey<T>*>(sw_smem);
    T* y = reinterpret_cast<T*>(sw_smem + lds.y);          // [L][n] filter rows, sorted order
    T* lr = reinterpret_cast<T*>(sw_smem + lds.lr);        // [m] (stage_r)
    T* rtop = reinterpret_cast<T*>(sw_smem + lds.rtop);    // [K]
    int32_t* sh_rows = reinterpret_cast<int32_t*>(sw_smem + lds.rows);
    uint16_t* perm = reinterpret_cast<uint16_t*>(sw_smem + lds.perm);
    uint8_t* lev = reinterpret_cast<uint8_t*>(sw_smem + lds.lev);
    __shared__ T sh_dl[SWI_LEVELS];
    __shared__ int32_t sh_first[SWI_LEVELS + 1];           // where every level begins
    __shared__ int32_t sh_unit[SWI_STAGES];
    __shared__ int32_t sh_big, sh_big_ready[SWI_SHARED], sh_big_unit[SWI_SHARED], sh_big_next[SWI_SHARED], sh_big_parts[SWI_SHARED];
    __shared__ T sh_big_thr[SWI_SHARED], sh_big_inner[SWI_SHARED];
    __shared__ int32_t sh_fail[SWI_SEEN], sh_fails;
    __shared__ unsigned long long sh_best;
    __shared__ T sh_s[SWE_WAVES];
    __shared__ int64_t sh_c[SWE_WAVES];

    const int64_t q = blockIdx.x;
    const int blk = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    Partial<T>* out = part + q * nb + blk;
    if (skip && skip[q]) {
        if (tid == 0) { Partial<T> e; e.s = (T)0; e.c = -1; *out = e; }
        return;
    }
    const int32_t* __restrict__ rows_g = rows_all + q * K;
    const uint8_t* __restrict__ vm = var_mask ? var_mask + q * n : nullptr;

    // ---- sort (bitonic; variables that may not move, and the padding, come last) -----------
    int32_t n2 = 64;
    while (n2 < n) n2 *= 2;
    {
        const int64_t row = rows_g[0];
        int32_t kk[SWI_EACH];
        T yy[SWI_EACH];
#pragma unroll
        for (int e = 0; e < SWI_EACH; ++e) {
            const int32_t j = tid + e * SWE_BLOCK, jc = j < n ? j : n - 1;
            kk[e] = kidx[(int64_t)jc * R + q];
            yy[e] = At ? At[row * n + jc] : A[row + jc * lda];
            if (j >= n || (vm && !vm[jc])) kk[e] = 255;
        }
#pragma unroll
        for (int e = 0; e < SWI_EACH; ++e) {
            const int32_t j = tid + e * SWE_BLOCK;
            if (j < n2) { SwapKey<T> key; key.set((uint32_t)kk[e], yy[e], (uint32_t)j); keys[j] = key; }
        }
        if (tid < nd) sh_dl[tid] = D[tid];
        if (tid < SWI_STAGES) sh_unit[tid] = 0;
        if (tid < SWI_SHARED) { sh_big_ready[tid] = 0; sh_big_next[tid] = 0; }
        if (tid < SWI_SEEN) sh_fail[tid] = rows_g[0];
        if (tid == 0) { sh_big = 0; sh_fails = 0; }
        if (tid == 0) sh_best = order_bits(Limits<T>::inf());
        __syncthreads();
        for (int32_t k = 2; k <= n2; k <<= 1) {
            for (int32_t d = k >> 1; d > 0; d >>= 1) {
                for (int32_t p = tid; p < n2 >> 1; p += SWE_BLOCK) {
                    const int32_t a = 2 * p - (p & (d - 1)), b = a + d;
                    const SwapKey<T> ka = keys[a], kb = keys[b];
                    if (kb.less(ka) == ((a & k) == 0)) { keys[a] = kb; keys[b] = ka; }
                }
                // pairs at most 64 apart stay inside the 128 keys of one wavefront
                if (d > 64 || (d == 1 && k >= 128)) __syncthreads();
                else { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); }
            }
        }
        __syncthreads();
        if (tid <= nd) {                                   // first position of every level
            int32_t lo = 0, hi = n;
            while (lo < hi) {
                const int32_t mid = (lo + hi) >> 1;
                if ((int32_t)keys[mid].level() < tid) lo = mid + 1; else hi = mid;
            }
            sh_first[tid] = lo;
        }
        SwapKey<T> mine[SWI_EACH];
#pragma unroll
        for (int e = 0; e < SWI_EACH; ++e) if (tid + e * SWE_BLOCK < n) mine[e] = keys[tid + e * SWE_BLOCK];
        __syncthreads();
        // the other filter rows: read along the row, then put in order in place
        for (int l = 1; l < lds.L; ++l) {
            const int64_t row_l = rows_g[l];
            for (int32_t j = tid; j < n; j += SWE_BLOCK) y[l * n + j] = At ? At[row_l * n + j] : A[row_l + j * lda];
        }
#pragma unroll
        for (int e = 0; e < SWI_EACH; ++e) {
            const int32_t p = tid + e * SWE_BLOCK;
            if (p < n) {
                perm[p] = (uint16_t)mine[e].var();
                lev[p] = (uint8_t)mine[e].level();
                y[p] = mine[e].entry();
            }
        }
        __syncthreads();
        for (int l = 1; l < lds.L; ++l) {
            T v[SWI_EACH];
#pragma unroll
            for (int e = 0; e < SWI_EACH; ++e) {
                // (a masked variable's place may hold a padding number: its entries are never looked at)
                const int32_t p = tid + e * SWE_BLOCK, j = perm[p < n ? p : n - 1];
                v[e] = y[l * n + (j < n ? j : n - 1)];
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < SWI_EACH; ++e)
                if (tid + e * SWE_BLOCK < n) y[l * n + tid + e * SWE_BLOCK] = v[e];
        }
    }
    for (int l = tid; l < K; l += SWE_BLOCK) {
        const int32_t row = rows_g[l];
        sh_rows[l] = row;
        rtop[l] = r[(int64_t)row * R + q];
    }
    if (lds.stage_r)
        for (int64_t i = tid; i < m; i += SWE_BLOCK) lr[i] = r[i * R + q];
    __syncthreads();

    uint32_t* queue = reinterpret_cast<uint32_t*>(sw_smem + lds.queue) + w * SWE_QCAP;
    const T sc = scale[q], t = st[q].t, t_below = value_below(t), r1 = rtop[0];
    const int32_t nv = __builtin_amdgcn_readfirstlane(sh_first[nd]);      // variables that may move
    const int32_t groups = (nv + 63) >> 6;
    T best_t = Limits<T>::inf(), others = Limits<T>::inf();
    int64_t best_c = -1;                                   // the wavefront's record (uniform)
    auto bound = [&]() -> T {
        T shared_t;
        from_order_bits(__hip_atomic_load(&sh_best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP), shared_t);
        return dmmv_min(dmmv_min(best_t, others), shared_t);
    };

    // The first `cnt` queued pairs, a lane each, on a few rows: more of large |r|, those that pairs failed at before, and
    // those of the two variables' largest entries (a swap of an outlier channel makes its new maximum there).  Then on
    // every row, the pair of the smallest error seen so far first, so that what it finds drops most others; and where it
    // finds nothing, the row it failed at is tried on the others.
    auto drain = [&](int cnt) {
        if (gbest) others = __hip_atomic_load(gbest + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool alive = lane < cnt;
        const uint32_t e = queue[alive ? lane : 0];
        const int32_t pu = (int32_t)(e >> 16), pv = (int32_t)(e & 0xFFFFu);
        const int64_t u = perm[pu], v = perm[pv];
        const T Ds = sc * (sh_dl[lev[pu]] - sh_dl[lev[pv]]);
        T seen = (T)0;                                     // largest |r'| on the rows tried
        for (int k = 0; k < lds.L; ++k) seen = dmmv_max(seen, dmmv_abs(dmmv_fma(Ds, y[k * n + pv] - y[k * n + pu], rtop[k])));
        T thr = dmmv_min(bound(), t_below);
        alive = alive && seen <= thr;
        auto r_at = [&](int64_t i) -> T { return lds.stage_r ? lr[i] : r[i * R + q]; };
        auto a_at = [&](int64_t i, int64_t j) -> T { return At ? At[i * n + j] : A[i + j * lda]; };
        auto rows4 = [&](int64_t i0, int64_t i1, int64_t i2, int64_t i3) {
            const T v0 = a_at(i0, v), v1 = a_at(i1, v), v2 = a_at(i2, v), v3 = a_at(i3, v);
            const T u0 = a_at(i0, u), u1 = a_at(i1, u), u2 = a_at(i2, u), u3 = a_at(i3, u);
            seen = dmmv_max(seen, dmmv_abs(dmmv_fma(Ds, v0 - u0, r_at(i0))));
            seen = dmmv_max(seen, dmmv_abs(dmmv_fma(Ds, v1 - u1, r_at(i1))));
            seen = dmmv_max(seen, dmmv_abs(dmmv_fma(Ds, v2 - u2, r_at(i2))));
            seen = dmmv_max(seen, dmmv_abs(dmmv_fma(Ds, v3 - u3, r_at(i3))));
            alive = seen <= thr;
        };
        const int n_rows = SWI_ROWS + (int)min(m >> 10, (int64_t)SWAP_KMAX), l_end = lds.L + n_rows < K ? lds.L + n_rows : K;
        const int tries = l_end - lds.L + SWI_SEEN;        // sh_rows[L .. l_end), then sh_fail
        for (int l0 = 0; l0 < tries && __any(alive); l0 += 4) {
            if (alive) {
                auto row = [&](int l) -> int32_t {
                    l = l < tries ? l : tries - 1;
                    return lds.L + l < l_end ? sh_rows[lds.L + l] : sh_fail[lds.L + l - l_end];
                };
                rows4(row(l0), row(l0 + 1), row(l0 + 2), row(l0 + 3));
            }
        }
        for (int h = 0; h < n_hot && __any(alive); h += 2) {
            if (alive) {
                int32_t row[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int64_t at = (int64_t)(h + x / 2 < n_hot ? h + x / 2 : h) * n + (x & 1 ? v : u);
                    row[x] = hot[at];
                }
                rows4(row[0], row[1], row[2], row[3]);
            }
        }
        while (true) {
            alive = alive && seen <= thr;
            if (!__any(alive)) break;
            const T least = wave_min(alive ? seen : Limits<T>::inf());
            const int src = __builtin_ctzll(__ballot(alive && seen == least));
            alive = alive && lane != src;
            const uint32_t se = (uint32_t)__builtin_amdgcn_readlane((int)e, src);
            const int32_t su = (int32_t)(se >> 16), sv = (int32_t)(se & 0xFFFFu);
            const int64_t ju = __builtin_amdgcn_readfirstlane(perm[su]), jv = __builtin_amdgcn_readfirstlane(perm[sv]);
            const T Dl = sc * (sh_dl[lev[su]] - sh_dl[lev[sv]]);
            const T* __restrict__ Au = A + ju * lda;
            const T* __restrict__ Av = A + jv * lda;
            if (gbest) others = __hip_atomic_load(gbest + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            T val = (T)0, wm = (T)0;
            int32_t at = 0;                                // the lane's row of val
            bool ok = true;
            for (int64_t base = 0; base < m && ok; base += 256) {
                T a[4], b[4], rr[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int64_t i = base + x * 64 + lane, ic = i < m ? i : m - 1;
                    a[x] = Au[ic];
                    b[x] = Av[ic];
                    rr[x] = r_at(ic);
                }
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const T w1 = dmmv_abs(dmmv_fma(Dl, b[x] - a[x], rr[x]));
                    const int64_t i = base + x * 64 + lane;
                    if (w1 > val) { val = w1; at = (int32_t)(i < m ? i : m - 1); }
                }
                wm = wave_max(val);
                ok = wm < t && !(wm > bound());         // (what the others have found meanwhile included)
            }
            if (ok) {
                const int64_t c = ju * n + jv;
                if (rec_less(wm, c, best_t, best_c)) {
                    best_t = wm;
                    best_c = c;
                    if (lane == 0) {
                        atomicMin(&sh_best, order_bits(wm));
                        if (gbest) share_best(gbest + q, wm);
                    }
                }
            } else {
                const int64_t row = __builtin_amdgcn_readlane(at, __builtin_ctzll(__ballot(val == wm)));
                if (lane == 0) sh_fail[atomicAdd(&sh_fails, 1) & (SWI_SEEN - 1)] = (int32_t)row;
                if (alive) seen = dmmv_max(seen, dmmv_abs(dmmv_fma(Ds, a_at(row, v) - a_at(row, u), r_at(row))));
            }
            thr = dmmv_min(bound(), t_below);
        }
    };

    const unsigned long long below = (1ull << lane) - 1ull;
    const int32_t units = groups * nd * slices;
    int qn = 0;                                            // queued pairs (uniform)
    // The pairs of a unit within thr0 and, from the second stage on, not within `inner`, which the stage before has seen to;
    // by lane: `upto` pairs up to and with this lane's, which are its variable with positions start + (number of the pair),
    // from gap_at on `gap` further.  Returns how many there are.
    int32_t upto = 0, start = 0, gap_at = 0, gap = 0, first_u = 0, first_v = 0;
    T Ds = (T)0;
    auto search = [&](int32_t unit, T thr0, T inner) -> int32_t {
        const int32_t slice = unit & (slices - 1), b = unit / slices / groups, g = unit / slices % groups;
        const int32_t s0 = __builtin_amdgcn_readfirstlane(sh_first[b]), len = __builtin_amdgcn_readfirstlane(sh_first[b + 1]) - s0;
        const int32_t pu = g * 64 + lane, puc = pu < nv ? pu : nv - 1;
        const int32_t lu = lev[puc];
        bool on = len > 0 && pu < nv && lu > b && (lane & (slices - 1)) == slice;
        if (!__any(on)) return 0;
        const T yu = y[puc];
        Ds = sc * (sh_dl[lu] - sh_dl[b]);
        auto f = [&](int32_t p) -> T { return dmmv_fma(Ds, y[p] - yu, r1); };
        const T f0 = f(s0), f1 = f(s0 + len - 1);
        on = on && f0 <= thr0 && f1 >= -thr0;              // (false where the step is not finite and gives no number)
        if (!__any(on)) return 0;
        int32_t top = 1;
        while (2 * top <= len) top *= 2;
        // how many of the level's variables have f <= v, and f < v; a bisection where some lane's are not all of them, or none
        auto up_to = [&](T v) -> int32_t {
            if (!__any(on && !(f1 <= v))) return len;
            int32_t at = 0;
            for (int32_t d = top; d > 0; d >>= 1) {
                const int32_t p = at + d;
                if (p <= len && f(s0 + (p < len ? p : len) - 1) <= v) at = p;
            }
            return at;
        };
        auto below_of = [&](T v) -> int32_t {
            if (!__any(on && !(f0 >= v))) return 0;
            int32_t at = 0;
            for (int32_t d = top; d > 0; d >>= 1) {
                const int32_t p = at + d;
                if (p <= len && !(f(s0 + (p < len ? p : len) - 1) >= v)) at = p;
            }
            return at;
        };
        const int32_t hi = up_to(thr0), lo = below_of(-thr0);
        int32_t in0 = lo, in1 = lo;
        if (inner >= (T)0) {                               // (thr0 may have come below `inner`: then nothing is left)
            in0 = below_of(-inner);
            in1 = up_to(inner);
            in0 = in0 > lo ? in0 : lo;
            in1 = in1 < hi ? in1 : hi;
            in1 = in1 > in0 ? in1 : in0;
        }
        const int32_t cnt = on && hi > lo ? hi - lo - (in1 - in0) : 0;
        upto = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t v = __shfl_up(upto, off, 64);
            if (lane >= off) upto += v;
        }
        start = s0 + lo - (upto - cnt);
        gap_at = s0 + in0;
        gap = in1 - in0;
        first_u = g * 64;
        first_v = s0;
        return __builtin_amdgcn_readlane(upto, 63);
    };
    // the 64 pairs from x0 of the unit searched last: the filter rows in LDS, what is left goes to the queue
    auto look = [&](int32_t x0, int32_t x1) {
        const int32_t x = x0 + lane;
        int32_t l = 0;                                     // lanes whose pairs all come before pair x
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            const int32_t v = __shfl(upto, l + d - 1, 64);
            if (v <= x) l += d;
        }
        bool alive = x < x1;
        const int32_t pa = first_u + l, at = __shfl(start, l, 64) + x;
        const int32_t hole = __shfl(gap_at, l, 64), wide = __shfl(gap, l, 64);
        const int32_t pb = alive ? at + (at >= hole ? wide : 0) : first_v;
        const T Dp = __shfl(Ds, l, 64);
        const T thr = dmmv_min(bound(), t_below);
        const int32_t pac = pa < nv ? pa : nv - 1;
        for (int k = 1; k < lds.L; ++k) {
            const T val = dmmv_abs(dmmv_fma(Dp, y[k * n + pb] - y[k * n + pac], rtop[k]));
            alive = alive & (val <= thr);
        }
        const unsigned long long bal = __ballot(alive);
        if (alive) queue[qn + __popcll(bal & below)] = ((uint32_t)pa << 16) | (uint32_t)pb;
        qn += __popcll(bal);
        __builtin_amdgcn_wave_barrier();
    };
    // The next pairs of stage s, [x0, x1) of a unit that has been searched: a unit of the stage, or when these are all
    // taken a part of one on the workgroup's list.  (Its writer comes to the list after writing, so none is left
    // over; an entry that is not ready yet is its writer's to see to.)
    int slot = 0;
    auto next = [&](int s, T reach, T inner, int32_t& x0, int32_t& x1) -> bool {
        while (true) {
            int32_t id = 0;
            if (lane == 0) id = atomicAdd(&sh_unit[s], 1);
            const int64_t unit = blk + (int64_t)nb * __builtin_amdgcn_readfirstlane(id);
            int32_t u_next, parts = 0, p = 0;
            T thr0, inner0 = inner;
            if (unit < units) {
                u_next = (int32_t)unit;
                thr0 = dmmv_min(bound(), reach);
            } else {
                if (slot >= SWI_SHARED || slot >= __builtin_amdgcn_readfirstlane(__hip_atomic_load(&sh_big, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))) return false;
                if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(&sh_big_ready[slot], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP))) {
                    parts = __builtin_amdgcn_readfirstlane(sh_big_parts[slot]);
                    if (lane == 0) p = atomicAdd(&sh_big_next[slot], 1);
                    p = __builtin_amdgcn_readfirstlane(p);
                }
                if (p >= parts) { ++slot; continue; }
                u_next = __builtin_amdgcn_readfirstlane(sh_big_unit[slot]);
                thr0 = sh_big_thr[slot];
                inner0 = sh_big_inner[slot];
            }
            x0 = 0;
            x1 = search(u_next, thr0, inner0);
            if (parts > 0) {
                x0 = p * SWI_PART;
                x1 = x0 + SWI_PART < x1 ? x0 + SWI_PART : x1;
            } else if (x1 > SWI_PART) {                    // a large one goes on the list, if there is room
                int32_t to = 0;
                if (lane == 0) to = atomicAdd(&sh_big, 1);
                to = __builtin_amdgcn_readfirstlane(to);
                if (to < SWI_SHARED) {
                    if (lane == 0) {
                        sh_big_unit[to] = u_next;
                        sh_big_parts[to] = (x1 + SWI_PART - 1) / SWI_PART;
                        sh_big_thr[to] = thr0;
                        sh_big_inner[to] = inner0;
                        __hip_atomic_store(&sh_big_ready[to], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    slot = to < slot ? to : slot;
                    x1 = 0;                                // (if it is all taken when this wavefront gets there, nothing is left)
                    continue;
                }
            }
            if (x0 < x1) return true;
        }
    };
    T inner = (T)-1;                                       // (nothing yet)
    for (int s = 0; s < SWI_STAGES; ++s) {
        const T share[SWI_STAGES] = {(T)0.75, (T)0.875, (T)0.9375, (T)0.96875, (T)1};
        if (few && s != 2 && s != SWI_STAGES - 1) continue;
        const T reach = dmmv_min(t * share[s], t_below);   // (the last one: t_below)
        if (gbest) others = __hip_atomic_load(gbest + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (bool more = true; more;) {
            int32_t x0 = 0, x1 = 0;
            more = next(s, reach, inner, x0, x1);
            do {
                if (x0 < x1) look(x0, x1);
                x0 += 64;
                if (qn >= 64 || (!more && qn > 0)) {       // (what is queued when nothing is left to take: at the end)
                    drain(qn < 64 ? qn : 64);
                    const uint32_t carry = 64 + lane < qn ? queue[64 + lane] : 0;
                    __builtin_amdgcn_wave_barrier();
                    if (64 + lane < qn) queue[lane] = carry;
                    __builtin_amdgcn_wave_barrier();
                    qn = qn > 64 ? qn - 64 : 0;
                }
            } while (x0 < x1 || (!more && qn > 0));
        }
        if (reach >= dmmv_min(bound(), t_below)) break;
        inner = reach;
    }
    if (lane == 0) { sh_s[w] = best_t; sh_c[w] = best_c; }
    __syncthreads();
    if (tid == 0) {
        T bs = sh_s[0];
        int64_t bc = sh_c[0];
        for (int x = 1; x < SWE_WAVES; ++x)
            if (rec_less(sh_s[x], sh_c[x], bs, bc)) { bs = sh_s[x]; bc = sh_c[x]; }
        Partial<T> p;
        p.s = bc < 0 ? (T)0 : bs;
        p.c = bc;
        *out = p;
    }
}

// ---- reduce the records of an instance, report, and carry the swap out.  One workgroup per
// instance.
template <class T>
__global__ __launch_bounds__(SW_BLOCK) void k_swap_apply(
    int64_t m, int64_t n, int64_t R, int32_t nb, int32_t apply, const T* __restrict__ A, int64_t lda,
    const T* __restrict__ D, const T* __restrict__ scale, int32_t* __restrict__ kidx,
    T* __restrict__ r, InstState<T>* __restrict__ st, const Partial<T>* __restrict__ part,
    int32_t* __restrict__ skip, int32_t mark_skip, dmmv_swap* __restrict__ best_out,
    T* __restrict__ best_t_out) {
    __shared__ T sh_s[SW_WAVES];
    __shared__ int64_t sh_c[SW_WAVES];
    __shared__ T sh_bs;
    __shared__ int64_t sh_bc;
    const int64_t q = blockIdx.x;
    if (skip && skip[q]) {
        if (threadIdx.x == 0) {
            if (best_out) { best_out[q].i = -1; best_out[q].j = -1; }
            if (best_t_out) best_t_out[q] = st[q].t;
        }
        return;
    }
    T s = (T)0;
    int64_t c = -1;
    for (int e = threadIdx.x; e < nb; e += SW_BLOCK) {
        const Partial<T> p = part[q * nb + e];
        if (rec_less(p.s, p.c, s, c)) { s = p.s; c = p.c; }
    }
    block_argmin(s, c, sh_s, sh_c);
    if (threadIdx.x == 0) { sh_bs = s; sh_bc = c; }
    __syncthreads();
    s = sh_bs;
    c = sh_bc;
    if (threadIdx.x == 0) {
        if (best_out) { best_out[q].i = c < 0 ? -1 : c / n; best_out[q].j = c < 0 ? -1 : c % n; }
        if (best_t_out) best_t_out[q] = c < 0 ? st[q].t : s;
        if (c < 0 && skip && mark_skip) skip[q] = 1;
    }
    if (c < 0 || !apply) return;
    const int64_t i = c / n, j = c % n;
    const int32_t ki = kidx[i * R + q], kj = kidx[j * R + q];
    const T diff = D[ki] - D[kj];
    const T Delta = scale[q] * diff;
    const T* __restrict__ Ai = A + i * lda;
    const T* __restrict__ Aj = A + j * lda;
    for (int64_t k = threadIdx.x; k < m; k += SW_BLOCK)
        r[k * R + q] = dmmv_fma(Delta, Aj[k] - Ai[k], r[k * R + q]);
    __syncthreads();                                       // every thread has read ki and kj
    if (threadIdx.x == 0) {
        kidx[i * R + q] = kj;
        kidx[j * R + q] = ki;
        st[q].t = s;
        st[q].moves += 1;
    }
}

__global__ void k_swap_clear(int32_t* skip, int64_t R) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q < R) skip[q] = 0;
}

// pairs of an instance whose variables are spread evenly over the levels
static int64_t swap_pairs(int64_t n, int32_t nd) { return n * n / 2 * (nd - 1) / nd; }

// Workgroups per instance: as many as the chip holds, one a compute unit, as long as each has some pairs (every one of them sorts
// for itself) - SWI_PAIRS of a single instance.  Several instances get up to four times as many pairs a workgroup: at a rounded
// start every workgroup has to find a good swap of its own before it learns of the others' (20 of 2048 x 512, 16 levels, 0.12 against
// 0.14 ms), at a local optimum they are the slower ones (4 of them 0.11 against 0.10).  Slices of units until every
// wavefront has two, while they hold SWI_SLICE pairs on the average.
constexpr int64_t SWI_PAIRS = 4096, SWI_SLICE = 256;
static void swap_sorted_grid(int64_t n, int64_t R, int32_t nd, int32_t most, int32_t* nb_out, int32_t* slices_out) {
    const int64_t units = ceil_div(n, 64) * nd, pairs = swap_pairs(n, nd);
    int64_t nb = ceil_div(256, R);
    const int64_t some = ceil_div(pairs, SWI_PAIRS * (R < 4 ? R : 4));
    if (nb > some) nb = some;
    if (nb > most) nb = most;
    if (nb < 1) nb = 1;
    int32_t slices = 1;
    while (slices < 64 && units * slices < nb * 2 * SWE_WAVES && pairs / (units * slices) > SWI_SLICE) slices *= 2;
    *nb_out = (int32_t)nb;
    *slices_out = slices;
}

template <class T>
dmmv_status swap_t(Ctx* c, int32_t k_eps, int32_t apply, bool use_skip, dmmv_swap* best, void* best_t) {
    const int64_t m = c->p.m, n = c->p.n, R = c->p.R;
    if (R == 0) return DMMV_OK;
    int32_t K = k_eps > 0 ? k_eps : 100;
    if (K > SWAP_KMAX) K = SWAP_KMAX;
    if ((int64_t)K > m) K = (int32_t)m;
    int32_t nb = c->swap_nb;
    int32_t* skip = use_skip ? c->swap_skip : nullptr;
    // A batch's workgroups share the best t' of their instance, so that what one finds prunes the others' pairs
    // (the buffer of the descent's packed scales is free outside a descent's loop).
    T* gbest = c->kind == KIND_BATCHED && nb > 1 ? (T*)c->cmp_scale : nullptr;
    // LDS: the K residuals and rows always; then D[k_j] and filter rows of A
    size_t used = (size_t)K * (sizeof(T) + sizeof(int32_t)) + 64;
    const bool dvl = used + (size_t)n * sizeof(T) <= SW_LDS_BUDGET;
    if (dvl) used += (size_t)n * sizeof(T);
    int64_t L = n > 0 ? (int64_t)((SW_LDS_BUDGET - used) / ((size_t)n * sizeof(T))) : 0;
    if (L > K) L = K;
    used += (size_t)L * n * sizeof(T);

    // Sorted variables where their keys and filter rows fit.  Under 64 variables the sort costs more than it saves
    // (100 x 17: 42 us without, 49 with; 256 x 64: 70 and 40).
    const bool sorted = K > 0 && n >= SWI_NMIN && n <= SWI_NMAX && c->p.nd <= SWI_LEVELS;
    SwapLds lds = {};
    int32_t slices = 1;
    if (sorted) lds = swap_lds(m, n, K, sizeof(T), sizeof(SwapKey<T>));
    if (lds.L > 0) {
        swap_sorted_grid(n, R, c->p.nd, c->swap_nb, &nb, &slices);
        // (a single instance has two words among the flags, which nothing else looks at)
        gbest = nb == 1 ? nullptr : c->kind == KIND_BATCHED ? (T*)c->cmp_scale : (T*)(c->flags + FLAG_SWAP_BEST);
    }
    if (K > 0)
        hipLaunchKernelGGL(k_swap_top<T>, dim3((unsigned)R), dim3(SW_BLOCK), 0, c->stream, m, R, K, (const T*)c->r,
                           (const int32_t*)skip, c->swap_rows, gbest);
    if (lds.L > 0) {
        // Rows of large entries, where the evaluation's lists of a batch are there.  Looking for them by a pass over A in every
        // search took longer than it saved: a single instance of 100 000 x 2000 (ms) 0.82 / 1.25, without 0.71 / 0.99.
        const uint16_t* hot = batched_lists_in_use(c) ? c->lists.crow : nullptr;
        DMMV_TRY(ensure_dynamic_lds(reinterpret_cast<const void*>(&k_swap_intervals<T>), (int)SWI_LDS));
        hipLaunchKernelGGL(k_swap_intervals<T>, dim3((unsigned)R, (unsigned)nb), dim3(SWE_BLOCK), lds.bytes, c->stream,
                           m, (int32_t)n, R, c->p.nd, nb, slices, swap_pairs(n, c->p.nd) <= SWI_FEW, K, lds, (const T*)c->p.A_dense, c->p.lda,
                           (const T*)(c->kind == KIND_BATCHED ? c->Xt : nullptr), (const T*)c->D_dev,
                           (const T*)c->scale_dev, (const int32_t*)c->kidx, (const T*)c->r,
                           (const InstState<T>*)c->state, c->o.var_mask, (const int32_t*)c->swap_rows,
                           hot, hot ? SWI_HOT : 0, (const int32_t*)skip, gbest, (Partial<T>*)c->swap_part);
    } else {
        DMMV_TRY(ensure_dynamic_lds(reinterpret_cast<const void*>(&k_swap_eval<T, true>), (int)SW_LDS_BUDGET));
        DMMV_TRY(ensure_dynamic_lds(reinterpret_cast<const void*>(&k_swap_eval<T, false>), (int)SW_LDS_BUDGET));
#define DMMV_SWAP_LAUNCH(DV)                                                                               \
        hipLaunchKernelGGL((k_swap_eval<T, DV>), dim3((unsigned)R, (unsigned)nb), dim3(SWE_BLOCK), used, c->stream, m, n, R, nb, K,       \
                           (int32_t)L, (const T*)c->p.A_dense, c->p.lda,                                       \
                           (const T*)(c->kind == KIND_BATCHED ? c->Xt : nullptr), (const T*)c->D_dev,          \
                           (const T*)c->scale_dev, (const int32_t*)c->kidx, (const T*)c->r,                    \
                           (const InstState<T>*)c->state, c->o.var_mask, (const int32_t*)c->swap_rows,         \
                           (const int32_t*)skip, gbest, (Partial<T>*)c->swap_part)
        if (dvl) DMMV_SWAP_LAUNCH(true);
        else DMMV_SWAP_LAUNCH(false);
#undef DMMV_SWAP_LAUNCH
    }
    hipLaunchKernelGGL(k_swap_apply<T>, dim3((unsigned)R), dim3(SW_BLOCK), 0, c->stream, m, n, R, nb, apply,
                       (const T*)c->p.A_dense, c->p.lda, (const T*)c->D_dev, (const T*)c->scale_dev, c->kidx,
                       (T*)c->r, (InstState<T>*)c->state, (const Partial<T>*)c->swap_part, skip,
                       use_skip ? 1 : 0, best, (T*)best_t);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

}  // namespace

int32_t swap_blocks_per_instance(const dmmv_problem& p) {
    // about 2048 workgroups in all, at most one per first variable
    int64_t nb = ceil_div(2048, p.R > 0 ? p.R : 1);
    if (nb > p.n) nb = p.n;
    if (nb < 1) nb = 1;
    return (int32_t)nb;
}

dmmv_status swap_clear_skip(Ctx* c) {
    if (!c->swap_skip) return fail(DMMV_ERR_STATE, "swap move: workspace is missing");
    if (c->p.R == 0) return DMMV_OK;
    hipLaunchKernelGGL(k_swap_clear, dim3((unsigned)ceil_div(c->p.R, 256)), dim3(256), 0, c->stream, c->swap_skip,
                       c->p.R);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

dmmv_status swap_move(Ctx* c, int32_t k_eps, int32_t apply, bool use_skip, dmmv_swap* best, void* best_t) {
    if (c->kind == KIND_CSC) return swap_move_csc(c, apply, use_skip, best, best_t);
    if (!c->swap_skip || !c->swap_rows || !c->swap_part)
        return fail(DMMV_ERR_STATE, "swap move: workspace is missing");
    return c->p.dtype == DMMV_F64 ? swap_t<double>(c, k_eps, apply, use_skip, best, best_t)
                                  : swap_t<float>(c, k_eps, apply, use_skip, best, best_t);
}

}  // namespace dmmv
