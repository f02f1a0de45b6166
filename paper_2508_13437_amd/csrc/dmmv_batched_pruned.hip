// Batched instances: the descent with exact pruning (options.prune), one workgroup per instance.
//
// The score of a move (j, k) is a maximum over all m rows, so the maximum over ANY subset of the
// rows is a lower bound of it, and a move can only win if its lower bound is below the score of
// the best move known (Corollary 1 turns the same observation into a filter for swaps: a move
// that does not fix the rows of largest |r| cannot improve).  Per iteration the workgroup
//   1. picks S = 16 screening rows: the rows with |r| above a bound are listed while the move before is applied, the 16
//      largest of them by rank (the row of largest |r| overall is always the first); the bound follows the 22nd
//      largest, which a single move hardly changes.  At the start, and where a move has left fewer than 10 or more than the list
//      holds, they are listed from all rows, with a bound that 22 rows or a few more reach;
//   2. bounds candidates from below by lb(j, k) = max_{i in S} |fma(delta, X_ij, r_i)| - 16 rows instead
//      of m - and keeps per variable its best candidate by (lb, k), found by walking outwards from
//      the current level on the side that lowers the row of largest |r| until lb rises;
//   3. takes candidates in ascending order of (lb, c), c = j nd + k - each wavefront among the
//      variables it screened - scores each one over all m rows (the same fma on
//      the same operands as the full evaluation, so the same bits); the wavefronts share the smallest score found so far
//      and do not wait for each other until their next candidate cannot win against it: every candidate not scored
//      then has score >= lb, above the best score found, or loses the tie on c;
//   4. applies the move if its score is below t.
// The result is the arg-min of the full table restricted to strictly improving moves, i.e. the
// move the full evaluation + selection would apply - found with a few full scores instead of
// n (nd - 1); a candidate's score is given up as soon as a row puts it above the best one.
// Many instances (4096 of 2048 x 4096, 16 levels, to their local optima: 8.3 ms, 9.9 before) are bound by the rows of X, 256 KiB an
// iteration, three quarters of which the L2 does not hold (8.9 TB/s into the compute units, 6.8 past the L2; the vector unit 64 % busy, 12 100 instructions an
// iteration; cycles for the four steps 2300, 35 300, 26 200, 5800); a fifth workgroup on a compute unit changes nothing.  Few instances
// are bound by latencies: 20 of 2048 x 4096 with eight wavefronts 1600, 13 700, 16 300 and 3300.
// What gave most: rows picked exactly instead of four from every wavefront's share (6.4 scores an iteration instead of 9.3); no barrier between
// scores (there were 5.5 rounds of one score a wavefront); requests ahead that are not under a condition, so that the
// compiler waits for the block it needs only.
// The listing from all rows found its bound by trial before (from 3/4 of the largest |r| on, up to seven times, then all rows): where |r| has
// a heavy tail that ended with arbitrary rows and thousands of scores for one move.  1000 instances of 500 x 1000 with 256 levels
// 3863 us, now 2263; 100 of 9000 x 100 under the outer loop 2888 and 2462, 2000 of 300 x 100 554 and 415.
// Tried and dropped: the first step on eight rows and the survivors queued for the other eight, 64 at a time (a line of X
// fetched per row and variable); a good move looked for first, to bound the others; eight more rows for the
// variables that are left; the candidates left after a wavefront's first score shared out by a queue (no gain: few are left, and
// ties cost more); sixteen wavefronts an instance; bounds and levels in one word, for a fifth workgroup.
// The instance's r (m values) and x (n level indices) live in LDS for the whole
// launch, so a launch can run any number of iterations without touching the other instances;
// an instance stops by itself at a local optimum.
#include <type_traits>

#include "dmmv_common.h"

namespace dmmv {

namespace {

constexpr int BP_S = 16;                         // screening rows
constexpr int BP_LIST = 64;                      // rows gathered to pick them from
constexpr int BP_WANT = 22;                      //   aimed at
constexpr int BP_FEWEST = 10;                    //   made do with
constexpr int64_t BP_MAX_ROWS = 16384;
constexpr int BP_DCAP = 256;                     // levels kept in LDS
constexpr size_t BP_LDS_LIMIT = 96 * 1024;       // dynamic LDS a workgroup may ask for

// the best move a wavefront has found (c < 0: none)
template <class T>
struct alignas(16) BpFound {
    T s;
    int32_t c;
};

// a non-negative number as an integer of the same order
__device__ __forceinline__ uint32_t bp_order(float v) { return __float_as_uint(v); }
__device__ __forceinline__ unsigned long long bp_order(double v) { return (unsigned long long)__double_as_longlong(v); }
__device__ __forceinline__ float bp_number(uint32_t v) { return __uint_as_float(v); }
__device__ __forceinline__ double bp_number(unsigned long long v) { return __longlong_as_double((long long)v); }

// max |f(u)| over the screening rows, three dependent steps
template <class T, class F>
__device__ __forceinline__ T bp_max(F f) {
    auto three = [](T a, T b, T c) { return dmmv_max(dmmv_max(a, b), c); };
    T p[5];
#pragma unroll
    for (int u = 0; u < 5; ++u) p[u] = three(dmmv_abs(f(3 * u)), dmmv_abs(f(3 * u + 1)), dmmv_abs(f(3 * u + 2)));
    return dmmv_max(three(p[0], p[1], p[2]), three(p[3], p[4], dmmv_abs(f(15))));
}

template <class T, int W>
struct BpShared {
    BpFound<T> found[W];                         // by each wavefront
    decltype(bp_order(T())) bound;               // smallest score found so far, t at first
    uint32_t peak[64 * W];                       // upper 32 bits of the largest |r| of every thread's rows
    int32_t list[BP_LIST];                       // rows of large |r|, the first one of largest
    int32_t listed;                              // how many there were to put behind it
};

// A candidate (j, k) as one number, ordered like the flat index: j in the upper bits, k in the lower 8 or 16 (an instance
// has under 2^15 variables: its r and x fit LDS).
// does (s, c) beat the best (bs, bc)?  bc < 0: nothing found yet, only scores below bs = t count
template <class T>
__device__ __forceinline__ bool bp_better(T s, int32_t c, T bs, int32_t bc) {
    return c >= 0 && (s < bs || (s == bs && bc >= 0 && c < bc));
}

// (score, candidate) minimum over the wavefront, the same in every lane; c < 0: no candidate
template <class T>
__device__ __forceinline__ void bp_argmin(T& s, int32_t& c) {
    const T smin = wave_min(c < 0 ? Limits<T>::inf() : s);
    uint32_t u = c >= 0 && s == smin ? (uint32_t)c : 0xFFFFFFFFu;
    u = min(u, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, DPP_QUAD_XOR1, 0xF, 0xF, true));
    u = min(u, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, DPP_QUAD_XOR2, 0xF, 0xF, true));
    u = min(u, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, DPP_ROW_HALF_MIRROR, 0xF, 0xF, true));
    u = min(u, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, DPP_ROW_MIRROR, 0xF, 0xF, true));
    const uint32_t a = min((uint32_t)__builtin_amdgcn_readlane((int)u, 0), (uint32_t)__builtin_amdgcn_readlane((int)u, 16));
    const uint32_t b = min((uint32_t)__builtin_amdgcn_readlane((int)u, 32), (uint32_t)__builtin_amdgcn_readlane((int)u, 48));
    c = (int32_t)min(a, b);
    s = smin;
}

// An entry of the row-major copy of X: uniform row offset + lane offset, in bytes (an instance's r and x fit LDS, which
// keeps the copy under 2^32 bytes).  A buffer load takes both as they are; a pointer per row costs a 64-bit addition
// per load and twice the scalar registers.
__device__ __forceinline__ float bp_entry(const __amdgpu_buffer_rsrc_t& rs, uint32_t lane_off, uint32_t row_off, float) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)lane_off, (int)row_off, 0));
}
__device__ __forceinline__ double bp_entry(const __amdgpu_buffer_rsrc_t& rs, uint32_t lane_off, uint32_t row_off, double) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)lane_off, (int)row_off, 0);
    return __hiloint2double((int)v[1], (int)v[0]);
}

__device__ __forceinline__ unsigned long long bp_ballot(bool v) { return __builtin_amdgcn_ballot_w64(v); }

// v of the lane that names this one (0: none does)
__device__ __forceinline__ float bp_permute(int to, float v) { return __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(v))); }
__device__ __forceinline__ double bp_permute(int to, double v) {
    return __hiloint2double(__builtin_amdgcn_ds_permute(to, __double2hiint(v)), __builtin_amdgcn_ds_permute(to, __double2loint(v)));
}

// KI: type of a level index in LDS (8 bits when nd <= 256, whose values then lie in LDS too).
// W: wavefronts of the workgroup.
// DEPTH: blocks of variables whose entries are requested ahead of the one that is walked.
// SIMD: wavefronts per SIMD that the registers must allow.
template <class T, class KI, int W, int DEPTH, int SIMD>
__global__ __launch_bounds__(64 * W, SIMD) void k_descent_batched_pruned(
    int64_t m, int64_t n, int32_t nd, int64_t R, const T* __restrict__ X, int64_t ldx,
    const T* __restrict__ Xt, const T* __restrict__ D, const T* __restrict__ scale,
    T* __restrict__ r, int32_t* __restrict__ kidx, InstState<T>* __restrict__ st, int32_t radius,
    const uint8_t* __restrict__ var_mask, int32_t steps, int32_t iters,
    dmmv_move* __restrict__ trace, T* __restrict__ trace_t) {
    constexpr int BP_BLOCK = 64 * W, BP_WAVES = W;
    constexpr int BP_UNROLL = W <= 4 ? 8 : sizeof(T) == 4 ? 16 : 8;      // independent global loads a thread issues before it uses them
    constexpr int AP_UNROLL = W <= 4 ? 8 : 4;               //   and where it applies a move
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BpShared<T, W> F;
    T* sh_r = reinterpret_cast<T*>(smem);                  // the instance's residual
    T* sh_D = sh_r + m;                                    // the levels, and the steps from each to the next lower and the next
    T* sh_down = sh_D + (sizeof(KI) == 1 ? nd : 0);         //   higher one (where they are kept in LDS)
    T* sh_up = sh_down + (sizeof(KI) == 1 ? nd : 0);
    T* sh_jmin = sh_up + (sizeof(KI) == 1 ? nd : 0);        // per variable: bound of its next candidate
    KI* sh_k = reinterpret_cast<KI*>(sh_jmin + n);          // current level of every variable
    KI* sh_jarg = sh_k + n;                                // per variable: level of its next candidate
    // one bit per variable: it has a candidate (words of 32, after the others at a multiple of four bytes)
    uint32_t* sh_has = reinterpret_cast<uint32_t*>(smem + ((((m + n + (sizeof(KI) == 1 ? 3 * nd : 0)) * (int64_t)sizeof(T) + 2 * n * (int64_t)sizeof(KI)) + 3) & ~3ll));
    constexpr int KSH = 8 * sizeof(KI);

    const int64_t q = blockIdx.x;
    InstState<T> z = st[q];
    if (z.done || steps <= 0) return;                      // the same for the whole workgroup
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the instance's column of r and of x: strided reads, eight in flight per thread
    for (int64_t i0 = tid; i0 < m; i0 += BP_BLOCK * BP_UNROLL) {
        T a[BP_UNROLL];
#pragma unroll
        for (int u = 0; u < BP_UNROLL; ++u) {
            const int64_t i = i0 + BP_BLOCK * u;
            a[u] = r[(i < m ? i : m - 1) * R + q];
        }
#pragma unroll
        for (int u = 0; u < BP_UNROLL; ++u) {
            const int64_t i = i0 + BP_BLOCK * u;
            if (i < m) sh_r[i] = a[u];
        }
    }
    for (int64_t j0 = tid; j0 < n; j0 += BP_BLOCK * BP_UNROLL) {
        int32_t a[BP_UNROLL];
#pragma unroll
        for (int u = 0; u < BP_UNROLL; ++u) {
            const int64_t j = j0 + BP_BLOCK * u;
            a[u] = kidx[(j < n ? j : n - 1) * R + q];
        }
#pragma unroll
        for (int u = 0; u < BP_UNROLL; ++u) {
            const int64_t j = j0 + BP_BLOCK * u;
            if (j < n) sh_k[j] = (KI)a[u];
        }
    }
    const T sc = scale[q];
    const uint8_t* __restrict__ vm = var_mask ? var_mask + q * n : nullptr;
    if (sizeof(KI) == 1)
        for (int32_t k = tid; k < nd; k += BP_BLOCK) {
            sh_D[k] = D[k];
            sh_down[k] = step_of(D[k > 0 ? k - 1 : 0], D[k], sc);
            sh_up[k] = step_of(D[k < nd - 1 ? k + 1 : k], D[k], sc);
        }
    auto level = [&](int32_t k) -> T { return sizeof(KI) == 1 ? sh_D[k] : D[k]; };
    // levels a variable at level kc may take: klo(kc) .. khi(kc) without kc
    auto klo = [&](int32_t kc) -> int32_t { return radius > 0 && kc - radius > 0 ? kc - radius : 0; };
    auto khi = [&](int32_t kc) -> int32_t { return radius > 0 && kc < nd - 1 - radius ? kc + radius : nd - 1; };
    bool dirty = false;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void*)Xt, 0, (int)(uint32_t)(m * n * (int64_t)sizeof(T)), 0x00020000);
    const int32_t n32 = (int32_t)n, m32 = (int32_t)m;
    // how many of the wavefront's keys are larger
    auto rank_of = [&](uint32_t key, bool upper) -> uint32_t {
        uint32_t rank = 0;
#pragma unroll
        for (int e = 0; e < 32; ++e) rank += (uint32_t)__builtin_amdgcn_readlane((int)key, e) > key ? 1u : 0u;
        if (upper) {
#pragma unroll
            for (int e = 32; e < 64; ++e) rank += (uint32_t)__builtin_amdgcn_readlane((int)key, e) > key ? 1u : 0u;
        }
        return rank;
    };
    // Rows with |r| of at least `bound` are listed for the screening rows to be picked from.
    const bool all_rows = m32 < BP_LIST;
    T bound = (T)0;
    // (by a whole wavefront: bit u of `large` lists row i0 + u * BP_BLOCK, of |r| a(u), as the first one where that is `largest`)
    auto list_rows = [&](uint32_t large, int32_t i0, T largest, auto count, auto a) {
        constexpr int N = decltype(count)::value;
        int32_t all = 0, at = 0;
#pragma unroll
        for (int u = 0; u < N; ++u) all += __popcll(bp_ballot((large >> u) & 1u));
        if (all == 0) return;
        if (lane == 0) at = 1 + atomicAdd(&F.listed, all);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const unsigned long long rows = bp_ballot((large >> u) & 1u);
            if (rows == 0ull) continue;
            if ((large >> u) & 1u) {
                const int32_t to = at + __popcll(rows & ((1ull << lane) - 1ull));
                if (a(u) == largest) F.list[0] = i0 + u * BP_BLOCK;
                if (to < BP_LIST) F.list[to] = i0 + u * BP_BLOCK;
            }
            at += __popcll(rows);
        }
    };
    // From all rows (a thread reads its own).  The bound is the BP_WANT-th largest of 64 maxima, each over the rows that are alike
    // modulo 64: as many rows reach it, and the few that a larger one of their share hides.
    auto list_all = [&]() {
        if (!all_rows) {
            T most = (T)0;
            for (int32_t i = tid; i < m32; i += BP_BLOCK) most = dmmv_max(most, dmmv_abs(sh_r[i]));
            F.peak[tid] = (uint32_t)(bp_order(most) >> (8 * sizeof(T) - 32));
        }
        if (tid == 0) { F.listed = 0; F.list[0] = -1; }
        __syncthreads();
        if (!all_rows) {
            uint32_t key = 0;
#pragma unroll
            for (int u = 0; u < BP_WAVES; ++u) key = max(key, F.peak[lane + 64 * u]);
            key = (key & ~63u) | (uint32_t)(63 - lane);     // (no two alike)
            const unsigned long long at = bp_ballot(rank_of(key, true) == BP_WANT - 1);
            const uint32_t of = (uint32_t)__builtin_amdgcn_readlane((int)key, __builtin_ctzll(at)) & ~63u;
            bound = bp_number((decltype(bp_order(T())))of << (8 * sizeof(T) - 32));
        }
        for (int32_t i0 = w * 64; i0 < m32; i0 += BP_BLOCK) {      // whole wavefronts
            const int32_t i = i0 + lane;
            const T a = dmmv_abs(sh_r[i < m32 ? i : m32 - 1]);
            list_rows(i < m32 && (a >= bound || a == z.t) ? 1u : 0u, i, z.t, std::integral_constant<int, 1>(), [&](int) { return a; });
        }
        __syncthreads();
    };
    list_all();

    for (int32_t step = 0; step < steps; ++step) {
        // ---- 1. screening rows -----------------------------------------------------------
        // The rows of largest |r| among those listed, by their ranks: every wavefront finds them for itself.
        T tr[BP_S];
        uint32_t row_off[BP_S];
        const int32_t row0 = F.list[0];
        if (row0 < 0) {                                    // m == 0: every score is 0 = t, nothing improves
            z.done = 1;
            z.best_s = z.t;
            break;
        }
        for (bool again = false;; again = true) {
            const int32_t listed = F.listed, behind = listed < BP_LIST - 1 ? listed : BP_LIST - 1;
            const int32_t top = F.list[0], row = lane <= behind ? F.list[lane] : top;
            const T v = sh_r[row];
            // Ranks by |r| in 32 bits, the last six replaced by the lane: no two alike, and which of two rows that differ by
            // less comes first is all the same.  (The row listed first is listed again further on: left out, as the places
            // past the end.)
            uint32_t key = (__float_as_uint((float)dmmv_abs(v)) & ~63u) | (uint32_t)(63 - lane);
            if (lane > behind || (lane > 0 && row == top)) key = 0;
            if (lane == 0) key = 0xFFFFFFFFu;
            const uint32_t rank = rank_of(key, behind >= 32);
            // lane `rank` takes the row; lanes that none is for repeat the first, which changes no maximum
            const int32_t to = key != 0 ? (int32_t)rank * 4 : 63 * 4;
            const int32_t got = __builtin_amdgcn_ds_permute(to, lane < 63 || key != 0 ? row + 1 : 0);
            const T r_got = bp_permute(to, v);
            const int32_t row_by_rank = got > 0 ? got - 1 : top;
            const T r_by_rank = got > 0 ? r_got : read_lane(v, 0);
            const uint32_t off_by_rank = (uint32_t)row_by_rank * (uint32_t)n * (uint32_t)sizeof(T);
#pragma unroll
            for (int u = 0; u < BP_S; ++u) {
                row_off[u] = (uint32_t)__builtin_amdgcn_readlane((int)off_by_rank, u);
                tr[u] = read_lane(r_by_rank, u);
            }
            if (all_rows) break;
            if (!again && (listed < BP_FEWEST || listed >= BP_LIST)) {      // too few to choose from, or more than were kept
                __syncthreads();
                list_all();
                continue;
            }
            // The bound of the next iteration, whose r differs by one move: the value of rank BP_WANT (of as many of them as the
            // list holds), or further down where there are fewer.
            if (listed >= BP_WANT) {
                const int32_t guess = BP_WANT * (BP_LIST - 1) / listed, at = listed < BP_LIST ? BP_WANT - 1 : guess > 2 ? guess : 2;
                bound = dmmv_abs(read_lane(r_by_rank, at));
            } else {
                const T from = dmmv_min(bound, z.t), span = dmmv_max(z.t - from, (T)0.02 * z.t);
                const T by = (T)(BP_WANT - listed) / (T)(listed > 0 ? listed : 1);
                bound = dmmv_max(from - (T)0.5 * span * dmmv_min(by, (T)1), (T)0);
            }
            break;
        }

        // ---- 2. per variable the best candidate by (lb, k) ----------------------------------
        // Only a step that lowers the row of largest |r| can improve, which fixes the step's sign; on
        // that side lb falls from t and then rises (lb is quasi-convex in k, as computed: D ascends and
        // rounding is monotone), so the levels are walked outwards until it rises - one or two
        // steps for most variables instead of all |D| levels, and none of the walk's results is missed:
        // what lies on the other side or beyond the rise is no better than t or than the best found.
        // The first step is taken for all 64 variables of a block, its size from a table; most blocks then have a
        // few variables left, and these walk on in place, 64 lanes or one.
        const T r_max = tr[0], t_now = dmmv_abs(r_max);
        for (int64_t i = tid; i < 2 * ((n + 63) / 64); i += BP_BLOCK) sh_has[i] = 0;
        if (tid == 0) F.bound = bp_order(t_now);
        __syncthreads();
        if (tid == 0) { F.listed = 0; F.list[0] = -1; }     // (every wavefront has its rows; a barrier follows before the next are listed)
        // the step to the next level up or down, 0 at the ends of D
        auto first_step = [&](int32_t kc, bool up) -> T {
            if (sizeof(KI) == 1) return sh_down[up ? nd + kc : kc];
            const int32_t k = up ? (kc < nd - 1 ? kc + 1 : kc) : (kc > 0 ? kc - 1 : 0);
            return step_of(level(k), level(kc), sc);
        };
        T ahead[DEPTH + 1][BP_S];
        int32_t ahead_k[DEPTH + 1];
        const int32_t first = w * 64;
        auto fetch = [&](int32_t j0, int to) {
            const int32_t jc = j0 + lane < n32 ? j0 + lane : n32 - 1;
            const uint32_t at = (uint32_t)jc * (uint32_t)sizeof(T);
            ahead_k[to] = sh_k[jc];
#pragma unroll
            for (int u = 0; u < BP_S; ++u) ahead[to][u] = bp_entry(rs_x, at, row_off[u], (T)0);
        };
        auto screen = [&](int32_t j0, const T* xs, int32_t kc) {
            const int32_t j = j0 + lane;
            auto bound_of = [&](T delta) -> T { return bp_max<T>([&](int u) { return dmmv_fma(delta, xs[u], tr[u]); }); };
            const bool up = (xs[0] < (T)0) == (r_max > (T)0);
            T delta = first_step(kc, up);
            T lb = bound_of(delta);
            bool walk = !(lb > t_now) && xs[0] != (T)0 && j < n32;      // (an entry 0 in that row lowers nothing)
            if (bp_ballot(walk) == 0ull) return;
            if (vm) walk = walk && vm[j < n32 ? j : n32 - 1] != 0;
            const int32_t end = up ? khi(kc) : klo(kc), dir = up ? 1 : -1;
            walk = walk && kc != end;
            const T dcur = level(kc);
            T prev = Limits<T>::inf();
            int32_t k = kc, jk = kc;
            while (bp_ballot(walk) != 0ull) {
                if (walk) {                                 // a step on: its bound is no larger than the one before
                    k += dir;
                    jk = lb < prev || !up ? k : jk;         // equal bounds: the lowest level stays
                    prev = lb;
                }
                walk = walk && k != end;
                if (bp_ballot(walk) == 0ull) break;
                delta = step_of(level(walk ? k + dir : k), dcur, sc);
                lb = bound_of(delta);
                walk = walk && !(lb > prev);
            }
            const bool found = jk != kc;
            const unsigned long long has = bp_ballot(found);
            if (found) {
                sh_jmin[j] = prev;
                sh_jarg[j] = (KI)jk;
            }
            if (lane < 2) sh_has[(j0 >> 5) + lane] = (uint32_t)(lane == 0 ? has : has >> 32);
        };
        // (requested unasked, the last variable's where there are no more: with the request under a condition the compiler waits
        // for all that is in flight before the first of them is used)
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) fetch(first + u * BP_BLOCK, u);
        for (int32_t j0 = first; j0 < n32; j0 += (DEPTH + 1) * BP_BLOCK) {      // whole wavefronts
#pragma unroll
            for (int u = 0; u <= DEPTH; ++u) {
                const int32_t ju = j0 + u * BP_BLOCK;
                fetch(ju + DEPTH * BP_BLOCK, (u + DEPTH) % (DEPTH + 1));
                if (u == 0 || ju < n32) screen(ju, ahead[u], ahead_k[u]);
            }
        }

        // ---- 3. candidates in ascending (lb, c) until none can beat the best score ---------
        // Every wavefront walks the candidates of ITS variables (those its threads screened) in
        // ascending (lb, c) and scores them one after the other, without waiting for the others.  It stops at a candidate that
        // loses to its own best (score, c), or whose lb is above the smallest score found by any wavefront: only above,
        // as that score comes without its c, and a candidate of the same score may have a smaller one.  For the same reason a
        // score equal to the shared one is kept, and the arg-min over F.found decides by c.  Then every candidate not scored
        // has score >= lb, which is above the best score, or the same with a larger c.
        // A lane keeps the best of the variables it looks after (16 at a time of the wavefront's blocks), and looks
        // them through again only when one of them has been scored.
        const int32_t groups = 4 * ((n32 - first + BP_BLOCK - 1) / BP_BLOCK);      // of 16, of this wavefront
        T mine_s;
        int32_t mine_c;
        auto look_through = [&]() {
            mine_s = Limits<T>::inf();
            mine_c = -1;
            for (int32_t g = lane; g < groups; g += 64) {
                const int32_t j0 = first + (g >> 2) * BP_BLOCK + (g & 3) * 16;
                uint32_t has = (sh_has[j0 >> 5] >> (j0 & 16)) & 0xFFFFu;
                while (has) {
                    const int32_t j = j0 + __builtin_ctz(has);
                    has &= has - 1;
                    const T v = sh_jmin[j];
                    if (v < mine_s) { mine_s = v; mine_c = (int32_t)(j << KSH) | (int32_t)sh_jarg[j]; }   // ties: the lowest j
                }
            }
        };
        __builtin_amdgcn_wave_barrier();
        look_through();                                    // (of what this wavefront has written itself)
        T best_s = z.t;                                    // only scores below t count
        int32_t best_c = -1;
        auto shared_bound = [&]() -> T { return bp_number(__hip_atomic_load(&F.bound, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)); };
        for (;;) {
            T s = mine_s;
            int32_t c = mine_c;
            bp_argmin(s, c);
            // (a bound equal to the best score another wavefront has found may still win by its number)
            if (!bp_better(s, c, best_s, best_c) || s > shared_bound()) break;      // the same for the whole wavefront
            const int32_t j = c >> KSH, k = c & ((1 << KSH) - 1);
            const T* __restrict__ col = X + ldx * j;
            // its score over all rows, BP_UNROLL loads in flight; a row past the end repeats row m - 1, which changes
            // no maximum
            T a[BP_UNROLL], xs[BP_S];
#pragma unroll
            for (int u = 0; u < BP_UNROLL; ++u) a[u] = col[lane + 64 * u < m32 ? lane + 64 * u : m32 - 1];
            // (the entries of the variable's next candidate's bounds go out with them)
#pragma unroll
            for (int u = 0; u < BP_S; ++u) xs[u] = bp_entry(rs_x, (uint32_t)j * (uint32_t)sizeof(T), row_off[u], (T)0);
            const int32_t kc = sh_k[j];
            const T dcur = level(kc);
            const T delta = step_of(level(k), dcur, sc);
            T acc = (T)0, least;
            for (int32_t i0 = lane;;) {
#pragma unroll
                for (int u = 0; u < BP_UNROLL; ++u) {
                    const int32_t i = i0 + 64 * u;
                    acc = dmmv_max(acc, dmmv_abs(dmmv_fma(delta, a[u], sh_r[i < m32 ? i : m32 - 1])));
                }
                i0 += 64 * BP_UNROLL;
                least = shared_bound();
                if (i0 - lane >= m32 || bp_ballot(acc > least) != 0ull) break;        // it has lost already: the rest cannot matter
#pragma unroll
                for (int u = 0; u < BP_UNROLL; ++u) {
                    const int32_t i = i0 + 64 * u;
                    a[u] = col[i < m32 ? i : m32 - 1];
                }
            }
            const T sfull = wave_max(acc);
            if (!(sfull > least) && bp_better(sfull, c, best_s, best_c)) { best_s = sfull; best_c = c; }
            if (sfull < least) {
                if (lane == 0) atomicMin(&F.bound, bp_order(sfull));
                least = sfull;
            }
            // what is left of this wavefront's comes behind (s, c)
            if (s > least) break;
            // this variable's next candidate: the smallest (lb, k) after (s, k); lanes take the levels
            T bl = Limits<T>::inf();
            int32_t bk = -1;
            const int32_t kend = khi(kc);
            for (int32_t k0 = klo(kc); k0 <= kend; k0 += 64) {
                const int32_t kk = k0 + lane;
                const bool ok = kk <= kend && kk != kc;
                const T dl = ok ? step_of(level(kk), dcur, sc) : (T)0;
                const T lb = bp_max<T>([&](int u) { return dmmv_fma(dl, xs[u], tr[u]); });
                const bool after = ok && (lb > s || (lb == s && kk > k));
                if (after && lb < bl) { bl = lb; bk = kk; }       // kk ascends per lane: ties keep the lowest
            }
            bp_argmin(bl, bk);
            if (lane == (int)((((j / BP_BLOCK) << 2) | ((j >> 4) & 3)) & 63)) {      // the lane that looks after it
                if (bk >= 0) { sh_jmin[j] = bl; sh_jarg[j] = (KI)bk; }
                else sh_has[j >> 5] &= ~(1u << (j & 31));
                look_through();
            }
        }
        if (lane == 0) {
            BpFound<T> f;
            f.s = best_s; f.c = best_c;
            F.found[w] = f;
        }
        __syncthreads();
        {
            const BpFound<T> f = F.found[lane & (BP_WAVES - 1)];
            best_s = f.s;
            best_c = f.c;
            bp_argmin(best_s, best_c);                     // -1: nothing below t
            best_c = best_s < t_now ? best_c : -1;
            if (best_c < 0) best_s = t_now;
        }

        // ---- 4. decide and apply ---------------------------------------------------------
        z.best_s = best_s;
        if (best_c < 0) { z.done = 1; break; }
        {
            const int64_t j = best_c >> KSH;
            const int32_t k = best_c & ((1 << KSH) - 1);
            const T delta = step_of(level(k), level(sh_k[j]), sc);
            const T* __restrict__ col = X + ldx * j;
            for (int32_t i0 = w * 64; i0 < m32; i0 += BP_BLOCK * AP_UNROLL) {      // whole wavefronts
                T a[AP_UNROLL];
                uint32_t large = 0;                        // which of these rows are listed
#pragma unroll
                for (int u = 0; u < AP_UNROLL; ++u) {
                    const int32_t i = i0 + lane + BP_BLOCK * u;
                    a[u] = col[i < m32 ? i : m32 - 1];
                }
#pragma unroll
                for (int u = 0; u < AP_UNROLL; ++u) {
                    const int32_t i = i0 + lane + BP_BLOCK * u;
                    if (i < m32) {
                        a[u] = dmmv_fma(delta, a[u], sh_r[i]);
                        sh_r[i] = a[u];
                        large |= (dmmv_abs(a[u]) >= bound || dmmv_abs(a[u]) == best_s ? 1u : 0u) << u;
                    }
                }
                // (the applied move's score is the new max |r|, bit for bit)
                list_rows(large, i0 + lane, best_s, std::integral_constant<int, AP_UNROLL>(), [&](int u) { return dmmv_abs(a[u]); });
            }
            __syncthreads();                               // everyone has read sh_k[j]
            if (tid == 0) {
                sh_k[j] = (KI)k;
                kidx[j * R + q] = k;
                if (z.moves < iters) {
                    const int64_t slot = q * (int64_t)iters + z.moves;
                    if (trace) { trace[slot].j = (int32_t)j; trace[slot].k = k; }
                    if (trace_t) trace_t[slot] = best_s;
                }
            }
            z.t = best_s;
            z.moves += 1;
            dirty = true;                                  // (sh_k is read again behind the next iteration's first barrier)
        }
    }

    if (dirty)
        for (int64_t i = tid; i < m; i += BP_BLOCK) r[i * R + q] = sh_r[i];
    if (tid == 0) {
        z.apply_j = -1;
        z.apply_k = -1;
        z.delta = (T)0;
        st[q] = z;
    }
}

static size_t bp_lds_bytes(int64_t m, int64_t n, int32_t nd, size_t esz) {
    return (size_t)(m + n) * esz + (size_t)n * 2 * (nd <= 256 ? 1 : 2);
}
// the variables' bits and the levels, on top of these
static size_t bp_lds_more(int64_t n, int32_t nd, size_t esz) { return 4 + (size_t)ceil_div(n, 64) * 8 + (nd <= BP_DCAP ? 3 * (size_t)nd * esz : 0); }
constexpr size_t BP_LDS_MOST = BP_LDS_LIMIT + 4096 + 3 * BP_DCAP * 8;

template <class T>
dmmv_status descent_t(Ctx* c, int32_t steps, int32_t iters, dmmv_move* trace, void* trace_t) {
    const int64_t m = c->p.m, n = c->p.n, R = c->p.R;
    const size_t lds = bp_lds_bytes(m, n, c->p.nd, sizeof(T)) + bp_lds_more(n, c->p.nd, sizeof(T));
    auto launch = [&](auto kernel, int waves) -> dmmv_status {
        DMMV_TRY(ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), (int)BP_LDS_MOST));
        hipLaunchKernelGGL(kernel, dim3((unsigned)R), dim3(64 * waves), lds, c->stream, m, n, c->p.nd, R,
                           (const T*)c->p.A_dense, c->p.lda, (const T*)c->Xt, (const T*)c->D_dev,
                           (const T*)c->scale_dev, (T*)c->r, c->kidx, (InstState<T>*)c->state, c->o.radius,
                           c->o.var_mask, steps, iters, trace, (T*)trace_t);
        DMMV_LAUNCH_CHECK();
        return DMMV_OK;
    };
    constexpr int64_t CU_LDS = 160 * 1024, CUS = 256;
    const int64_t by_lds = CU_LDS / (int64_t)(lds + sizeof(BpShared<T, 4>)), by_number = ceil_div(R, CUS);
    const int64_t on_cu = by_lds < by_number ? by_lds : by_number;         // instances that a compute unit holds at a time
    // Eight wavefronts an instance where these are no more than two (an instance's iteration is a chain of latencies then), four
    // beyond, for instances that do not fill more, and where it is LDS alone that keeps others away and the screening (n) is what takes
    // longest.  us of whole calls to the local optima, four and eight (always four, by another choice of screening rows, in brackets):
    // 20 of 2048 x 4096 1931 and 1413 (2445), 250 2088 and 1657 (3280), 500 2300 and 1947 (3377), 600 2384 and 2346 (3423), 1000 2838 and
    // 3308 (3654); 20 of 2048 x 768 608 and 517 (921); 400 of 300 x 300 359 and 344 (423); 100 of 9000 x 100 984 and 690 (1741), 500 of
    // 600 x 100 358 and 339 (411), one of 8000 x 30 in fp64 2344 and 1815 (2145); 1000 of 16 000 x 2000 6794 and 5790 (9492); but 400 of
    // 300 x 200 309 and 303 (379), 60 000 of 8 x 8 525 and 1462 (533; the kernel alone), 1000 of 4000 x 4000 in fp64 12 599 and 12 714.
    const bool eight = (by_number <= 2 || (by_lds <= 2 && m > n)) && (n > 256 || m > 512);
    // Of four, one block of variables is requested ahead where no more than five share a compute unit anyway, and where there are many
    // blocks; else the registers that it takes cost more.  us without and with (in brackets with registers for six): 4096 of 2048 x 4096
    // 9029 and 8718 (8805), 1000 of 1024 x 2048 1466 and 1400 (1437), 600 of 2048 x 100 472 and 445 (464), 2000 of 1024 x 2048 2209 and 2170
    // (2141), 4000 3398 and 3451 (3329); but 2000 of 300 x 1000 1191 and 1263 (1222), 10 000 of 300 x 300 1420 and 1611 (1513).  Of eight
    // none: with none, one and two blocks ahead 20 of 2048 x 768 517, 534, 547; 500 of 2048 x 4096 1947, 1960, 2075 (20 of them 1413, 1399,
    // 1459); in fp64 500 of 2048 x 4000 4623, 4641, 5447.
    constexpr int MORE = sizeof(T) == 4 ? 6 : 4;
    auto with = [&](auto ki) -> dmmv_status {
        typedef decltype(ki) KI;
        if (eight) return launch(k_descent_batched_pruned<T, KI, 8, 0, 2>, 8);
        if (on_cu <= 5) return launch(k_descent_batched_pruned<T, KI, 4, 1, 4>, 4);
        return n > 1024 ? launch(k_descent_batched_pruned<T, KI, 4, 1, MORE>, 4) : launch(k_descent_batched_pruned<T, KI, 4, 0, MORE>, 4);
    };
    return c->p.nd > BP_DCAP ? with(uint16_t()) : with(uint8_t());
}

}  // namespace

static bool bp_fits(int64_t m, int64_t n, int32_t nd, int64_t R, size_t esz) {
    return n > 0 && R <= INT32_MAX && m <= BP_MAX_ROWS && bp_lds_bytes(m, n, nd, esz) <= BP_LDS_LIMIT;
}

bool batched_pruned_asked(const dmmv_problem& p, const dmmv_options& o) {
    return !p.csr_rowptr && (p.R > 1 || p.scale) && o.prune && !o.keep_going && o.l2_rule != 1 && o.l2_rule != 2 &&
           bp_fits(p.m, p.n, p.nd, p.R, p.dtype == DMMV_F64 ? 8 : 4);
}

bool batched_pruned_applicable(const Ctx* c) {
    // a batch, or a dense single instance (a batch of one: r [m][1], x [n][1], scale 1, with the
    // row-major copy of A that dmmv_create makes for options.prune)
    // - only a small one: one workgroup scores it, so a table of more than 2^24 pairs, or more than
    // 64 levels per variable (a thread walks the levels of its variable), is left to the chip-wide
    // full evaluation
    const bool small_dense = c->kind == KIND_DENSE && c->Xt != nullptr && c->p.nd <= 64 &&
                             c->p.m * c->p.n * (int64_t)c->p.nd <= ((int64_t)1 << 24);
    const bool kind_ok = c->kind == KIND_BATCHED || small_dense;
    if (!kind_ok || !c->o.prune || c->o.keep_going || c->cmp_on) return false;
    if (c->o.l2_rule == 1 || c->o.l2_rule == 2) return false;      // a bound on the score alone does not order (score, l2 change)
    return bp_fits(c->p.m, c->p.n, c->p.nd, c->p.R, c->esz);
}

dmmv_status batched_descent_pruned(Ctx* c, int32_t steps, int32_t iters, dmmv_move* trace, void* trace_t) {
    if (!batched_pruned_applicable(c)) return fail(DMMV_ERR_STATE, "pruned batched descent: not applicable to this handle");
    if (steps <= 0) return DMMV_OK;
    return c->p.dtype == DMMV_F64 ? descent_t<double>(c, steps, iters, trace, trace_t)
                                  : descent_t<float>(c, steps, iters, trace, trace_t);
}

}  // namespace dmmv
