// Batched instances: the descent with exact pruning (options.prune), one workgroup per instance.
//
// The score of a move (j, k) is a maximum over all m rows, so the maximum over ANY subset of the
// rows is a lower bound of it, and a move can only win if its lower bound is below the score of
// the best move known (Corollary 1 turns the same observation into a filter for swaps: a move
// that does not fix the rows of largest |r| cannot improve).  Per iteration the workgroup
//   1. picks S = 16 screening rows: of each lane's rows the one of largest |r|, and of these the four largest of each
//      wavefront (the row of largest |r| overall is always one of them; the wavefronts share the rows evenly);
//   2. bounds candidates from below by lb(j, k) = max_{i in S} |fma(delta, X_ij, r_i)| - 16 rows instead
//      of m - and keeps per variable its best candidate by (lb, k), found by walking outwards from
//      the current level on the side that lowers the row of largest |r| until lb rises;
//   3. takes candidates in ascending order of (lb, c), c = j nd + k - each wavefront among the
//      variables it screened, one per round - scores each one over all m rows (the same fma on
//      the same operands as the full evaluation, so the same bits), and stops when no wavefront's
//      next candidate has (lb, c) below the best (score, c) found: every candidate not scored
//      then has score >= lb >= that best score, and loses the tie on c;
//   4. applies the move if its score is below t.
// The result is the arg-min of the full table restricted to strictly improving moves, i.e. the
// move the full evaluation + selection would apply - found with a few full scores instead of
// n (nd - 1); a candidate's score is given up as soon as a row puts it above the best one.
// On 2048 x 4096 with 16 levels an iteration spends 42 % of its time on step 2 (256 KiB of X each, most of it past the
// L2), 47 % on step 3 (eleven scores in five and a half rounds of dependent loads) and 6 % on step 1.  The 4096
// instances of that layer take 10.1 ms to their local optima, the residual's 0.5 ms included; 23.7 with all levels of every
// variable screened and every score finished, and 14.5 before the first step came from a table and a buffer load, the
// screening rows from one pass over r, and a lane kept the best of its variables instead of looking through them all in
// every round.  Tried: the first step on eight rows and the survivors queued for the other eight, 64 at a time (a line of X
// fetched per row and variable: 11.7 ms); a good move looked for first, to bound the others (12.2); eight more rows for the
// variables that are left (4.8 rounds, but 10.6).
// The instance's r (m values) and x (n level indices) live in LDS for the whole
// launch, so a launch can run any number of iterations without touching the other instances;
// an instance stops by itself at a local optimum.
#include <type_traits>

#include "dmmv_common.h"

namespace dmmv {

namespace {

constexpr int BP_BLOCK = 256;
constexpr int BP_WAVES = BP_BLOCK / 64;
constexpr int BP_TOPW = 4;                       // screening rows a wavefront contributes
constexpr int BP_S = BP_WAVES * BP_TOPW;         // screening rows
constexpr int64_t BP_MAX_ROWS = 16384;
constexpr int BP_DCAP = 256;                     // levels kept in LDS
constexpr size_t BP_LDS_LIMIT = 96 * 1024;       // dynamic LDS a workgroup may ask for
constexpr int BP_UNROLL = 8;                     // independent global loads a thread issues before it uses them

template <class T>
struct BpShared {
    T D[BP_DCAP];
    T step[2][BP_DCAP];                          // from a level to the next lower and the next higher one
    T top_r[BP_S];
    int32_t top_row[BP_S];
    T round_s[2][BP_WAVES];                      // score and candidate each wavefront scored in a round
    int32_t round_c[2][BP_WAVES];                //   (-1: it had none left that could win)
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

// KI: type of a level index in LDS (8 bits when nd <= 256, whose values then lie in LDS too).
// AHEAD: the next block of variables' entries are requested before this one is walked.  With a single block (n <= 256) there
// is none, and the registers it takes cost a wavefront per SIMD: 60 000 instances of 8 x 8, 30 moves, 1193 us with it
// and 1043 without (fp64 1927 and 1527).
// The wavefronts per SIMD asked for are what the kernel had before it kept a step table: one to nine registers more had cost one of
// them (60 000 instances of 8 x 8 in fp64 1525 us, then 1558, 1237 with it back; 2000 of 64 x 64 1854, 2250, 1971).  Not so in fp32
// with AHEAD, where the fifth wavefront is worth less than the register it spills (4096 of 2048 x 4096: 0.5 %).
// FEW: an instance has fewer rows than the workgroup threads.
template <class T, class KI, bool AHEAD, bool FEW>
__global__ __launch_bounds__(BP_BLOCK, sizeof(T) == 4 ? (AHEAD ? 1 : 6) : (AHEAD ? 3 : 4)) void k_descent_batched_pruned(
    int64_t m, int64_t n, int32_t nd, int64_t R, const T* __restrict__ X, int64_t ldx,
    const T* __restrict__ Xt, const T* __restrict__ D, const T* __restrict__ scale,
    T* __restrict__ r, int32_t* __restrict__ kidx, InstState<T>* __restrict__ st, int32_t radius,
    const uint8_t* __restrict__ var_mask, int32_t steps, int32_t iters,
    dmmv_move* __restrict__ trace, T* __restrict__ trace_t) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BpShared<T> F;
    T* sh_r = reinterpret_cast<T*>(smem);                  // the instance's residual
    T* sh_jmin = sh_r + m;                                 // per variable: bound of its next candidate
    KI* sh_k = reinterpret_cast<KI*>(sh_jmin + n);          // current level of every variable
    KI* sh_jarg = sh_k + n;                                // per variable: level of its next candidate
    // one bit per variable: it has a candidate (words of 32, after the others at a multiple of four bytes)
    uint32_t* sh_has = reinterpret_cast<uint32_t*>(smem + (((m + n) * (int64_t)sizeof(T) + 2 * n * (int64_t)sizeof(KI) + 3) & ~3ll));
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
            F.D[k] = D[k];
            F.step[0][k] = step_of(D[k > 0 ? k - 1 : 0], D[k], sc);
            F.step[1][k] = step_of(D[k < nd - 1 ? k + 1 : k], D[k], sc);
        }
    auto level = [&](int32_t k) -> T { return sizeof(KI) == 1 ? F.D[k] : D[k]; };
    // levels a variable at level kc may take: klo(kc) .. khi(kc) without kc
    auto klo = [&](int32_t kc) -> int32_t { return radius > 0 && kc - radius > 0 ? kc - radius : 0; };
    auto khi = [&](int32_t kc) -> int32_t { return radius > 0 && kc < nd - 1 - radius ? kc + radius : nd - 1; };
    bool dirty = false;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void*)Xt, 0, (int)(uint32_t)(m * n * (int64_t)sizeof(T)), 0x00020000);
    const int32_t n32 = (int32_t)n, m32 = (int32_t)m;
    // A lane's rows: every 256th.  FEW of them are split into a quarter for each wavefront, or the first ones would hold them
    // all and the others propose no screening rows: 2000 instances of 64 x 64, 16 levels, 1542 us with four rows, 168 with sixteen.
    const int32_t quarter = (m32 + BP_WAVES - 1) / BP_WAVES;
    const int32_t first_row = !FEW ? tid : lane < quarter ? w * quarter + lane : m32;
    __syncthreads();

    for (int32_t step = 0; step < steps; ++step) {
        // ---- 1. screening rows -----------------------------------------------------------
        {
            // (the largest of every lane's rows, and of these the largest four: a lane's second row is not looked for,
            // which leaves the largest of all and rarely misses one of the others)
            T bv = (T)-1;
            int32_t bi = -1;
            for (int32_t i = first_row; i < m32; i += BP_BLOCK) {
                const T a = dmmv_abs(sh_r[i]);
                if (a > bv) { bv = a; bi = i; }
            }
            for (int round = 0; round < BP_TOPW; ++round) {
                T s = -bv;                                  // largest |r| = smallest -|r|; ties: lowest row
                int32_t c = bi;
                bp_argmin(s, c);
                if (lane == 0) {                            // the largest of every share first, then the second, ..
                    F.top_row[round * BP_WAVES + w] = c;
                    F.top_r[round * BP_WAVES + w] = c >= 0 ? sh_r[c] : (T)0;
                }
                if (bi == c) bi = -1;
            }
        }
        __syncthreads();
        // The row of largest |r| of all goes to entry 0 (row 0 belongs to wavefront 0, so there is one whenever m > 0); a
        // share with fewer rows than BP_TOPW repeats it, which changes no maximum.
        int32_t um = 0;
#pragma unroll
        for (int x = 1; x < BP_WAVES; ++x) if (F.top_row[x] >= 0 && dmmv_abs(F.top_r[x]) > dmmv_abs(F.top_r[um])) um = x;
        const int32_t row0 = F.top_row[um], row_x = F.top_row[tid & (BP_S - 1)];
        const T r0 = F.top_r[um], r_x = F.top_r[tid & (BP_S - 1)];
        const int32_t row_0 = F.top_row[0];
        const T r_0 = F.top_r[0];
        __syncthreads();
        if (tid < BP_S) {
            const bool first = tid == 0, swapped = tid == um && um != 0;
            const int32_t row = first ? row0 : swapped ? row_0 : row_x;
            F.top_row[tid] = row < 0 ? row0 : row;
            F.top_r[tid] = first || row < 0 ? r0 : swapped ? r_0 : r_x;
        }
        __syncthreads();
        if (row0 < 0) {                                    // m == 0: every score is 0 = t, nothing improves
            z.done = 1;
            z.best_s = z.t;
            break;
        }
        T tr[BP_S];
        uint32_t row_off[BP_S];
#pragma unroll
        for (int u = 0; u < BP_S; ++u) {
            tr[u] = F.top_r[u];
            row_off[u] = (uint32_t)__builtin_amdgcn_readfirstlane(F.top_row[u]) * (uint32_t)n * (uint32_t)sizeof(T);
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
        __syncthreads();
        // the step to the next level up or down, 0 at the ends of D
        auto first_step = [&](int32_t kc, bool up) -> T {
            if (sizeof(KI) == 1) return F.step[up ? 1 : 0][kc];
            const int32_t k = up ? (kc < nd - 1 ? kc + 1 : kc) : (kc > 0 ? kc - 1 : 0);
            return step_of(level(k), level(kc), sc);
        };
        T nx[BP_S];
        auto fetch = [&](int32_t j0) {
            const uint32_t at = (uint32_t)(j0 + lane < n32 ? j0 + lane : n32 - 1) * (uint32_t)sizeof(T);
#pragma unroll
            for (int u = 0; u < BP_S; ++u) nx[u] = bp_entry(rs_x, at, row_off[u], (T)0);
        };
        const int32_t first = tid - lane;
        if (AHEAD && first < n32) fetch(first);
        for (int32_t j0 = first; j0 < n32; j0 += BP_BLOCK) {        // whole wavefronts
            const int32_t j = j0 + lane;
            const int32_t jc = j < n32 ? j : n32 - 1;
            const int32_t kc = sh_k[jc];
            if (!AHEAD) fetch(j0);
            T xs[BP_S];
#pragma unroll
            for (int u = 0; u < BP_S; ++u) xs[u] = nx[u];
            if (AHEAD && j0 + BP_BLOCK < n32) fetch(j0 + BP_BLOCK);
            auto bound_of = [&](T delta) -> T {
                T lb = (T)0;
#pragma unroll
                for (int u = 0; u < BP_S; ++u) lb = dmmv_max(lb, dmmv_abs(dmmv_fma(delta, xs[u], tr[u])));
                return lb;
            };
            const bool up = (xs[0] < (T)0) == (r_max > (T)0);
            T delta = first_step(kc, up);
            T lb = bound_of(delta);
            bool walk = !(lb > t_now) && xs[0] != (T)0 && j < n32;      // (an entry 0 in that row lowers nothing)
            if (__ballot(walk) == 0ull) continue;
            if (vm) walk = walk && vm[jc] != 0;
            T prev = t_now, jbest = Limits<T>::inf();
            const int32_t end = up ? khi(kc) : klo(kc), dir = up ? 1 : -1;
            walk = walk && kc != end;
            const T dcur = level(kc);
            int32_t k = kc, jk = 0;
            while (__ballot(walk) != 0ull) {
                if (walk) {
                    k += dir;
                    if (lb < jbest || !up) { jbest = lb; jk = k; }     // equal bounds: the lowest level stays
                    prev = lb;
                }
                walk = walk && k != end;
                if (__ballot(walk) == 0ull) break;
                delta = step_of(level(walk ? k + dir : k), dcur, sc);
                lb = bound_of(delta);
                walk = walk && !(lb > prev);
            }
            const bool found = jbest < Limits<T>::inf();
            const unsigned long long has = __ballot(found);
            if (found) {
                sh_jmin[j] = jbest;
                sh_jarg[j] = (KI)jk;
            }
            if (lane < 2) sh_has[(j0 >> 5) + lane] = (uint32_t)(lane == 0 ? has : has >> 32);
        }

        // ---- 3. candidates in ascending (lb, c) until none can beat the best score ---------
        // Every wavefront walks the candidates of ITS variables (those its threads screened) in
        // ascending (lb, c) and scores one per round, as long as that candidate can still beat the
        // best (score, c) the workgroup knew when the round began; the rounds end when no
        // wavefront had such a candidate.  Then every candidate not scored has
        // (lb, c) >= (best score, its c), hence score >= lb >= best score, and loses the tie on c.
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
        for (int parity = 0;; parity ^= 1) {
            T s = mine_s;
            int32_t c = mine_c;
            bp_argmin(s, c);
            const bool live = bp_better(s, c, best_s, best_c);   // the same for the whole wavefront
            T sfull = (T)0;
            if (live) {
                const int32_t j = c >> KSH, k = c & ((1 << KSH) - 1);
                const int32_t kc = sh_k[j];
                const T dcur = level(kc);
                const T delta = step_of(level(k), dcur, sc);
                // (the entries of its next candidate's bounds go out with the first of the column's)
                T xs[BP_S];
#pragma unroll
                for (int u = 0; u < BP_S; ++u) xs[u] = bp_entry(rs_x, (uint32_t)j * (uint32_t)sizeof(T), row_off[u], (T)0);
                // its score over all rows, eight loads in flight; a row past the end repeats row m - 1, which changes
                // no maximum
                const T* __restrict__ col = X + ldx * j;
                T acc = (T)0;
                for (int32_t i0 = lane; i0 < m32; i0 += 64 * BP_UNROLL) {
                    T a[BP_UNROLL];
#pragma unroll
                    for (int u = 0; u < BP_UNROLL; ++u) {
                        const int32_t i = i0 + 64 * u;
                        a[u] = col[i < m32 ? i : m32 - 1];
                    }
#pragma unroll
                    for (int u = 0; u < BP_UNROLL; ++u) {
                        const int32_t i = i0 + 64 * u;
                        acc = dmmv_max(acc, dmmv_abs(dmmv_fma(delta, a[u], sh_r[i < m32 ? i : m32 - 1])));
                    }
                    if (__ballot(acc > best_s) != 0ull) break;        // it has lost already: the rest cannot matter
                }
                // this variable's next candidate: the smallest (lb, k) after (s, k); lanes take the levels
                T bl = Limits<T>::inf();
                int32_t bk = -1;
                const int32_t kend = khi(kc);
                for (int32_t k0 = klo(kc); k0 <= kend; k0 += 64) {
                    const int32_t kk = k0 + lane;
                    const bool ok = kk <= kend && kk != kc;
                    const T dl = ok ? step_of(level(kk), dcur, sc) : (T)0;
                    T lb = (T)0;
#pragma unroll
                    for (int u = 0; u < BP_S; ++u) lb = dmmv_max(lb, dmmv_abs(dmmv_fma(dl, xs[u], tr[u])));
                    const bool after = ok && (lb > s || (lb == s && kk > k));
                    if (after && lb < bl) { bl = lb; bk = kk; }       // kk ascends per lane: ties keep the lowest
                }
                bp_argmin(bl, bk);
                if (lane == (int)((((j >> 8) << 2) | ((j >> 4) & 3)) & 63)) {      // the lane that looks after it
                    if (bk >= 0) { sh_jmin[j] = bl; sh_jarg[j] = (KI)bk; }
                    else sh_has[j >> 5] &= ~(1u << (j & 31));
                    look_through();
                }
                sfull = wave_max(acc);
            }
            if (lane == 0) { F.round_s[parity][w] = sfull; F.round_c[parity][w] = live ? c : -1; }
            __syncthreads();
            bool any = false;
#pragma unroll
            for (int u = 0; u < BP_WAVES; ++u) {
                const T us = F.round_s[parity][u];
                const int32_t uc = F.round_c[parity][u];
                any = any || uc >= 0;
                if (bp_better(us, uc, best_s, best_c)) { best_s = us; best_c = uc; }
            }
            if (!any) break;                               // the same for the whole workgroup
            // the other pair of slots is written next: a wavefront gets there only after every
            // wavefront has passed this round's barrier, i.e. has read the slots of the round before
        }

        // ---- 4. decide and apply ---------------------------------------------------------
        z.best_s = best_s;
        if (best_c < 0) { z.done = 1; break; }
        {
            const int64_t j = best_c >> KSH;
            const int32_t k = best_c & ((1 << KSH) - 1);
            const T delta = step_of(level(k), level(sh_k[j]), sc);
            const T* __restrict__ col = X + ldx * j;
            for (int64_t i0 = tid; i0 < m; i0 += BP_BLOCK * BP_UNROLL) {
                T a[BP_UNROLL];
#pragma unroll
                for (int u = 0; u < BP_UNROLL; ++u) {
                    const int64_t i = i0 + BP_BLOCK * u;
                    a[u] = col[i < m ? i : m - 1];
                }
#pragma unroll
                for (int u = 0; u < BP_UNROLL; ++u) {
                    const int64_t i = i0 + BP_BLOCK * u;
                    if (i < m) sh_r[i] = dmmv_fma(delta, a[u], sh_r[i]);
                }
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
            z.t = best_s;                                  // the applied move's score is the new max |r|, bit for bit
            z.moves += 1;
            dirty = true;
            __syncthreads();
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
static size_t bp_lds_bits(int64_t n) { return 4 + (size_t)ceil_div(n, 64) * 8; }      // the variables' bits, on top of these
constexpr size_t BP_LDS_MOST = BP_LDS_LIMIT + 4096;

template <class T>
dmmv_status descent_t(Ctx* c, int32_t steps, int32_t iters, dmmv_move* trace, void* trace_t) {
    const int64_t m = c->p.m, n = c->p.n, R = c->p.R;
    const size_t lds = bp_lds_bytes(m, n, c->p.nd, sizeof(T)) + bp_lds_bits(n);
    auto launch = [&](auto kernel) -> dmmv_status {
        DMMV_TRY(ensure_dynamic_lds(reinterpret_cast<const void*>(kernel), (int)BP_LDS_MOST));
        hipLaunchKernelGGL(kernel, dim3((unsigned)R), dim3(BP_BLOCK), lds, c->stream, m, n, c->p.nd, R,
                           (const T*)c->p.A_dense, c->p.lda, (const T*)c->Xt, (const T*)c->D_dev,
                           (const T*)c->scale_dev, (T*)c->r, c->kidx, (InstState<T>*)c->state, c->o.radius,
                           c->o.var_mask, steps, iters, trace, (T*)trace_t);
        DMMV_LAUNCH_CHECK();
        return DMMV_OK;
    };
    // (512 threads per instance, which then screen 32 rows: 26.8 ms against 14.0 on 4096 instances of 2048 x 4096 and 8.0 against
    // 5.3 on 1024, but 2.6 against 3.9 on 100 and 2.3 against 3.6 on 20; not taken.  1024 threads: 237 and 66 ms, 16 on 100)
    auto with = [&](auto ki, auto ahead) -> dmmv_status {
        typedef decltype(ki) KI;
        constexpr bool AHEAD = decltype(ahead)::value;
        return m < BP_BLOCK ? launch(k_descent_batched_pruned<T, KI, AHEAD, true>) : launch(k_descent_batched_pruned<T, KI, AHEAD, false>);
    };
    if (c->p.nd > BP_DCAP) return n > BP_BLOCK ? with(uint16_t(), std::true_type()) : with(uint16_t(), std::false_type());
    return n > BP_BLOCK ? with(uint8_t(), std::true_type()) : with(uint8_t(), std::false_type());
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
