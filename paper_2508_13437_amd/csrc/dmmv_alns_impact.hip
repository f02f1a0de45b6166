// Impact weights of a batch (worst-remove, fp32) over rows of X sorted by |X_ij|.
//
// A term of the impact sum reaches 1 exactly when |X_ij| is at least a limit that depends on the row and the instance
// alone (dmmv_alns.hip has the inequality), so with the entries of every row of X in descending order the terms that
// count are a prefix of the row's list: one binary search per row and instance replaces a comparison per entry, and no
// queue is needed to gather what passed.  X never changes, so the lists are made once per handle (144 us for 2048 x 4096).
// What a list holds of an entry is its reciprocal, the only form in which the term uses it.
//
// One workgroup takes one instance and a chunk of rows; the instance's sums lie in LDS (8 n bytes).  A wavefront takes
// up to 32 of the rows at a time: first lane = row, for the limit, the search (its dependent loads overlap over the lanes
// and the wavefronts) and the row's constants, then row by row, lane = entry of the list, the next 128 entries requested
// before these are evaluated.  The integers are added with LDS atomics, so neither their order nor the split of the rows
// over workgroups changes a weight.
// Listed half of 1024 instances of 2048 x 4096, 347 terms a row on the average: 1780 us by k_alns_impact_batched and the
// two launches it needs, now 456; of 20 instances of 2048 x 768, 66 and 27.  Where most terms count (a small alpha) a row costs its n terms,
// by the short route as well: 512 of 2048 x 4096, 3 iterations, 7.9 ms with alpha = 0.01 (12.5 by k_alns_impact_batched), 14.2 with
// 0 (21.5; 28.8 with such rows left to the exact evaluation).  33 vector instructions per 64 terms; the scalar unit
// (addresses and a row's constants: 53 instructions before two loads of 64 entries shared them, 820 us), the vector unit
// and the LDS (table and sums, conflicts included) are each busy half of the time or less, the rest is the latency of the
// loads and the uneven length of the instances' lists.
#include <type_traits>

#include "dmmv_alns_common.h"

namespace dmmv {

namespace {

constexpr int IL_WAVES = 8;                    // wavefronts of a workgroup: they share the sums
constexpr int IL_THREADS = 64 * IL_WAVES;
constexpr int64_t IL_MIN_VARS = 129;           // below, k_alns_impact_batched's narrow form
constexpr int64_t IL_MAX_VARS = 8192;          // an instance's sums in 64 KiB of LDS
constexpr int IL_BIN_SHIFT = 17;               // a bin of |X_ij|: 64 to the octave
constexpr int IL_BINS = 2048;                  // bins of a row from its largest entry's down, the last holds all that is below
constexpr int IL_TABLE = 256;                  // 2^(f/256)

// The entries of a row of X by bins of descending |X_ij| (in any order within a bin): 1 / |X_ij| in 64 bits and j.  One
// workgroup per row, a counting sort.  (A full sort of the row, bitonic in LDS: 232 us for 2048 rows of 4096.)
__global__ __launch_bounds__(256) void k_alns_order_rows(int64_t n, const float* __restrict__ Xt, double* __restrict__ inv,
                                                         uint16_t* __restrict__ col) {
    __shared__ int32_t start[IL_BINS];
    __shared__ uint32_t sh_w[4];
    const int64_t at = (int64_t)blockIdx.x * n;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int32_t n32 = (int32_t)n;
    for (int b = tid; b < IL_BINS; b += 256) start[b] = 0;
    auto key = [&](int32_t j) -> uint32_t { return __float_as_uint(__builtin_fabsf(Xt[at + j])) >> IL_BIN_SHIFT; };
    uint32_t top = 0;
    for (int32_t j = tid; j < n32; j += 256) { const uint32_t k = key(j); top = k > top ? k : top; }
    for (int off = 1; off < 64; off <<= 1) { const uint32_t o = __shfl_xor(top, off, 64); top = o > top ? o : top; }
    if (lane == 0) sh_w[w] = top;
    __syncthreads();
    for (int u = 0; u < 4; ++u) top = sh_w[u] > top ? sh_w[u] : top;
    auto bin = [&](int32_t j) -> uint32_t { const uint32_t d = top - key(j); return d < IL_BINS ? d : IL_BINS - 1; };
    for (int32_t j = tid; j < n32; j += 256) atomicAdd(&start[bin(j)], 1);
    __syncthreads();
    {
        constexpr int PER = IL_BINS / 256;
        int32_t h[PER], all = 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) { h[u] = start[PER * tid + u]; all += h[u]; }
        int32_t upto = all;
        for (int off = 1; off < 64; off <<= 1) { const int32_t o = __shfl_up(upto, off, 64); if (lane >= off) upto += o; }
        if (lane == 63) sh_w[w] = (uint32_t)upto;
        __syncthreads();
        int32_t before = upto - all;
        for (int u = 0; u < w; ++u) before += (int32_t)sh_w[u];
#pragma unroll
        for (int u = 0; u < PER; ++u) { start[PER * tid + u] = before; before += h[u]; }
    }
    __syncthreads();
    for (int32_t j = tid; j < n32; j += 256) {
        const int32_t p = atomicAdd(&start[bin(j)], 1);
        inv[at + p] = 1.0 / (double)__builtin_fabsf(Xt[at + j]);
        col[at + p] = (uint16_t)j;
    }
}

// grid: instance, chunk of rows.  The wavefronts of a workgroup take `lanes` rows of the chunk at a time, in turn.
__global__ __launch_bounds__(IL_THREADS, 8) void k_alns_impact_lists(
    int64_t m, int32_t n, int64_t R, const double* __restrict__ inv, const uint16_t* __restrict__ col,
    const float* __restrict__ scale_q, const float* __restrict__ r, const InstState<float>* __restrict__ st, double alpha,
    uint64_t* __restrict__ weight, int32_t lanes, int32_t chunk_rows, const AlnsState* __restrict__ S) {
    extern __shared__ unsigned long long sums[];            // [n]
    __shared__ double exp2t[IL_TABLE];
    __shared__ int32_t next_rows;
    const int64_t q = blockIdx.x;
    if (S[q].d_op != 1) return;
    const int lane = threadIdx.x & 63;
    for (int32_t j = threadIdx.x; j < n; j += IL_THREADS) sums[j] = 0;
    if (threadIdx.x < IL_TABLE) exp2t[threadIdx.x] = exp2((double)threadIdx.x / IL_TABLE);
    if (threadIdx.x == 0) next_rows = 0;
    const double t = (double)st[q].t, sc = (double)scale_q[q], scale = alns_impact_scale(t);
    const double rate_q = -0x1.71547652b82fep+0 * IL_TABLE * alpha / sc;
    const uint32_t entries = (uint32_t)m * (uint32_t)n;
    const __amdgpu_buffer_rsrc_t rs_inv = __builtin_amdgcn_make_buffer_rsrc((void*)inv, 0, (int)(entries * 8), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_col = __builtin_amdgcn_make_buffer_rsrc((void*)col, 0, (int)(entries * 2), 0x00020000);
    __syncthreads();
    const int32_t i_begin = (int32_t)blockIdx.y * chunk_rows;
    const int32_t i_end = i_begin + chunk_rows < (int32_t)m ? i_begin + chunk_rows : (int32_t)m;
    for (;;) {
        int32_t taken = 0;
        if (lane == 0) taken = atomicAdd(&next_rows, lanes);
        const int32_t i0 = i_begin + __builtin_amdgcn_readfirstlane(taken);
        if (i0 >= i_end) break;
        const int32_t i = i0 + lane;
        const bool row_on = lane < lanes && i < i_end;
        const double sk = __builtin_fabs((double)r[(int64_t)(row_on ? i : i0) * R + q]), v = sk * scale;
        double rate = (t - sk) * rate_q;
        const uint32_t first = (uint32_t)(row_on ? i : i0) * (uint32_t)n;      // entry of the lists
        int32_t len = 0;                                    // terms of the row that may reach 1
        bool whole = false;                                 //   the whole row, not a prefix that the limit ends
        if (row_on && v >= 0.999) {
            // (the limit lowered by 1 %, which covers the roundings on both sides: a term left out is 0)
            const float lim = (float)((t - sk) * alpha / (sc * ((log(v) + 0.01) * 1.01)));
            const double* __restrict__ row = inv + first;
            const uint32_t edge = __float_as_uint(lim) >> IL_BIN_SHIFT, top = __float_as_uint((float)(1.0 / row[0])) >> IL_BIN_SHIFT;
            int32_t hi = n;
            if (!(rate > -1e300)) {
                len = lim < Limits<float>::inf() ? n : 0;
                rate = __builtin_nan("");                   // (leaves every term to the exact evaluation)
            } else if (edge <= top && top - edge >= IL_BINS - 1) {      // the limit lies in the bin of all that is small
                len = n;
                whole = true;
            } else {
                const double most = 1.0 / (double)__uint_as_float(edge << IL_BIN_SHIFT);
                while (len < hi) {
                    const int32_t mid = (len + hi) >> 1;
                    if (row[mid] <= most) len = mid + 1; else hi = mid;
                }
            }
        }
        const unsigned long long all_whole = __ballot(whole);
        unsigned long long todo = __ballot(len > 0);
        if (todo == 0ull) continue;
        int rr = __builtin_ctzll(todo), p = 0;              // row and first place of the 128 entries at hand
        double x[2], next_x[2];
        uint32_t j[2], next_j[2];
        // (lanes past the end of a row read the next one's entries, those past the last row zeros)
        auto fetch = [&](uint32_t from) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const auto d = __builtin_amdgcn_raw_buffer_load_b64(rs_inv, lane * 8 + 512 * u, (int)(from * 8), 0);
                next_x[u] = __hiloint2double((int)d[1], (int)d[0]);
                next_j[u] = __builtin_amdgcn_raw_buffer_load_b16(rs_col, lane * 2 + 128 * u, (int)(from * 2), 0);
            }
        };
        fetch((uint32_t)__builtin_amdgcn_readlane((int)first, rr));
        while (todo != 0ull) {
            const int have = __builtin_amdgcn_readlane(len, rr);
            const double row_rate = read_lane(rate, rr), row_base = read_lane(v, rr);
            uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)first, rr);
            todo &= todo - 1;
            const int next_rr = todo ? __builtin_ctzll(todo) : rr;
            const uint32_t next_from = (uint32_t)__builtin_amdgcn_readlane((int)first, next_rr);
            for (p = 0; p < have; p += 128) {
#pragma unroll
                for (int u = 0; u < 2; ++u) { x[u] = next_x[u]; j[u] = next_j[u]; }
                from += 128;
                fetch(p + 128 < have ? from : next_from);
                // the term: base 2^(y / 256) with y = rate / |x| <= 0, by a table of 2^(f / 256) and a polynomial of degree
                // 3.  Relative error below 2^-41 (polynomial 2^-42.7; y, below 25 octaves, 2^-46) and the term below 2^24,
                // so the integer part is that of alns_impact_term unless the fraction is within 2^-15 of an integer.
                // (WHOLE: entries far below the limit too, whose terms, below 2^24 2^-26, are 0.)
                auto evaluate = [&](int u, auto whole_row) {
                    constexpr bool WHOLE = decltype(whole_row)::value;
                    const double y = row_rate * x[u];
                    const double kf = __builtin_rint(y), z = y - kf;
                    constexpr double C = 0x1.62e42fefa39efp-1 / IL_TABLE;
                    double e = __builtin_fma(z, C * C * C / 6.0, C * C / 2.0);
                    e = __builtin_fma(e, z, C);
                    e = __builtin_fma(e, z, 1.0);
                    const int k = (int)kf;
                    const double g = __builtin_ldexp(e * (row_base * exp2t[k & (IL_TABLE - 1)]), k >> 8);
                    const double down = __builtin_floor(g);
                    uint32_t term = (uint32_t)down;
                    bool ok = __builtin_fabs((g - down) - 0.5) < 0.5 - 0x1p-15;
                    if (WHOLE && y < -26.0 * IL_TABLE) { term = 0; ok = true; }
                    if (p + 64 * u + lane < have) {
                        if (!ok) term = (uint32_t)alns_impact_term(__builtin_fabs(sc * (double)(float)(1.0 / x[u])), read_lane(sk, rr), t, alpha, scale);
                        if (term) atomicAdd(&sums[j[u]], (unsigned long long)term);
                    }
                };
                if ((all_whole >> rr) & 1) {
                    evaluate(0, std::true_type());
                    if (p + 64 < have) evaluate(1, std::true_type());
                } else {
                    evaluate(0, std::false_type());
                    if (p + 64 < have) evaluate(1, std::false_type());
                }
            }
            rr = next_rr;
        }
    }
    __syncthreads();
    for (int32_t e = threadIdx.x; e < n; e += IL_THREADS)
        if (sums[e] != 0) atomicAdd((unsigned long long*)&weight[q * n + e], sums[e]);
}

}  // namespace

bool alns_impact_lists_applicable(const dmmv_problem& p) {
    return p.dtype == DMMV_F32 && p.m > 0 && p.n >= IL_MIN_VARS && p.n <= IL_MAX_VARS && p.m * p.n * 8 < (int64_t)UINT32_MAX;
}

dmmv_status alns_impact_lists_build(Ctx* c) {
    hipLaunchKernelGGL(k_alns_order_rows, dim3((unsigned)c->p.m), dim3(256), 0, c->stream, c->p.n, (const float*)c->Xt,
                       c->alns_row_inv, c->alns_row_col);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

// alns_weight (all zero before) <- the sums of the worst-remove instances
dmmv_status alns_impact_lists(Ctx* c, double alpha) {
    const int64_t m = c->p.m, R = c->p.R, about = ceil_div(R, 2) * m;      // rows of all instances: about half are listed
    // Rows a wavefront takes at a time: a search needs as many dependent loads for one row as for 64, but a small batch is
    // spread over more wavefronts (the kernel, us: 20 instances of 2048 x 768: 8 rows 27, 4 28, 16 60; 1024 of 2048 x 4096: 32 rows
    // 456, 64 484, 16 473; whole calls of 20 iterations with 1, 2, 4 and 8 rows: 3 of 64 x 2000 1293, 1378, 1514, 1777; 20 of 300 x 1000 1249,
    // 1265, 1300, 1444; 4 of 2048 x 768 1274, 1217, 1197, 1249; of 10: 20 of 1000 x 1000 845, 758, 744, 767).  Eight times as many a workgroup
    // (sixteen: 33 us with 4 rows, 479 with 32).
    int32_t lanes = 1;
    while (lanes < 32 && about >= 4096 * (int64_t)lanes) lanes *= 2;
    const int32_t chunk_rows = IL_WAVES * lanes;
    hipLaunchKernelGGL(k_alns_impact_lists, dim3((unsigned)R, (unsigned)ceil_div(m, chunk_rows)), dim3(IL_THREADS),
                       (size_t)c->p.n * sizeof(uint64_t), c->stream, m, (int32_t)c->p.n, R, c->alns_row_inv, c->alns_row_col,
                       (const float*)c->scale_dev, (const float*)c->r, (const InstState<float>*)c->state, alpha, c->alns_weight,
                       lanes, chunk_rows, (const AlnsState*)c->alns_state);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

}  // namespace dmmv
