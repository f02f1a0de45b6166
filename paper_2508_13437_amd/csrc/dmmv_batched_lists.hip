// Batched evaluation (fp32) that scores a move over the rows that can decide it.
//
// The score of a move is max_i |fma(delta, X_ij, r_i)|, and a row can only raise it if |r_i| or |X_ij| is
// large.  Keep the rows of an instance in descending |r_i| and the rows of a column in descending
// |X_ij|; after the first p of both, every row not met yet has |r_i| <= a and |X_ij| <= c, so its value is
// at most fma(|delta|, c, a) - as computed, rounding is monotone - and once the running maximum of every
// value of D has reached that bound the maximum is final (the threshold algorithm for top-1 queries
// of Fagin, Lotem and Naor, PODS 2001).  The result is the exact score, bit for bit; a tile that the lists do not
// decide is scored over all rows.
// On activations with heavy tails some 50 of 2048 rows decide a tile at a rounded start and 150 at a local
// optimum.  The kernel that scores all rows (k_eval_batched) is bound by the vector unit's multiply-adds, and
// with an instance per lane it cannot skip rows: 18.3 ms for 4096 instances of 2048 x 4096 with 16
// levels, 2.8 ms for 500, 0.37 ms for 20 of 2048 x 768 with 8; this one, its two launches before it
// included, 0.95, 0.20 and 0.05 ms.  Bound by the vector unit still (about 27 instructions per row and 15
// values); three wavefronts per SIMD (165 registers: 33 spill at four).
// Whether the lists decide depends on the data, so what they may cost is bounded: a tile walks at most a quarter of m of
// either (half of the rows in all), and after an eighth it looks whether the bound at that point is within reach of the
// maxima it has; if not, it goes to all rows at once.  The walk over all rows uses a uniform pointer: 2.0 times as fast as
// with an address computed per row.  Worst case, rows all alike and every move lowering all of them (us; all rows with
// an instance per lane, then this kernel): 2048 x 2048, 256 instances, 16 levels 1026 and 732; 1024 x 1024, 256, 4 levels 109 and
// 96; 300 x 2048, 256, 16 levels 153 and 152.  Only on batches that fill the chip by themselves is something lost there: 1024 x
// 2048, 2000 instances, 16 / 8 / 4 levels 2415 / 1133 / 494 and 2609 / 1390 / 892, against 381 / 209 / 141 at a local optimum on
// heavy-tailed and 381 / 206 / 140 on uniform data.
//
// Per handle: the LT_LEN rows of largest |X_ij| of every column (k_list_top on the columns of X), at create, or at the
// first evaluation where the descents are pruned and never come here.
// Per evaluation: r transposed to [instance][row], the LT_LEN rows of largest |r| of every instance
// (k_list_top on those), then k_eval_lists: a workgroup holds one instance's r in LDS, lane = variable,
// the instance's rows are uniform (X read along its row-major copy), the column's rows are gathered
// from LDS.
#include <type_traits>

#include "dmmv_common.h"

namespace dmmv {

namespace {

constexpr int LT_LEN = 256;                     // rows a list holds at most
constexpr int LT_STEP = 16;                     // rows of either list between two looks at the bound
constexpr int LT_MARKS = LT_LEN / LT_STEP + 1;  // bounds: what is left before rows 0, 16, .. 256
constexpr int LT_BINS = 1024;
constexpr int64_t LT_MAX_ROWS = 16384;          // r of an instance in LDS (64 KiB)
constexpr int64_t LT_MIN_ROWS = 256;            // below, scoring all rows is as quick as sorting some

// The rows of largest |v| of a vector, in descending order: at most LT_LEN of them, row[p * sp + q * sq]
// and val likewise (filled up with row 0, which changes no maximum), and mark[p / LT_STEP] = the largest
// |v| among the rows that are not among the first p.  One workgroup per vector.  A row's bin is its
// distance from the maximum in the bits of |v| (128 bins per octave); whole bins are taken while they
// fit, so equal values cannot overflow the list - it is just shorter.
__global__ __launch_bounds__(256) void k_list_top(int64_t m, int64_t count, const float* __restrict__ v, int64_t ldv,
                                                  uint16_t* __restrict__ row, float* __restrict__ val,
                                                  float* __restrict__ mark, int64_t sp, int64_t sq) {
    __shared__ int32_t hist[LT_BINS];
    __shared__ uint32_t key[LT_LEN];
    __shared__ int32_t idx[LT_LEN];
    __shared__ float sorted[LT_LEN];
    __shared__ uint32_t sh_w[4];
    __shared__ int32_t sh_i[4];
    __shared__ int32_t sh_n, sh_edge;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t q = blockIdx.x;
    if (q >= count) return;
    const float* __restrict__ x = v + q * ldv;
    for (int b = tid; b < LT_BINS; b += 256) hist[b] = 0;
    if (tid == 0) sh_n = 0;
    auto each = [&](auto use) {                    // eight loads of a thread in flight
        for (int64_t i0 = tid; i0 < m; i0 += 8 * 256) {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = x[i0 + u * 256 < m ? i0 + u * 256 : m - 1];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u * 256 < m) use((int32_t)(i0 + u * 256), __float_as_uint(__builtin_fabsf(a[u])));
        }
    };
    auto block_umax = [&](uint32_t t) -> uint32_t {
        for (int off = 1; off < 64; off <<= 1) { const uint32_t o = __shfl_xor(t, off, 64); t = o > t ? o : t; }
        __syncthreads();
        if (lane == 0) sh_w[w] = t;
        __syncthreads();
        uint32_t r = sh_w[0];
        for (int u = 1; u < 4; ++u) r = sh_w[u] > r ? sh_w[u] : r;
        return r;
    };
    uint32_t top = 0;
    each([&](int32_t, uint32_t b) { top = b > top ? b : top; });
    top = block_umax(top);
    auto bin_of = [&](uint32_t b) -> int32_t {
        const int32_t d = (int32_t)(top >> 16) - (int32_t)(b >> 16);
        return d < LT_BINS ? d : LT_BINS - 1;
    };
    each([&](int32_t, uint32_t b) { atomicAdd(&hist[bin_of(b)], 1); });
    __syncthreads();
    // the last bin that still fits: thread t owns bins 4 t .. 4 t + 3 (the last bin, which holds all that is far
    // below, is never taken)
    {
        int32_t h[4], s = 0;
        for (int u = 0; u < 4; ++u) { h[u] = hist[4 * tid + u]; s += h[u]; }
        int32_t inc = s;
        for (int off = 1; off < 64; off <<= 1) { const int32_t o = __shfl_up(inc, off, 64); if (lane >= off) inc += o; }
        if (lane == 63) sh_i[w] = inc;
        __syncthreads();
        int32_t before = inc - s;
        for (int u = 0; u < w; ++u) before += sh_i[u];
        int32_t edge = -1;                         // highest of this thread's bins with everything up to it fitting
        for (int u = 0; u < 4; ++u) {
            before += h[u];
            if (before <= LT_LEN && 4 * tid + u < LT_BINS - 1) edge = 4 * tid + u;
        }
        const uint32_t e = block_umax((uint32_t)(edge + 1));
        if (tid == 0) sh_edge = (int32_t)e - 1;
        __syncthreads();
    }
    const int32_t edge = sh_edge;
    uint32_t rest = 0;
    each([&](int32_t i, uint32_t b) {
        if (bin_of(b) <= edge) {
            const int32_t p = atomicAdd(&sh_n, 1);
            key[p] = b;
            idx[p] = i;
        } else {
            rest = b > rest ? b : rest;
        }
    });
    rest = block_umax(rest);                       // (its barriers also publish the list)
    const int32_t n = sh_n;
    int32_t rank = 0;
    if (tid < n) {
        const uint32_t mine = key[tid];
        const int32_t mi = idx[tid];
        for (int32_t e = 0; e < n; ++e) {
            const uint32_t k = key[e];
            rank += k > mine || (k == mine && idx[e] < mi);
        }
        sorted[rank] = __uint_as_float(mine);
        row[rank * sp + q * sq] = (uint16_t)mi;
        val[rank * sp + q * sq] = x[mi];
    } else if (tid < LT_LEN) {
        row[tid * sp + q * sq] = 0;
        val[tid * sp + q * sq] = x[0];
    }
    __syncthreads();
    if (tid < LT_MARKS) {
        const int32_t p = tid * LT_STEP;
        mark[tid * sp + q * (sq == 1 ? 1 : LT_MARKS)] = p < n ? sorted[p] : __uint_as_float(rest);
    }
}

// grid.x = instance, grid.y = chunk of 256 * `groups` variables (four wavefronts x 64 variables x groups).
// KT values of D per pass; ROT (nd = KT + 1): the KT values after the lane's own one, cyclically, the
// null move enters with its known score t (as in k_eval_batched).
template <int KT, bool ROT>
__global__ __launch_bounds__(256, KT == 15 ? 3 : 4) void k_eval_lists(
    int64_t m, int64_t n, int64_t R, int32_t nd, int32_t groups, const float* __restrict__ Xt,
    const float* __restrict__ D, const int32_t* __restrict__ kidx, const float* __restrict__ scale,
    const float* __restrict__ rT, const uint16_t* __restrict__ rrow, const float* __restrict__ rval,
    const float* __restrict__ rmark, const uint16_t* __restrict__ crow, const float* __restrict__ cval,
    const float* __restrict__ cmark, int32_t look, int32_t most, int32_t radius, const uint8_t* __restrict__ var_mask,
    const InstState<float>* __restrict__ st, float* __restrict__ scores, Partial<float>* __restrict__ part) {
    extern __shared__ __align__(16) unsigned char smem[];
    float* sh_r = reinterpret_cast<float*>(smem);           // [m]
    float* shD = sh_r + m;                                  // [nd]
    float* sh_out = shD + nd;                               // ROT and scores: [4][64][nd + 1]
    __shared__ int32_t sh_row[LT_LEN];
    __shared__ float sh_val[LT_LEN], sh_mark[LT_MARKS];
    __shared__ float sh_s[4];
    __shared__ int64_t sh_c[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t q = blockIdx.x;
    float bs = 0.0f;
    int64_t bc = -1;
    const bool skip = part && !scores && st[q].done;        // a stopped instance scores nothing
    if (!skip) {
        for (int64_t i0 = tid; i0 < m; i0 += 8 * 256) {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = rT[q * m + (i0 + u * 256 < m ? i0 + u * 256 : m - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u * 256 < m) sh_r[i0 + u * 256] = a[u];
        }
        for (int32_t k = tid; k < nd; k += 256) shD[k] = D[k];
        sh_row[tid] = rrow[q * LT_LEN + tid];
        sh_val[tid] = rval[q * LT_LEN + tid];
        if (tid < LT_MARKS) sh_mark[tid] = rmark[q * LT_MARKS + tid];
    }
    __syncthreads();
    if (!skip) {
        const float sc = scale[q], t_now = st[q].t;
        for (int32_t gr = 0; gr < groups; ++gr) {
            const int64_t j0 = ((blockIdx.y * (int64_t)groups + gr) * 4 + w) * 64;
            if (j0 >= n) break;                             // whole wavefronts; no barrier below
            const int64_t j = j0 + lane;
            const int64_t jc = j < n ? j : n - 1;
            const uint32_t lc = (uint32_t)(jc - j0);
            const int32_t kcur = kidx[jc * R + q];
            const float dcur = shD[kcur];
            const bool var_ok = var_mask ? var_mask[q * n + jc] != 0 : true;
            for (int32_t k0 = 0; k0 < (ROT ? 1 : nd); k0 += KT) {
                float delta[KT], acc[KT];
#pragma unroll
                for (int v = 0; v < KT; ++v) {
                    int32_t k;
                    if (ROT) { k = kcur + 1 + v; k = k >= nd ? k - nd : k; }
                    else k = k0 + v < nd ? k0 + v : nd - 1;
                    delta[v] = step_of(shD[k], dcur, sc);
                    acc[v] = 0.0f;
                }
                bool final = false;
                for (int32_t p = 0; p < most && !final; p += LT_STEP) {
                    // the next rows of the column's list and of the instance's, all loads first
                    float x[LT_STEP], cx[LT_STEP], cr[LT_STEP];
                    uint16_t ci[LT_STEP];
                    // (uniform pointers that walk; the stride is opaque, or its multiples fill the scalar registers)
                    int64_t stride = n;
                    asm volatile("" : "+s"(stride));
                    const uint16_t* __restrict__ cr_p = crow + (int64_t)p * n + j0;
                    const float* __restrict__ cv_p = cval + (int64_t)p * n + j0;
#pragma unroll
                    for (int u = 0; u < LT_STEP; ++u) {
                        ci[u] = cr_p[lc];
                        cx[u] = cv_p[lc];
                        cr_p += stride;
                        cv_p += stride;
                    }
                    const float c = (cmark + (int64_t)(p + LT_STEP) / LT_STEP * n + j0)[lc];
#pragma unroll
                    for (int u = 0; u < LT_STEP; ++u)
                        x[u] = (Xt + (int64_t)__builtin_amdgcn_readfirstlane(sh_row[p + u]) * n + j0)[lc];
#pragma unroll
                    for (int u = 0; u < LT_STEP; ++u) cr[u] = sh_r[ci[u]];
#pragma unroll
                    for (int u = 0; u < LT_STEP; u += 2)
#pragma unroll
                        for (int v = 0; v < KT; ++v)
                            acc[v] = dmmv_max(dmmv_max(acc[v], dmmv_abs(dmmv_fma(delta[v], cx[u], cr[u]))),
                                              dmmv_abs(dmmv_fma(delta[v], cx[u + 1], cr[u + 1])));
#pragma unroll
                    for (int u = 0; u < LT_STEP; u += 2) {
                        const float r0 = sh_val[p + u], r1 = sh_val[p + u + 1];
#pragma unroll
                        for (int v = 0; v < KT; ++v)
                            acc[v] = dmmv_max(dmmv_max(acc[v], dmmv_abs(dmmv_fma(delta[v], x[u], r0))),
                                              dmmv_abs(dmmv_fma(delta[v], x[u + 1], r1)));
                    }
                    const float a = sh_mark[(p + LT_STEP) / LT_STEP];
                    bool ok = true;
#pragma unroll
                    for (int v = 0; v < KT; ++v) ok = ok && acc[v] >= dmmv_fma(dmmv_abs(delta[v]), c, a);
                    final = __ballot(!ok) == 0ull;
                    if (p + LT_STEP == look && !final) {    // is the bound after `most` rows within reach?
                        const float ce = (cmark + (int64_t)(most / LT_STEP) * n + j0)[lc], ae = sh_mark[most / LT_STEP];
                        ok = true;
#pragma unroll
                        for (int v = 0; v < KT; ++v) ok = ok && acc[v] >= dmmv_fma(dmmv_abs(delta[v]), ce, ae);
                        if (__ballot(!ok) != 0ull) break;
                    }
                }
                if (!final) {                               // the lists do not decide: all rows
                    const float* __restrict__ xp = Xt + j0;     // (uniform pointer and stride as above)
                    int64_t stride = n;
                    asm volatile("" : "+s"(stride));
                    int64_t i0 = 0;
                    for (; i0 + LT_STEP <= m; i0 += LT_STEP) {
                        float x[LT_STEP];
#pragma unroll
                        for (int u = 0; u < LT_STEP; ++u) { x[u] = xp[lc]; xp += stride; }
#pragma unroll
                        for (int u = 0; u < LT_STEP; u += 2) {
                            const float r0 = sh_r[i0 + u], r1 = sh_r[i0 + u + 1];
#pragma unroll
                            for (int v = 0; v < KT; ++v)
                                acc[v] = dmmv_max(dmmv_max(acc[v], dmmv_abs(dmmv_fma(delta[v], x[u], r0))),
                                                  dmmv_abs(dmmv_fma(delta[v], x[u + 1], r1)));
                        }
                    }
                    for (; i0 < m; ++i0, xp += stride) {
                        const float x = xp[lc], ri = sh_r[i0];
#pragma unroll
                        for (int v = 0; v < KT; ++v) acc[v] = dmmv_max(acc[v], dmmv_abs(dmmv_fma(delta[v], x, ri)));
                    }
                }
                float* out = sh_out + (w * 64 + lane) * (nd + 1);
#pragma unroll
                for (int v = 0; v < KT; ++v) {
                    int32_t k;
                    if (ROT) { k = kcur + 1 + v; k = k >= nd ? k - nd : k; }
                    else { k = k0 + v; if (k >= nd) continue; }
                    float s = acc[v];
                    if (!cand_allowed(kcur, k, radius, var_ok)) s = Limits<float>::inf();
                    const int64_t cidx = j * (int64_t)nd + k;
                    if (scores) {
                        if (ROT) out[k] = s;
                        else if (j < n) scores[q * (n * (int64_t)nd) + cidx] = s;
                    }
                    if (j < n && rec_less(s, cidx, bs, bc)) { bs = s; bc = cidx; }
                }
                if (ROT) {                                  // the null move: fma(0, a, r) = r, score t
                    const int64_t cidx = j * (int64_t)nd + kcur;
                    if (scores) out[kcur] = t_now;
                    if (j < n && rec_less(t_now, cidx, bs, bc)) { bs = t_now; bc = cidx; }
                }
                if (ROT && scores) {                        // the tile's scores are contiguous in the table
                    __builtin_amdgcn_wave_barrier();
                    float* dst = scores + q * (n * (int64_t)nd) + j0 * nd;
                    const int32_t have = (int32_t)((n - j0 < 64 ? n - j0 : 64) * nd);
                    constexpr int ND = KT + 1;
                    for (int32_t e = lane; e < have; e += 64) dst[e] = sh_out[(w * 64 + e / ND) * (ND + 1) + e % ND];
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
    }
    if (part) {
        block_argmin(bs, bc, sh_s, sh_c);
        if (tid == 0) {
            Partial<float> p;
            p.s = bs;
            p.c = bc;
            part[blockIdx.y * R + q] = p;
        }
    }
}

__global__ void k_list_transpose(const float* __restrict__ in, int64_t rows, int64_t cols, float* __restrict__ out) {
    __shared__ float tile[32][33];
    const int64_t c0 = blockIdx.x * 32ll, r0 = blockIdx.y * 32ll;
    for (int dy = threadIdx.y; dy < 32; dy += blockDim.y) {
        const int64_t rr = r0 + dy, cc = c0 + threadIdx.x;
        if (rr < rows && cc < cols) tile[dy][threadIdx.x] = in[rr * cols + cc];
    }
    __syncthreads();
    for (int dy = threadIdx.y; dy < 32; dy += blockDim.y) {
        const int64_t cc = c0 + dy, rr = r0 + threadIdx.x;
        if (rr < rows && cc < cols) out[cc * rows + rr] = tile[threadIdx.x][dy];
    }
}

}  // namespace

// Taken for fp32 batches whose r fits LDS and whose lists are worth sorting.
bool batched_lists_applicable(const dmmv_problem& p, const dmmv_options& o) {
    return p.dtype == DMMV_F32 && o.batched_eval != 2 && p.m >= LT_MIN_ROWS && p.m <= LT_MAX_ROWS && p.n > 0 && p.n <= (1 << 23) &&
           p.R <= (1 << 23) && p.nd <= 4096;   // a workgroup of 256 threads for each column and each instance: under 2^32 threads
}

size_t batched_lists_bytes(const dmmv_problem& p, bool late, ListTables* t, char* base) {
    size_t off = 0;
    auto take = [&](auto** out, size_t bytes) {
        off = (off + 255) / 256 * 256;
        *out = reinterpret_cast<std::remove_reference_t<decltype(*out)>>(base ? base + off : nullptr);
        off += bytes;
    };
    ListTables dummy;
    if (!t) t = &dummy;
    if (!late) take(&t->rT, (size_t)p.R * p.m * sizeof(float));
    take(&t->rval, (size_t)p.R * LT_LEN * sizeof(float));
    take(&t->rmark, (size_t)p.R * LT_MARKS * sizeof(float));
    take(&t->cval, (size_t)p.n * LT_LEN * sizeof(float));
    take(&t->cmark, (size_t)p.n * LT_MARKS * sizeof(float));
    take(&t->rrow, (size_t)p.R * LT_LEN * sizeof(uint16_t));
    take(&t->crow, (size_t)p.n * LT_LEN * sizeof(uint16_t));
    return off;
}

// the kernel of a number of levels, as launch(kernel, rot)
template <class F>
static dmmv_status with_kernel(int32_t nd, F launch) {
    if (nd == 16) return launch(k_eval_lists<15, true>, true);
    if (nd == 8) return launch(k_eval_lists<7, true>, true);
    if (nd == 4) return launch(k_eval_lists<3, true>, true);
    if (nd > 8) return launch(k_eval_lists<16, false>, false);
    if (nd > 4) return launch(k_eval_lists<8, false>, false);
    return launch(k_eval_lists<4, false>, false);
}

static size_t eval_lds(const dmmv_problem& p, bool rot, bool table) {
    return (size_t)(p.m + p.nd) * sizeof(float) + (rot && table ? (size_t)4 * 64 * (p.nd + 1) * sizeof(float) : 0);
}

static dmmv_status build_lists(Ctx* c) {
    const ListTables& t = c->lists;
    hipLaunchKernelGGL(k_list_top, dim3((unsigned)c->p.n), dim3(256), 0, c->stream, c->p.m, c->p.n, (const float*)c->p.A_dense,
                       c->p.lda, t.crow, t.cval, t.cmark, c->p.n, (int64_t)1);
    DMMV_LAUNCH_CHECK();
    c->lists_ready = true;
    return DMMV_OK;
}

bool batched_lists_in_use(const Ctx* c) { return c->use_lists && c->lists_ready; }

// The columns' lists of a handle that was created without them.  Not inside a capture: the captured sort would run at a
// replay, perhaps after an eager call that relied on it; such a call scores all rows.
dmmv_status batched_lists_first_use(Ctx* c) {
    if (c->lists_ready) return DMMV_OK;
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &capturing) != hipSuccess) {
        (void)hipGetLastError();
        return DMMV_OK;
    }
    return capturing == hipStreamCaptureStatusNone ? build_lists(c) : DMMV_OK;
}

dmmv_status batched_lists_prepare(Ctx* c) {
    if (!c->lists_late) DMMV_TRY(build_lists(c));
    // (here and not at a launch: an evaluation may be captured)
    return with_kernel(c->p.nd, [&](auto kernel, bool rot) -> dmmv_status {
        return eval_lds(c->p, rot, true) > 64 * 1024 ? ensure_dynamic_lds((const void*)kernel, 128 * 1024) : DMMV_OK;
    });
}

// variables per workgroup: as many as leave some 4096 workgroups, so that staging r is shared
static int32_t list_groups(int64_t n, int64_t R) {
    const int64_t all = ceil_div(n, 256);
    int64_t g = all * R / 4096;
    if (g > 8) g = 8;
    if (g > all) g = all;
    return (int32_t)(g < 1 ? 1 : g);
}

int64_t batched_lists_records(int64_t n, int64_t R) { return ceil_div(ceil_div(n, 256), list_groups(n, R)); }

// a `part`-th of the rows in whole steps, one at least and the list's length at most
static int32_t list_limit(int64_t m, int64_t part) {
    const int64_t rows = m / part / LT_STEP * LT_STEP;
    return (int32_t)(rows < LT_STEP ? LT_STEP : rows > LT_LEN ? LT_LEN : rows);
}

dmmv_status batched_eval_lists(Ctx* c, void* scores, bool want_partials) {
    const ListTables& t = c->lists;
    const int64_t m = c->p.m, n = c->p.n, R = c->p.R;
    hipLaunchKernelGGL(k_list_transpose, dim3((unsigned)ceil_div(R, 32), (unsigned)ceil_div(m, 32)), dim3(32, 8), 0, c->stream,
                       (const float*)c->r, m, R, t.rT);
    hipLaunchKernelGGL(k_list_top, dim3((unsigned)R), dim3(256), 0, c->stream, m, R, (const float*)t.rT, m, t.rrow, t.rval,
                       t.rmark, (int64_t)1, (int64_t)LT_LEN);
    const int32_t groups = list_groups(n, R);
    const int32_t most = list_limit(m, 4), look = list_limit(m, 8);
    return with_kernel(c->p.nd, [&](auto kernel, bool rot) -> dmmv_status {
        hipLaunchKernelGGL(kernel, dim3((unsigned)R, (unsigned)batched_lists_records(n, R)), dim3(256),
                           eval_lds(c->p, rot, scores != nullptr), c->stream, m, n, R,
                           c->p.nd, groups, (const float*)c->Xt, (const float*)c->D_dev, (const int32_t*)c->kidx,
                           (const float*)c->scale_dev, (const float*)t.rT, t.rrow, t.rval, t.rmark, t.crow, t.cval, t.cmark,
                           look, most, c->o.radius, c->o.var_mask, (const InstState<float>*)c->state, (float*)scores,
                           want_partials ? (Partial<float>*)c->partials : nullptr);
        DMMV_LAUNCH_CHECK();
        return DMMV_OK;
    });
}

}  // namespace dmmv
