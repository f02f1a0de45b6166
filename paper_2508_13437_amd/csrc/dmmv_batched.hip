// Batched path: R independent instances share the dense matrix X (m x n).  Instance q has
// its own target b_q, scale s_q, index vector and residual.
//
// Mapping: one lane per instance.  Within a wavefront all 64 lanes work on the same entry
// X_ij, so X is read through the scalar unit (one s_load feeds 64 instances) and every
// per-instance array is laid out instance-contiguous ([row][R], [var][R]) so that lane
// accesses coalesce.  The maximum over rows is then a serial loop inside each lane: no
// cross-lane reduction at all.  Each lane keeps KT x TJ running maxima (KT values of D for TJ
// adjacent variables) in registers.
#include "dmmv_common.h"

namespace dmmv {

// ---- layout helpers -------------------------------------------------------------------------
// out[c][r] = in[r][c] for an in matrix of `rows` x `cols` with row stride ld_in
template <class T>
__global__ void k_transpose(const T* __restrict__ in, int64_t rows, int64_t cols, int64_t ld_in,
                            T* __restrict__ out, int64_t ld_out) {
    __shared__ T tile[32][33];
    const int64_t c0 = blockIdx.x * 32ll, r0 = blockIdx.y * 32ll;
    for (int dy = threadIdx.y; dy < 32; dy += blockDim.y) {
        int64_t rr = r0 + dy, cc = c0 + threadIdx.x;
        if (rr < rows && cc < cols) tile[dy][threadIdx.x] = in[rr * ld_in + cc];
    }
    __syncthreads();
    for (int dy = threadIdx.y; dy < 32; dy += blockDim.y) {
        int64_t cc = c0 + dy, rr = r0 + threadIdx.x;
        if (rr < rows && cc < cols) out[cc * ld_out + rr] = tile[threadIdx.x][dy];
    }
}

template <class T>
static void launch_transpose(hipStream_t s, const T* in, int64_t rows, int64_t cols, int64_t ld_in,
                             T* out, int64_t ld_out) {
    if (rows == 0 || cols == 0) return;
    dim3 grid((unsigned)ceil_div(cols, 32), (unsigned)ceil_div(rows, 32));
    hipLaunchKernelGGL(k_transpose<T>, grid, dim3(32, 8), 0, s, in, rows, cols, ld_in, out, ld_out);
}

// x values [R][n] <-> kidx [n][R], 1024 at a time through LDS so that both are read and written along their rows (an
// element per thread in the order of one of them took 99 and 57 us for 4096 x 4096 and 19 and 14 for 500 x 4096; now 37 and
// 27, 9 and 6).  A tile is 2^wsh variables x the instances that make it 1024: 32 x 32, or as narrow as the batch is
// (100 000 instances of one variable left 31 of 32 lanes idle with 32 x 32: a dmmv_set_x 28 us in fp64, now 24, of which 22 are its wait for the host).
// Values are looked up in a copy of D in LDS where it fits, four a thread at a time, so that their reads are in flight together.
constexpr int XV_LEVELS = 1024, XV_TILE = 1024, XV_LDS = 1536;      // (2^wsh | 1) * (1024 >> wsh) at most
template <class T, bool SQUARE>                             // (SQUARE: 32 x 32, the shifts as constants)
__global__ __launch_bounds__(256) void k_values_to_index_batched(const T* __restrict__ x, const T* __restrict__ D,
                                                                 int32_t nd, int64_t n, int64_t R, int32_t log_wide,
                                                                 int32_t* __restrict__ kidx, int32_t* flags) {
    __shared__ int32_t tile[SQUARE ? 32 * 33 : XV_LDS];
    __shared__ T sh_d[XV_LEVELS];
    const int wsh = SQUARE ? 5 : log_wide, hsh = 10 - wsh, wide = 1 << wsh, pitch = wide | 1;
    const int64_t j0 = (int64_t)blockIdx.x << wsh, q0 = (blockIdx.y + blockIdx.z * (int64_t)gridDim.y) << hsh;
    if (q0 >= R) return;
    const bool in_lds = nd <= XV_LEVELS;
    T v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u;
        const int64_t q = q0 + (e >> wsh), j = j0 + (e & (wide - 1));
        v[u] = x[(q < R ? q : R - 1) * n + (j < n ? j : n - 1)];
    }
    for (int32_t k = threadIdx.x; in_lds && k < nd; k += 256) sh_d[k] = D[k];
    __syncthreads();
    int32_t lo[4] = {0, 0, 0, 0};                           // a value of D is among the `len` levels from here on
    for (int32_t len = nd; len > 1;) {
        const int32_t half = len >> 1;
        T d[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) d[u] = in_lds ? sh_d[lo[u] + half - 1] : D[lo[u] + half - 1];
#pragma unroll
        for (int u = 0; u < 4; ++u) lo[u] += d[u] < v[u] ? half : 0;
        len -= half;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u;
        if (!((in_lds ? sh_d[lo[u]] : D[lo[u]]) == v[u])) { atomicOr(&flags[FLAG_ERROR], ERRBIT_X_NOT_IN_D); lo[u] = 0; }
        tile[(e >> wsh) * pitch + (e & (wide - 1))] = lo[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u, tq = e & ((1 << hsh) - 1), tj = e >> hsh;
        const int64_t j = j0 + tj, q = q0 + tq;
        if (j < n && q < R) kidx[j * R + q] = tile[tq * pitch + tj];
    }
}

template <class T, bool SQUARE>
__global__ __launch_bounds__(256) void k_index_to_values_batched(const int32_t* __restrict__ kidx, const T* __restrict__ D,
                                                                 int64_t n, int64_t R, int32_t log_wide, T* __restrict__ x) {
    __shared__ T tile[SQUARE ? 32 * 33 : XV_LDS];
    const int wsh = SQUARE ? 5 : log_wide, hsh = 10 - wsh, wide = 1 << wsh, pitch = wide | 1;
    const int64_t j0 = (int64_t)blockIdx.x << wsh, q0 = (blockIdx.y + blockIdx.z * (int64_t)gridDim.y) << hsh;
    if (q0 >= R) return;
    int32_t k[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u;
        const int64_t j = j0 + (e >> hsh), q = q0 + (e & ((1 << hsh) - 1));
        k[u] = kidx[(j < n ? j : n - 1) * R + (q < R ? q : R - 1)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u;
        tile[(e & ((1 << hsh) - 1)) * pitch + (e >> hsh)] = D[k[u]];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u;
        const int64_t q = q0 + (e >> wsh), j = j0 + (e & (wide - 1));
        if (j < n && q < R) x[q * n + j] = tile[(e >> wsh) * pitch + (e & (wide - 1))];
    }
}

static int32_t values_wsh(int64_t n, int64_t R) {
    int32_t a = 0, b = 0;                                   // whole powers of two from n and R on, 32 at most
    while (a < 5 && 1ll << a < n) ++a;
    while (b < 5 && 1ll << b < R) ++b;
    return a < 5 ? a : 10 - b;
}
static dim3 values_grid(int64_t n, int64_t R) {
    const int32_t wsh = values_wsh(n, R);
    const int64_t gq = ceil_div(R, XV_TILE >> wsh), gy = gq < 32768 ? gq : 32768;
    return dim3((unsigned)ceil_div(n, 1ll << wsh), (unsigned)gy, (unsigned)ceil_div(gq, gy));
}

// ---- residual -------------------------------------------------------------------------------
// lane = instance, TI rows per lane at a time.  Column-major X: the TI rows of column j are
// contiguous, read with one scalar load.  Order over j is ascending per (row, instance).
template <class T, int TI>
__global__ __launch_bounds__(256) void k_residual_batched(
    int64_t m, int64_t n, int64_t R, const T* __restrict__ X, int64_t ldx, const T* __restrict__ D,
    int32_t nd, const int32_t* __restrict__ kidx, const T* __restrict__ scale,
    const T* __restrict__ Bt, T* __restrict__ r) {
    extern __shared__ unsigned char smem[];
    T* shD = reinterpret_cast<T*>(smem);
    for (int k = threadIdx.x; k < nd; k += blockDim.x) shD[k] = D[k];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t q = blockIdx.x * 64ll + lane;
    const int64_t qc = q < R ? q : R - 1;
    const int64_t i0 = (blockIdx.y * 4ll + w) * TI;
    if (i0 >= m) return;
    T acc[TI];
#pragma unroll
    for (int u = 0; u < TI; ++u) acc[u] = (T)0;
    // the level indices of RJ variables are fetched together (one memory latency for RJ
    // variables); the order of the additions stays j ascending
    constexpr int RJ = 8;
    for (int64_t j0 = 0; j0 < n; j0 += RJ) {
        int32_t kk[RJ];
#pragma unroll
        for (int e = 0; e < RJ; ++e) kk[e] = kidx[(j0 + e < n ? j0 + e : n - 1) * R + qc];
#pragma unroll
        for (int e = 0; e < RJ; ++e) {
            if (j0 + e >= n) break;                          // the same for the whole wavefront
            const T v = shD[kk[e]];
            const T* __restrict__ xp = X + ldx * (j0 + e) + i0;
#pragma unroll
            for (int u = 0; u < TI; ++u) {
                const T a = (i0 + u < m) ? xp[u] : (T)0;
                acc[u] = dmmv_fma(a, v, acc[u]);
            }
        }
    }
    if (q < R) {
        const T sc = scale[q];
#pragma unroll
        for (int u = 0; u < TI; ++u)
            if (i0 + u < m) r[(i0 + u) * R + q] = dmmv_fma(acc[u], sc, -Bt[(i0 + u) * R + q]);
    }
}

// The same sums for large batches: the 4 wavefronts of a workgroup take 4 groups of 64 instances
// and the SAME RT rows, so a tile of X (RC columns x RT rows) is staged once in LDS for all 256
// instances and read back as broadcasts (every lane of a wavefront needs the same entry), instead
// of travelling through the scalar cache once per wavefront.  Order over j ascending as above.
constexpr int RT = 32;                      // rows per lane
constexpr int RC = 32;                      // columns per staged tile

template <class T>
__global__ __launch_bounds__(256) void k_residual_batched_tiled(
    int64_t m, int64_t n, int64_t R, const T* __restrict__ X, int64_t ldx, const T* __restrict__ D,
    int32_t nd, const int32_t* __restrict__ kidx, const T* __restrict__ scale,
    const T* __restrict__ Bt, T* __restrict__ r) {
    extern __shared__ unsigned char smem[];
    T* shD = reinterpret_cast<T*>(smem);
    __shared__ __align__(16) T tile[2][RC][RT];
    for (int k = threadIdx.x; k < nd; k += blockDim.x) shD[k] = D[k];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t q = (blockIdx.x * 4ll + w) * 64 + lane;
    const int64_t qc = q < R ? q : R - 1;
    const int64_t i0 = blockIdx.y * (int64_t)RT;
    // staging: thread t fetches 4 consecutive rows (t % 8) * 4 .. + 3 of column t / 8 of the tile
    const int sc_col = threadIdx.x >> 3, sc_row = (threadIdx.x & 7) * 4;
    T stage[4];
    auto fetch = [&](int64_t j0) {
        const int64_t j = j0 + sc_col < n ? j0 + sc_col : n - 1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + sc_row + u;
            stage[u] = X[ldx * j + (i < m ? i : m - 1)];     // rows past the end are never stored below
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int u = 0; u < 4; ++u) tile[buf][sc_col][sc_row + u] = stage[u];
    };
    T acc[RT];
#pragma unroll
    for (int u = 0; u < RT; ++u) acc[u] = (T)0;
    fetch(0);
    stash(0);
    __syncthreads();
    int buf = 0;
    for (int64_t j0 = 0; j0 < n; j0 += RC, buf ^= 1) {
        if (j0 + RC < n) fetch(j0 + RC);                     // the next tile travels while this one is used
        constexpr int RJ = 8;
        for (int jc0 = 0; jc0 < RC; jc0 += RJ) {
            int32_t kk[RJ];
#pragma unroll
            for (int e = 0; e < RJ; ++e) {
                const int64_t j = j0 + jc0 + e;
                kk[e] = kidx[(j < n ? j : n - 1) * R + qc];
            }
#pragma unroll
            for (int e = 0; e < RJ; ++e) {
                if (j0 + jc0 + e >= n) break;                // the same for the whole workgroup
                const T v = shD[kk[e]];
#pragma unroll
                for (int u = 0; u < RT; ++u) acc[u] = dmmv_fma(tile[buf][jc0 + e][u], v, acc[u]);
            }
        }
        if (j0 + RC < n) stash(buf ^ 1);
        __syncthreads();
    }
    if (q < R) {
        const T sc = scale[q];
#pragma unroll
        for (int u = 0; u < RT; ++u)
            if (i0 + u < m) r[(i0 + u) * R + q] = dmmv_fma(acc[u], sc, -Bt[(i0 + u) * R + q]);
    }
}

// per-instance max |r|: lane = instance, the rows split over workgroups and their wavefronts, the maxima
// joined through memory (|r| >= 0: the bit patterns order like the values).  One workgroup per 64 instances
// walked its 2048 rows one at a time: 39 us for 500 instances, now 9 with the clearing launch.
// Few rows (ONE): a single workgroup per 64 instances after all, sixteen wavefronts with eight rows in flight
// each, which stores its maxima: no clearing launch.
constexpr int MB_ROWS = 128;                               // rows per workgroup (32 per wavefront)
constexpr int64_t MB_ONE_ROWS = 512;                       // up to four passes of a wavefront in one workgroup
template <class T>
__global__ void k_clear_t(int64_t R, InstState<T>* st) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q < R) st[q].t = (T)0;
}
__device__ __forceinline__ void raise_to(float* p, float v) { atomicMax(reinterpret_cast<unsigned int*>(p), __float_as_uint(v)); }
__device__ __forceinline__ void raise_to(double* p, double v) {
    atomicMax(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v));
}
template <class T, bool ONE>
__global__ __launch_bounds__(ONE ? 1024 : 256) void k_maxabs_batched(int64_t m, int64_t R, const T* __restrict__ r,
                                                                     InstState<T>* st) {
    constexpr int WAVES = ONE ? 16 : 4;
    __shared__ T sh[WAVES][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t q = blockIdx.x * 64ll + lane;
    const int64_t qc = q < R ? q : R - 1;
    const int64_t rows = ONE ? m : MB_ROWS;                // per workgroup and pass
    T v = (T)0;
    for (int64_t b0 = blockIdx.y * rows; b0 < m; b0 += gridDim.y * rows)
        for (int64_t i0 = b0 + w; i0 < b0 + rows && i0 < m; i0 += WAVES * 8) {
            T a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = r[(i0 + WAVES * u < m ? i0 + WAVES * u : i0) * R + qc];
#pragma unroll
            for (int u = 0; u < 8; ++u) v = dmmv_max(v, dmmv_abs(a[u]));
        }
    sh[w][lane] = v;
    __syncthreads();
    if (w == 0 && q < R) {
#pragma unroll
        for (int ww = 1; ww < WAVES; ++ww) v = dmmv_max(v, sh[ww][lane]);
        if (ONE) st[q].t = v;
        else raise_to(&st[q].t, v);
    }
}

#ifndef DMMV_BATCHED_RB
#define DMMV_BATCHED_RB 8      // rows of X and r whose loads are in flight together
#endif

// ---- evaluation -----------------------------------------------------------------------------
// grid.x = group of 64 instances, grid.y = chunk of `chunk_cols` variables.  A block has four
// wavefronts; each takes tiles of TJ variables of the chunk in turn.  For nd > KT the values
// of D are covered KT at a time.  Xt is the row-major copy of X, so the TJ entries of a row
// are one scalar load.
// ROT (nd = KT + 1): the null move is not computed at all.  Every lane takes the KT values
// AFTER its own current one, cyclically (the steps are per-lane registers anyway), and the null
// move enters the table and the arg-min with its known score t.
template <class T, int KT, int TJ, bool ROT = false, int RB = DMMV_BATCHED_RB>
__global__ __launch_bounds__(256) void k_eval_batched(
    int64_t m, int64_t n, int64_t R, int32_t nd, int32_t chunk_cols, const T* __restrict__ Xt,
    const T* __restrict__ D, const int32_t* __restrict__ kidx, const T* __restrict__ scale,
    const T* __restrict__ r, int32_t radius, const uint8_t* __restrict__ var_mask,
    const InstState<T>* __restrict__ st, T* __restrict__ scores, Partial<T>* __restrict__ part) {
    extern __shared__ unsigned char smem[];
    T* shD = reinterpret_cast<T*>(smem);
    __shared__ T sh_s[4][64];
    __shared__ int64_t sh_c[4][64];
    for (int k = threadIdx.x; k < nd; k += blockDim.x) shD[k] = D[k];
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t q = blockIdx.x * 64ll + lane;
    const bool live = q < R;
    const int64_t qc = live ? q : R - 1;
    const T sc = scale[qc];
    const T t_now = st[qc].t;
    const bool skip = part && !scores && st[qc].done;   // stopped instances score nothing
    const int64_t jbeg = blockIdx.y * (int64_t)chunk_cols;
    const int64_t jend = jbeg + chunk_cols < n ? jbeg + chunk_cols : n;

    T bs = (T)0;
    int64_t bc = -1;
    // whole wavefront stopped: nothing to do (uniform branch)
    const bool wave_idle = __builtin_amdgcn_readfirstlane(__ballot(!skip && live) == 0ull ? 1 : 0) != 0;
    if (!wave_idle) {
        for (int64_t j0 = jbeg + w * TJ; j0 < jend; j0 += 4 * TJ) {
            int32_t kcur[TJ];
            T dcur[TJ];
#pragma unroll
            for (int u = 0; u < TJ; ++u) {
                const int64_t j = j0 + u < n ? j0 + u : n - 1;
                kcur[u] = kidx[j * R + qc];
                dcur[u] = shD[kcur[u]];
            }
            for (int32_t k0 = 0; k0 < (ROT ? 1 : nd); k0 += KT) {
                T delta[TJ][KT], acc[TJ][KT];
#pragma unroll
                for (int u = 0; u < TJ; ++u)
#pragma unroll
                    for (int v = 0; v < KT; ++v) {
                        int32_t k;
                        if (ROT) { k = kcur[u] + 1 + v; k = k >= nd ? k - nd : k; }
                        else k = k0 + v < nd ? k0 + v : nd - 1;
                        delta[u][v] = step_of(shD[k], dcur[u], sc);
                        acc[u][v] = (T)0;
                    }
                if (ROT) {
                    // the value indices are recomputed after the row loop rather than kept in
                    // registers across it
#pragma unroll
                    for (int u = 0; u < TJ; ++u) asm volatile("" : "+v"(kcur[u]));
                }
                if (j0 + TJ <= n) {
                    // RB rows per pass: all their loads (r in vector registers, the X tile in
                    // scalar registers) are issued before the first row is scored, so one pass
                    // of a wavefront computes for longer than the loads of the other resident
                    // wavefront take.
                    const T* __restrict__ xrow = Xt + j0;
#pragma unroll RB
                    for (int64_t i = 0; i < m; ++i) {
                        const T ri = r[i * R + qc];
                        const T* __restrict__ xp = xrow + i * n;
#pragma unroll
                        for (int u = 0; u < TJ; ++u) {
                            const T a = xp[u];
#pragma unroll
                            for (int v = 0; v < KT; ++v)
                                acc[u][v] = dmmv_max(acc[u][v], dmmv_abs(dmmv_fma(delta[u][v], a, ri)));
                        }
                    }
                } else {
                    // ragged last tile: element-wise bounds
                    for (int64_t i = 0; i < m; ++i) {
                        const T ri = r[i * R + qc];
#pragma unroll
                        for (int u = 0; u < TJ; ++u) {
                            const int64_t j = j0 + u < n ? j0 + u : n - 1;
                            const T a = Xt[i * n + j];
#pragma unroll
                            for (int v = 0; v < KT; ++v)
                                acc[u][v] = dmmv_max(acc[u][v], dmmv_abs(dmmv_fma(delta[u][v], a, ri)));
                        }
                    }
                }
                if (live && !skip) {
#pragma unroll
                    for (int u = 0; u < TJ; ++u) {
                        const int64_t j = j0 + u;
                        if (j >= jend) continue;                 // (no break: keeps acc in registers)
                        const bool var_ok = var_mask ? var_mask[q * n + j] != 0 : true;
#pragma unroll
                        for (int v = 0; v < KT; ++v) {
                            int32_t k;
                            if (ROT) { k = kcur[u] + 1 + v; k = k >= nd ? k - nd : k; }
                            else { k = k0 + v; if (k >= nd) continue; }
                            T val = acc[u][v];
                            if (!cand_allowed(kcur[u], k, radius, var_ok)) val = Limits<T>::inf();
                            const int64_t cidx = j * (int64_t)nd + k;
                            if (scores) scores[q * (n * (int64_t)nd) + cidx] = val;
                            if (rec_less(val, cidx, bs, bc)) { bs = val; bc = cidx; }
                        }
                        if (ROT) {                               // the null move: fma(0, a, r) = r, score t
                            const int64_t cidx = j * (int64_t)nd + kcur[u];
                            if (scores) scores[q * (n * (int64_t)nd) + cidx] = t_now;
                            if (rec_less(t_now, cidx, bs, bc)) { bs = t_now; bc = cidx; }
                        }
                    }
                }
            }
        }
    }
    if (part) {
        sh_s[w][lane] = bs;
        sh_c[w][lane] = bc;
        __syncthreads();
        if (w == 0 && live) {
            T s = sh_s[0][lane];
            int64_t c = sh_c[0][lane];
#pragma unroll
            for (int ww = 1; ww < 4; ++ww)
                if (rec_less(sh_s[ww][lane], sh_c[ww][lane], s, c)) { s = sh_s[ww][lane]; c = sh_c[ww][lane]; }
            Partial<T> p; p.s = s; p.c = c;
            part[blockIdx.y * R + q] = p;
        }
    }
}

// ---- apply ----------------------------------------------------------------------------------
// lane = instance; each instance updates with its own column of X (a gather).  grid.y splits
// the rows; the block with blockIdx.y == 0 also updates x, t and the trace.
template <class T>
__global__ void k_apply_batched(int64_t m, int64_t n, int64_t R, const T* __restrict__ X,
                                int64_t ldx, T* __restrict__ r, int32_t* __restrict__ kidx,
                                InstState<T>* st, int32_t t_from_score, int32_t iters,
                                dmmv_move* trace, T* trace_t, int32_t rows_per_block,
                                const int32_t* __restrict__ orig) {
    const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (q >= R) return;
    const int32_t j = st[q].apply_j;
    if (j < 0) return;
    const T delta = st[q].delta;
    const T* __restrict__ col = X + ldx * (int64_t)j;
    const int64_t i0 = blockIdx.y * (int64_t)rows_per_block;
    const int64_t i1 = i0 + rows_per_block < m ? i0 + rows_per_block : m;
    // eight rows' loads in flight (one row at a time the pass runs at the latency of its loads: 87 us for 500
    // instances of 2048 rows in blocks of 256 rows, now 13 in blocks of 64)
    for (int64_t ib = i0; ib < i1; ib += 8) {
        T a[8], x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = ib + u < i1 ? ib + u : i1 - 1;
            a[u] = col[i];
            x[u] = r[i * R + q];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (ib + u < i1) r[(ib + u) * R + q] = dmmv_fma(delta, a[u], x[u]);
    }
    if (blockIdx.y == 0) {
        const int32_t k = st[q].apply_k;
        const int32_t moves = st[q].moves;
        kidx[(int64_t)j * R + q] = k;
        if (t_from_score) {
            const T best_s = st[q].best_s;
            st[q].t = best_s;
            if (moves < iters) {
                const int64_t slot = (orig ? (int64_t)orig[q] : q) * (int64_t)iters + moves;   // caller's instance number
                if (trace) { trace[slot].j = j; trace[slot].k = k; }
                if (trace_t) trace_t[slot] = best_s;
            }
        }
        st[q].moves = moves + 1;
    }
}

// =========================================================================================
// host dispatch
// =========================================================================================
template <class T>
static dmmv_status build_t(Ctx* c) {
    const int64_t m = c->p.m, n = c->p.n, R = c->p.R;
    // X is column-major m x n = row-major n x m with stride lda; Xt[i][j] = X[j][i]
    launch_transpose<T>(c->stream, (const T*)c->p.A_dense, n, m, c->p.lda, (T*)c->Xt, n);
    // B is [R][m]; Bt[i][q]
    launch_transpose<T>(c->stream, (const T*)c->p.b, R, m, m, (T*)c->Bt, R);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
static dmmv_status residual_t(Ctx* c) {
    const int64_t m = c->p.m, n = c->p.n, R = c->p.R;
    if (m == 0) return DMMV_OK;
    // rows per lane: every variable's level index is read once per TI rows, so tall matrices take
    // many rows per lane (as long as the launch still fills the chip)
    auto launch = [&](auto kernel, int ti) {
        dim3 grid((unsigned)ceil_div(R, 64), (unsigned)ceil_div(m, 4 * ti));
        hipLaunchKernelGGL(kernel, grid, dim3(256), (size_t)c->p.nd * sizeof(T), c->stream,
                           m, n, R, (const T*)c->p.A_dense, c->p.lda, (const T*)c->D_dev, c->p.nd,
                           (const int32_t*)c->kidx, (const T*)c->scale_dev, (const T*)c->Bt, (T*)c->r);
    };
    if (R >= 256 && ceil_div(R, 256) * ceil_div(m, RT) >= 512) {
        dim3 grid((unsigned)ceil_div(R, 256), (unsigned)ceil_div(m, RT));
        hipLaunchKernelGGL(k_residual_batched_tiled<T>, grid, dim3(256), (size_t)c->p.nd * sizeof(T), c->stream,
                           m, n, R, (const T*)c->p.A_dense, c->p.lda, (const T*)c->D_dev, c->p.nd,
                           (const int32_t*)c->kidx, (const T*)c->scale_dev, (const T*)c->Bt, (T*)c->r);
    } else if (ceil_div(R, 64) * ceil_div(m, 4 * 32) >= 512) {
        launch(k_residual_batched<T, 32>, 32);
    } else {
        launch(k_residual_batched<T, 8>, 8);
    }
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
static dmmv_status maxabs_t(Ctx* c) {
    if (c->p.m <= MB_ONE_ROWS) {
        hipLaunchKernelGGL((k_maxabs_batched<T, true>), dim3((unsigned)ceil_div(c->p.R, 64)), dim3(1024), 0, c->stream, c->p.m,
                           c->p.R, (const T*)c->r, (InstState<T>*)c->state);
        DMMV_LAUNCH_CHECK();
        return DMMV_OK;
    }
    int64_t rows = ceil_div(c->p.m, MB_ROWS);
    if (rows > 65535) rows = 65535;
    hipLaunchKernelGGL(k_clear_t<T>, dim3((unsigned)ceil_div(c->p.R, 256)), dim3(256), 0, c->stream, c->p.R, (InstState<T>*)c->state);
    hipLaunchKernelGGL((k_maxabs_batched<T, false>), dim3((unsigned)ceil_div(c->p.R, 64), (unsigned)rows), dim3(256), 0, c->stream,
                       c->p.m, c->p.R, (const T*)c->r, (InstState<T>*)c->state);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T, int KT, int TJ, bool ROT = false>
static dmmv_status eval_launch(Ctx* c, void* scores, bool want_partials) {
    dim3 grid((unsigned)ceil_div(c->p.R, 64), (unsigned)c->n_partials);
    hipLaunchKernelGGL((k_eval_batched<T, KT, TJ, ROT>), grid, dim3(256), (size_t)c->p.nd * sizeof(T), c->stream,
                       c->p.m, c->p.n, c->p.R, c->p.nd, c->chunk_cols, (const T*)c->Xt,
                       (const T*)c->D_dev, (const int32_t*)c->kidx, (const T*)c->scale_dev,
                       (const T*)c->r, c->o.radius, c->o.var_mask, (const InstState<T>*)c->state,
                       (T*)scores, want_partials ? (Partial<T>*)c->partials : nullptr);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
static dmmv_status eval_t(Ctx* c, void* scores, bool want_partials) {
    if ((size_t)c->p.nd * sizeof(T) > 48 * 1024)
        return fail(DMMV_ERR_UNSUPPORTED, "batched path: nd = %d does not fit the LDS value table", c->p.nd);
    // the usual code widths (4, 3 and 2 bits) in fp32: without computing the null move
    // (in fp64 the variant needs more than the 256 registers that two wavefronts per SIMD leave)
    if (sizeof(T) == 4) {
        if (c->p.nd == 16) return eval_launch<float, 15, 4, true>(c, scores, want_partials);
        if (c->p.nd == 8) return eval_launch<float, 7, 8, true>(c, scores, want_partials);
        if (c->p.nd == 4) return eval_launch<float, 3, 8, true>(c, scores, want_partials);
    }
    if (c->p.nd > 8) return eval_launch<T, 16, 4>(c, scores, want_partials);
    if (c->p.nd > 4) return eval_launch<T, 8, 8>(c, scores, want_partials);
    return eval_launch<T, 4, 8>(c, scores, want_partials);
}

template <class T>
static dmmv_status apply_t(Ctx* c, bool t_from_score, int32_t iters, dmmv_move* trace, void* trace_t) {
    const int64_t m = c->p.m, R = c->p.R;
    // 64 rows a block, more where the rows would take more blocks than a grid's second dimension holds
    const int32_t rows_per_block = (int32_t)(m > 65535ll * 64 ? ceil_div(m, 65535) : 64);
    dim3 grid((unsigned)ceil_div(R, 64), (unsigned)(m > 0 ? ceil_div(m, rows_per_block) : 1));
    hipLaunchKernelGGL(k_apply_batched<T>, grid, dim3(64), 0, c->stream, m, c->p.n, R,
                       (const T*)c->p.A_dense, c->p.lda, (T*)c->r, c->kidx, (InstState<T>*)c->state,
                       (int32_t)t_from_score, iters, trace, (T*)trace_t, rows_per_block,
                       c->cmp_on ? (const int32_t*)c->cmp_orig : nullptr);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
static dmmv_status set_x_t(Ctx* c, const void* x) {
    const int32_t wsh = values_wsh(c->p.n, c->p.R);
    hipLaunchKernelGGL((wsh == 5 ? k_values_to_index_batched<T, true> : k_values_to_index_batched<T, false>), values_grid(c->p.n, c->p.R), dim3(256), 0, c->stream,
                       (const T*)x, (const T*)c->D_dev, c->p.nd, c->p.n, c->p.R, wsh, c->kidx, c->flags);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

template <class T>
static dmmv_status get_x_t(Ctx* c, const int32_t* kidx, void* x) {
    const int32_t wsh = values_wsh(c->p.n, c->p.R);
    hipLaunchKernelGGL((wsh == 5 ? k_index_to_values_batched<T, true> : k_index_to_values_batched<T, false>), values_grid(c->p.n, c->p.R), dim3(256), 0, c->stream,
                       kidx, (const T*)c->D_dev, c->p.n, c->p.R, wsh, (T*)x);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

// =========================================================================================
// dropping stopped instances from the descent
// =========================================================================================
// Instances stop at different iterations, and a wavefront works as long as one of its 64
// instances does.  At the host's polling points the instances still running are therefore
// gathered into a dense "virtual" batch of their own (same layouts, stride = their number),
// which the loop's kernels then work on; orig[p] is the caller's number of virtual instance p.
// Before a new gather, and at the end, the virtual batch is scattered back into the full arrays.
template <class T>
__global__ void k_cmp_scatter(int64_t m, int64_t n, int64_t Rv, int64_t Rf, const int32_t* __restrict__ orig,
                              const T* __restrict__ r_v, T* __restrict__ r_f,
                              const int32_t* __restrict__ k_v, int32_t* __restrict__ k_f,
                              const InstState<T>* __restrict__ st_v, InstState<T>* __restrict__ st_f) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t e = t0; e < m * Rv; e += stride) r_f[(e / Rv) * Rf + orig[e % Rv]] = r_v[e];
    for (int64_t e = t0; e < n * Rv; e += stride) k_f[(e / Rv) * Rf + orig[e % Rv]] = k_v[e];
    for (int64_t p = t0; p < Rv; p += stride) st_f[orig[p]] = st_v[p];
}

// the running instances in ascending order (single workgroup); their number goes to
// flags[FLAG_ACTIVE]
template <class T>
__global__ __launch_bounds__(1024) void k_cmp_list(int64_t Rf, const InstState<T>* __restrict__ st_f,
                                                   int32_t* __restrict__ orig, int32_t* flags) {
    __shared__ int32_t sh_cnt[16];
    __shared__ int32_t sh_base;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (threadIdx.x == 0) sh_base = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < Rf; b0 += 1024) {
        const int64_t q = b0 + threadIdx.x;
        const bool on = q < Rf && !st_f[q].done;
        const unsigned long long bal = __ballot(on);
        if (lane == 0) sh_cnt[w] = __popcll(bal);
        __syncthreads();
        int32_t before = 0, all = 0;
        for (int u = 0; u < 16; ++u) { if (u < w) before += sh_cnt[u]; all += sh_cnt[u]; }
        const int32_t base = sh_base;
        if (on) orig[base + before + __popcll(bal & ((1ull << lane) - 1ull))] = (int32_t)q;
        __syncthreads();
        if (threadIdx.x == 0) sh_base = base + all;
        __syncthreads();
    }
    if (threadIdx.x == 0) flags[FLAG_ACTIVE] = sh_base;
}

template <class T>
__global__ void k_cmp_gather(int64_t m, int64_t n, int64_t Rv, int64_t Rf, const int32_t* __restrict__ orig,
                             const T* __restrict__ r_f, T* __restrict__ r_v,
                             const int32_t* __restrict__ k_f, int32_t* __restrict__ k_v,
                             const InstState<T>* __restrict__ st_f, InstState<T>* __restrict__ st_v,
                             const T* __restrict__ sc_f, T* __restrict__ sc_v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t e = t0; e < m * Rv; e += stride) r_v[e] = r_f[(e / Rv) * Rf + orig[e % Rv]];
    for (int64_t e = t0; e < n * Rv; e += stride) k_v[e] = k_f[(e / Rv) * Rf + orig[e % Rv]];
    for (int64_t p = t0; p < Rv; p += stride) { st_v[p] = st_f[orig[p]]; sc_v[p] = sc_f[orig[p]]; }
}

template <class T>
static dmmv_status compact_scatter_t(Ctx* c) {
    hipLaunchKernelGGL(k_cmp_scatter<T>, dim3(2048), dim3(256), 0, c->stream, c->p.m, c->p.n, c->p.R, c->cmp_full_R,
                       (const int32_t*)c->cmp_orig, (const T*)c->r, (T*)c->cmp_full_r, (const int32_t*)c->kidx,
                       c->cmp_full_kidx, (const InstState<T>*)c->state, (InstState<T>*)c->cmp_full_state);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

static void compact_to_full(Ctx* c) {
    c->r = c->cmp_full_r; c->kidx = c->cmp_full_kidx; c->state = c->cmp_full_state;
    c->scale_dev = c->cmp_full_scale; c->p.R = c->cmp_full_R;
    c->cmp_on = false;
}

// At a polling point of the descent: how many instances still run (HOST, *active_out), and the
// loop's arrays re-pointed at a virtual batch of just those when that is worth it.
template <class T>
static dmmv_status compact_t(Ctx* c, int32_t* active_out) {
    if (c->cmp_on) {
        DMMV_TRY(compact_scatter_t<T>(c));
        compact_to_full(c);
    }
    const int64_t Rf = c->p.R, m = c->p.m, n = c->p.n;
    hipLaunchKernelGGL(k_cmp_list<T>, dim3(1), dim3(1024), 0, c->stream, Rf, (const InstState<T>*)c->state,
                       c->cmp_orig, c->flags);
    int32_t active = 0;
    DMMV_HIP_CHECK(hipMemcpyAsync(&active, &c->flags[FLAG_ACTIVE], sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    DMMV_HIP_CHECK(hipStreamSynchronize(c->stream));
    *active_out = active;
    if (active == 0 || (int64_t)active * 4 > Rf * 3) return DMMV_OK;      // nothing left, or not worth it
    c->cmp_full_r = c->r; c->cmp_full_kidx = c->kidx; c->cmp_full_state = c->state;
    c->cmp_full_scale = c->scale_dev; c->cmp_full_R = Rf;
    hipLaunchKernelGGL(k_cmp_gather<T>, dim3(2048), dim3(256), 0, c->stream, m, n, (int64_t)active, Rf,
                       (const int32_t*)c->cmp_orig, (const T*)c->cmp_full_r, (T*)c->cmp_r,
                       (const int32_t*)c->cmp_full_kidx, c->cmp_kidx, (const InstState<T>*)c->cmp_full_state,
                       (InstState<T>*)c->cmp_state, (const T*)c->cmp_full_scale, (T*)c->cmp_scale);
    DMMV_LAUNCH_CHECK();
    c->r = c->cmp_r; c->kidx = c->cmp_kidx; c->state = c->cmp_state; c->scale_dev = c->cmp_scale;
    c->p.R = active;
    c->cmp_on = true;
    return DMMV_OK;
}

dmmv_status batched_compact(Ctx* c, int32_t* active_out) {
    return c->p.dtype == DMMV_F64 ? compact_t<double>(c, active_out) : compact_t<float>(c, active_out);
}
// back to the caller's batch (no-op when the loop never left it)
dmmv_status batched_compact_end(Ctx* c) {
    if (!c->cmp_on) return DMMV_OK;
    dmmv_status st = c->p.dtype == DMMV_F64 ? compact_scatter_t<double>(c) : compact_scatter_t<float>(c);
    compact_to_full(c);
    return st;
}

// row-major copy of a column-major matrix alone (a dense single instance that uses the batch's
// pruned descent needs nothing else of the batched layouts)
dmmv_status batched_build_xt(Ctx* c) {
    if (c->p.dtype == DMMV_F64)
        launch_transpose<double>(c->stream, (const double*)c->p.A_dense, c->p.n, c->p.m, c->p.lda, (double*)c->Xt, c->p.n);
    else
        launch_transpose<float>(c->stream, (const float*)c->p.A_dense, c->p.n, c->p.m, c->p.lda, (float*)c->Xt, c->p.n);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

dmmv_status batched_build(Ctx* c) {
    if (c->eval_mfma) DMMV_TRY(batched_eval_mfma_build(c));
    if (c->use_lists) DMMV_TRY(batched_lists_prepare(c));
    return c->p.dtype == DMMV_F64 ? build_t<double>(c) : build_t<float>(c);
}
dmmv_status batched_residual(Ctx* c) { return c->p.dtype == DMMV_F64 ? residual_t<double>(c) : residual_t<float>(c); }
dmmv_status batched_maxabs(Ctx* c) { return c->p.dtype == DMMV_F64 ? maxabs_t<double>(c) : maxabs_t<float>(c); }
dmmv_status batched_eval(Ctx* c, void* s, bool p) {
    if (c->eval_mfma) return batched_eval_mfma(c, s, p);
    if (c->use_lists) DMMV_TRY(batched_lists_first_use(c));
    if (batched_lists_in_use(c)) return batched_eval_lists(c, s, p);
    return c->p.dtype == DMMV_F64 ? eval_t<double>(c, s, p) : eval_t<float>(c, s, p);
}
dmmv_status batched_apply(Ctx* c, bool tf, int32_t iters, dmmv_move* trace, void* trace_t) {
    return c->p.dtype == DMMV_F64 ? apply_t<double>(c, tf, iters, trace, trace_t) : apply_t<float>(c, tf, iters, trace, trace_t);
}
dmmv_status batched_set_x(Ctx* c, const void* x) { return c->p.dtype == DMMV_F64 ? set_x_t<double>(c, x) : set_x_t<float>(c, x); }
dmmv_status batched_get_x_from(Ctx* c, const int32_t* kidx, void* x) {
    if (c->p.n * c->p.R == 0) return DMMV_OK;
    return c->p.dtype == DMMV_F64 ? get_x_t<double>(c, kidx, x) : get_x_t<float>(c, kidx, x);
}
dmmv_status batched_get_x(Ctx* c, void* x) { return batched_get_x_from(c, c->kidx, x); }
dmmv_status batched_set_r(Ctx* c, const void* r) {
    // caller layout [R][m] -> internal [m][R]
    if (c->p.dtype == DMMV_F64) launch_transpose<double>(c->stream, (const double*)r, c->p.R, c->p.m, c->p.m, (double*)c->r, c->p.R);
    else launch_transpose<float>(c->stream, (const float*)r, c->p.R, c->p.m, c->p.m, (float*)c->r, c->p.R);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}
dmmv_status batched_get_r(Ctx* c, void* r) {
    if (c->p.dtype == DMMV_F64) launch_transpose<double>(c->stream, (const double*)c->r, c->p.m, c->p.R, c->p.R, (double*)r, c->p.m);
    else launch_transpose<float>(c->stream, (const float*)c->r, c->p.m, c->p.R, c->p.R, (float*)r, c->p.m);
    DMMV_LAUNCH_CHECK();
    return DMMV_OK;
}

}  // namespace dmmv
