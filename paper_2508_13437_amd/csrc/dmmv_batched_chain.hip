// Batched residual in sequential order on the matrix cores (fp32).
//
// The contract fixes r_iq = fma(acc, s_q, -b_iq) with acc = fma(X_ij, D[k_jq], acc) for j ascending.
// v_mfma_f32_*x1 has K = 1: one instruction adds ONE column's rank-1 term to a tile, one fused
// multiply-add per element rounded once, so issuing it once per column in ascending order IS that
// chain (the l2 changes use the same form).  The matrix cores do it at twice the rate at which the
// vector unit issues v_fma_f32, and an operand is read once per 64 x 16 .. 128 x 64 outputs
// instead of once per 32.
//
// The codes' values V[j][q] = D[k_jq] are written first (n R w bytes, a streaming pass, 2 % of the
// product's time): vector instructions do not overlap with the matrix cores', so a look-up inside the loop would
// add its issue time to every column.  The loop itself holds no vector instruction: raw buffer loads
// (descriptor + scalar column offset + constant lane offset), two operand register sets taking
// turns.  max |r| per instance comes out of the same launch (integer maximum of the bit patterns,
// order-free).
#include "dmmv_common.h"

namespace dmmv {

namespace {

typedef __attribute__((__vector_size__(32 * sizeof(float)))) float floatx32;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

// V[e] = D[kidx[e]]; also clears the maxima that the product raises
__global__ __launch_bounds__(256) void k_chain_values(int64_t total, int64_t R, int32_t nd, const float* __restrict__ D,
                                                      const int32_t* __restrict__ kidx, float* __restrict__ V,
                                                      InstState<float>* __restrict__ st) {
    extern __shared__ float shD[];
    for (int k = threadIdx.x; k < nd; k += blockDim.x) shD[k] = D[k];
    __syncthreads();
    const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = t0; q < R; q += stride) st[q].t = 0.0f;
    for (int64_t e = t0; e < total; e += stride) V[e] = shD[kidx[e]];
}

// One tile shape of the K = 1 matrix instruction.
struct Mfma32 {                                   // 64 rows x 32 instances, two blocks of 32 x 32
    typedef floatx32 acc_t;
    static constexpr int NV = 32, COLS = 32;
    static __device__ __forceinline__ acc_t mul(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_32x32x1f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int v, int lane) { return 32 * (v / 16) + 8 * ((v % 16) / 4) + 4 * (lane >> 5) + v % 4; }
};
struct Mfma16 {                                   // 64 rows x 16 instances, four blocks of 16 x 16
    typedef floatx16 acc_t;
    static constexpr int NV = 16, COLS = 16;
    static __device__ __forceinline__ acc_t mul(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x1f32(a, b, c, 0, 0, 0); }
    static __device__ __forceinline__ int row(int v, int lane) { return 16 * (v / 4) + 4 * (lane >> 4) + v % 4; }
};

// A wavefront owns TA x TB tiles of M; a workgroup holds WA x WB wavefronts.  U columns' operands are
// requested while the U columns before them are multiplied.
template <class M, int TA, int TB, int WA, int WB, int U>
__global__ __launch_bounds__(64 * WA * WB) void k_residual_chain(
    int64_t m, int64_t n, int64_t R, const float* __restrict__ X, int64_t ldx, const float* __restrict__ V,
    const float* __restrict__ scale, const float* __restrict__ Bt, float* __restrict__ r, InstState<float>* __restrict__ st) {
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int64_t i0 = (blockIdx.x * (int64_t)WA + w % WA) * (64 * TA);
    const int64_t q0 = (blockIdx.y * (int64_t)WB + w / WA) * (M::COLS * TB);
    if (i0 >= m || q0 >= R) return;                         // whole wavefronts only
    // byte offsets inside X and V fit 32 bits (checked on the host); lanes past an edge repeat the last element
    uint32_t oa[TA], ob[TB];
#pragma unroll
    for (int a = 0; a < TA; ++a) { const int64_t i = i0 + 64 * a + lane; oa[a] = 4u * (uint32_t)(i < m ? i : m - 1); }
#pragma unroll
    for (int b = 0; b < TB; ++b) { const int64_t q = q0 + M::COLS * b + lane % M::COLS; ob[b] = 4u * (uint32_t)(q < R ? q : R - 1); }
    typename M::acc_t c[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < M::NV; ++v) c[a][b][v] = 0.0f;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, (int)(uint32_t)((ldx * (n - 1) + m) * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_v = __builtin_amdgcn_make_buffer_rsrc((void*)V, 0, (int)(uint32_t)(n * R * 4), 0x00020000);
    const uint32_t xstride = (uint32_t)ldx * 4u, vstride = (uint32_t)R * 4u;
    const int32_t cols = (int32_t)n;
    float pa[TA][U], pb[TB][U], sa[TA][U], sb[TB][U];       // the two operand sets
    auto load = [&](float (&A)[TA][U], float (&B)[TB][U], int32_t j0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t j = (uint32_t)(j0 + u < cols ? j0 + u : cols - 1);
#pragma unroll
            for (int a = 0; a < TA; ++a) A[a][u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_x, (int)oa[a], (int)(j * xstride), 0));
#pragma unroll
            for (int b = 0; b < TB; ++b) B[b][u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_v, (int)ob[b], (int)(j * vstride), 0));
        }
    };
    auto step = [&](const float (&A)[TA][U], const float (&B)[TB][U], int u) {
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b) c[a][b] = M::mul(A[a][u], B[b][u], c[a][b]);
    };
    // whole pairs of sets without a test per column, then the columns that are left
    load(pa, pb, 0);
    int32_t j0 = 0;
    for (; j0 + 2 * U <= cols; j0 += 2 * U) {
        load(sa, sb, j0 + U);
#pragma unroll
        for (int u = 0; u < U; ++u) step(pa, pb, u);
        load(pa, pb, j0 + 2 * U);                           // past the end: repeats of the last column, not used
#pragma unroll
        for (int u = 0; u < U; ++u) step(sa, sb, u);
    }
    if (j0 + U < cols) load(sa, sb, j0 + U);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (j0 + u < cols) step(pa, pb, u);                 // uniform
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (j0 + U + u < cols) step(sa, sb, u);
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        const int64_t q = q0 + M::COLS * b + lane % M::COLS;
        const int64_t qc = q < R ? q : R - 1;
        const float sc = scale[qc];
        float t = 0.0f;
#pragma unroll
        for (int a = 0; a < TA; ++a) {
            float bt[M::NV];
#pragma unroll
            for (int v = 0; v < M::NV; ++v) {
                const int64_t i = i0 + 64 * a + M::row(v, lane);
                bt[v] = Bt[(i < m ? i : m - 1) * R + qc];
            }
#pragma unroll
            for (int v = 0; v < M::NV; ++v) {
                const int64_t i = i0 + 64 * a + M::row(v, lane);
                const float y = dmmv_fma(c[a][b][v], sc, -bt[v]);
                if (i < m && q < R) { r[i * R + q] = y; t = dmmv_max(t, dmmv_abs(y)); }
            }
        }
        // lanes that share an instance first, then one integer maximum per instance and wavefront
        for (int off = M::COLS; off < 64; off <<= 1) t = dmmv_max(t, __shfl_xor(t, off, 64));
        if (lane < M::COLS && q < R) atomicMax(reinterpret_cast<int*>(&st[q].t), __float_as_int(t));
    }
}

}  // namespace

bool batched_chain_applicable(const Ctx* c) {
    const int64_t lim = (int64_t)1 << 32;
    return c->kind == KIND_BATCHED && c->p.dtype == DMMV_F32 && !c->cmp_on && c->p.m > 0 && c->p.n > 0 &&
           c->p.R <= 65535 * 16 &&   // the grid's second dimension, at the smallest tile's 16 instances
           (c->p.lda * (c->p.n - 1) + c->p.m) * 4 < lim && c->p.n * c->p.R * 4 < lim;
}

dmmv_status batched_chain_residual(Ctx* c) {
    const int64_t m = c->p.m, n = c->p.n, R = c->p.R;
    // the buffer of the descent's packed level indices is free outside a descent's loop and has V's size
    float* V = reinterpret_cast<float*>(c->cmp_kidx);
    InstState<float>* st = (InstState<float>*)c->state;
    const int64_t vb = ceil_div(n * R, 1024);
    hipLaunchKernelGGL(k_chain_values, dim3((unsigned)(vb < 4096 ? vb : 4096)), dim3(256), (size_t)c->p.nd * sizeof(float), c->stream,
                       n * R, R, c->p.nd, (const float*)c->D_dev, (const int32_t*)c->kidx, V, st);
    DMMV_LAUNCH_CHECK();
    auto launch = [&](auto kernel, int64_t rows, int64_t insts, int threads) -> dmmv_status {
        hipLaunchKernelGGL(kernel, dim3((unsigned)ceil_div(m, rows), (unsigned)ceil_div(R, insts)), dim3(threads), 0, c->stream,
                           m, n, R, (const float*)c->p.A_dense, c->p.lda, (const float*)V, (const float*)c->scale_dev,
                           (const float*)c->Bt, (float*)c->r, st);
        DMMV_LAUNCH_CHECK();
        return DMMV_OK;
    };
    // The tile: an instruction's time per column is fixed, so a launch takes (columns) x (rounds of
    // workgroups over 256 compute units) x (a wavefront's time per column).  Measured on n = 4096, ns per
    // column and round: 128 x 64 per wavefront 123 (one workgroup per compute unit), 64 x 32 36 (45 when
    // a SIMD has one wavefront only), 64 x 16 31; small launches, 64 x 16 with one wavefront per
    // workgroup 23.  Total at R = 128 / 500 / 1024 / 4096 of m = 2048: 94 / 138 / 189 / 545 us with the tile
    // taken, against 498 / 504 / 506 / 545 with the largest tile and 1610 / 1610 / 1744 / 2206 on the vector unit.
    const int64_t few = ceil_div(m, 64) * ceil_div(R, 16);
    if (few <= 512) return launch(k_residual_chain<Mfma16, 1, 1, 1, 1, 24>, 64, 16, 64);
    auto rounds = [&](int64_t rows, int64_t insts) { return ceil_div(ceil_div(m, rows) * ceil_div(R, insts), 256); };
    const int64_t t16 = 31 * rounds(128, 32), t64 = 123 * rounds(256, 128);
    int64_t t32 = 36 * rounds(128, 64);
    if (t32 < 45) t32 = 45;
    if (t16 <= t32 && t16 <= t64) return launch(k_residual_chain<Mfma16, 1, 1, 2, 2, 24>, 128, 32, 256);
    if (t32 <= t64) return launch(k_residual_chain<Mfma32, 1, 1, 2, 2, 16>, 128, 64, 256);
    return launch(k_residual_chain<Mfma32, 2, 2, 2, 2, 6>, 256, 128, 256);
}

}  // namespace dmmv
