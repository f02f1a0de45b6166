// Batched products in sequential order on the matrix cores (fp32): the residual and G = X^T R_mat of the l2 changes.
//
// The contract fixes r_iq = fma(acc, s_q, -b_iq) with acc = fma(X_ij, D[k_jq], acc) for j ascending.
// v_mfma_f32_*x1 has K = 1: one instruction adds ONE column's rank-1 term to a tile, one fused
// multiply-add per element rounded once, so issuing it once per column in ascending order IS that
// chain.  The matrix cores do it at twice the rate at which the
// vector unit issues v_fma_f32, and an operand is read once per 64 x 16 .. 64 x 64 outputs
// instead of once per 32.
//
// The codes' values V[j][q] = D[k_jq] are written first (n R w bytes, a streaming pass, 2 % of the
// product's time): vector instructions do not overlap with the matrix cores', so a look-up inside the loop would
// add its issue time to every column.  The loop itself holds no vector instruction: raw buffer loads
// (descriptor + scalar column offset + constant lane offset), two operand register sets taking
// turns.  A wavefront issues one instruction at a time, so what stands between two products counts: one register
// holds the V operands of two or four columns, an address costs one scalar addition, and the loads are spread
// between the products.  max |r| per instance comes out of the same launch (integer maximum of the bit patterns,
// order-free).
//
// G_jq = acc with acc = fma(X_ij, r_iq, acc) for i ascending is the same product with the rows of X in the place
// of its columns and r in that of V: the same loop, another end.  (A kernel of its own with 128 x 64 per wavefront only took
// 0.64 ms on 4096 x 4096 with 1376 instances, whose 176 workgroups left a third of the chip idle, and 0.59 on 2048 x 4096
// with 4096; with the tile and the workgroups a compute unit of the rule below 0.38 and 0.54.)
#include <type_traits>

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

// f(0), f(1), .. f(N - 1) with the number as a constant
template <int N, int I = 0, class F>
__device__ __forceinline__ void each_column(const F& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>());
        each_column<N, I + 1>(f);
    }
}

// One tile shape of the K = 1 matrix instruction.  Its blocks of rows share the instances, so a register of 64 lanes
// holds the instances' values of COLUMNS columns, and the instruction reads the group of lanes it is told to (blgp).
struct Mfma32 {                                   // 64 rows x 32 instances, two blocks of 32 x 32
    typedef floatx32 acc_t;
    static constexpr int NV = 32, COLS = 32, COLUMNS = 2;
    template <int C>
    static __device__ __forceinline__ acc_t mul(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_32x32x1f32(a, b, c, 0, 0, 1 + C); }
    static __device__ __forceinline__ int row(int v, int lane) { return 32 * (v / 16) + 8 * ((v % 16) / 4) + 4 * (lane >> 5) + v % 4; }
};
struct Mfma16 {                                   // 64 rows x 16 instances, four blocks of 16 x 16
    typedef floatx16 acc_t;
    static constexpr int NV = 16, COLS = 16, COLUMNS = 4;
    template <int C>
    static __device__ __forceinline__ acc_t mul(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x1f32(a, b, c, 0, 0, 4 + C); }
    static __device__ __forceinline__ int row(int v, int lane) { return 16 * (v / 4) + 4 * (lane >> 4) + v % 4; }
};

// A wavefront owns TA x TB tiles of M; a workgroup holds WA x WB wavefronts.  U columns' operands are
// requested while the U columns before them are multiplied.
template <class M, int TA, int TB, int WA, int WB, int U, int PER, bool RES>
__global__ __launch_bounds__(64 * WA * WB, PER) void k_chain_product(
    int64_t m, int64_t n, int64_t R, const float* __restrict__ X, int64_t ldx, const float* __restrict__ V,
    const float* __restrict__ scale, const float* __restrict__ Bt, float* __restrict__ out, InstState<float>* __restrict__ st) {
    constexpr int G = M::COLUMNS, UB = U / G;
    static_assert(U % G == 0, "whole registers of instances' values");
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int64_t i0 = (blockIdx.x * (int64_t)WA + w % WA) * (64 * TA);
    const int64_t q0 = (blockIdx.y * (int64_t)WB + w / WA) * (M::COLS * TB);
    if (i0 >= m || q0 >= R) return;                         // whole wavefronts only
    // byte offsets inside X and V fit 32 bits (checked on the host); lanes past an edge repeat the last element
    const uint32_t xstride = (uint32_t)ldx * 4u, vstride = (uint32_t)R * 4u;
    const int32_t cols = (int32_t)n;
    uint32_t oa[TA], ob[TB], og[TB];                        // (ob: this lane's column of a group included)
#pragma unroll
    for (int a = 0; a < TA; ++a) { const int64_t i = i0 + 64 * a + lane; oa[a] = 4u * (uint32_t)(i < m ? i : m - 1); }
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        const int64_t q = q0 + M::COLS * b + lane % M::COLS;
        ob[b] = 4u * (uint32_t)(q < R ? q : R - 1);
        og[b] = ob[b] + (uint32_t)(lane / (64 / G)) * vstride;
    }
    typename M::acc_t c[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < M::NV; ++v) c[a][b][v] = 0.0f;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void*)X, 0, (int)(uint32_t)((ldx * (n - 1) + m) * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_v = __builtin_amdgcn_make_buffer_rsrc((void*)V, 0, (int)(uint32_t)(n * R * 4), 0x00020000);
    float pa[TA][U], pb[TB][UB], sa[TA][U], sb[TB][UB];     // the two operand sets
    auto get = [](const __amdgpu_buffer_rsrc_t& rs, uint32_t lane_off, uint32_t off) -> float {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)lane_off, (int)off, 0));
    };
    auto multiply = [&](const float (&A)[TA][U], const float (&B)[TB][UB], auto u) {
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b) c[a][b] = M::template mul<u.value % G>(A[a][u.value], B[b][u.value / G], c[a][b]);
    };
    // One set is multiplied while U columns from j0, all of them there, are requested into the other: a load takes one
    // addition on the scalar unit, and they go out between the products, whose time hides theirs.
    auto both = [&](const float (&A)[TA][U], const float (&B)[TB][UB], float (&An)[TA][U], float (&Bn)[TB][UB], int32_t j0) {
        uint32_t ox = (uint32_t)j0 * xstride, ov = (uint32_t)j0 * vstride;
        each_column<U>([&](auto u) {
#pragma unroll
            for (int a = 0; a < TA; ++a) An[a][u.value] = get(rs_x, oa[a], ox);
            ox += xstride;
            asm volatile("" : "+s"(ox));                    // (opaque, or the strides' multiples fill the scalar registers)
            if (u.value % G == 0) {
#pragma unroll
                for (int b = 0; b < TB; ++b) Bn[b][u.value / G] = get(rs_v, og[b], ov);
                ov += (uint32_t)G * vstride;
                asm volatile("" : "+s"(ov));
            }
            multiply(A, B, u);
            __builtin_amdgcn_sched_barrier(0);              // the order is as written: a set ahead, not a few loads
        });
    };
    // U columns from j0, of which some may be past the end: an operand of X is 0 there and one of V is -0, and their
    // product, -0, leaves every sum as it is.
    auto load = [&](float (&A)[TA][U], float (&B)[TB][UB], int32_t j0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool there = j0 + u < cols;
            const uint32_t j = (uint32_t)(there ? j0 + u : cols - 1);
#pragma unroll
            for (int a = 0; a < TA; ++a) {
                const float x = get(rs_x, oa[a], j * xstride);
                A[a][u] = there ? x : 0.0f;
            }
            if (u % G == 0) {
                const int32_t jl = j0 + u + lane / (64 / G);
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    const float x = get(rs_v, ob[b] + (uint32_t)(jl < cols ? jl : cols - 1) * vstride, 0);
                    B[b][u / G] = jl < cols ? x : -0.0f;
                }
            }
        }
    };
    load(pa, pb, 0);
    int32_t j0 = 0;                                         // first column of the set in pa, pb
    for (; j0 + 3 * U <= cols; j0 += 2 * U) {
        both(pa, pb, sa, sb, j0 + U);
        both(sa, sb, pa, pb, j0 + 2 * U);
    }
    for (; j0 < cols; j0 += 2 * U) {                        // under 3 U columns
        load(sa, sb, j0 + U);
        each_column<U>([&](auto u) { multiply(pa, pb, u); });
        if (j0 + U < cols) {
            load(pa, pb, j0 + 2 * U);
            each_column<U>([&](auto u) { multiply(sa, sb, u); });
        }
    }
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        const int64_t q = q0 + M::COLS * b + lane % M::COLS;
        const int64_t qc = q < R ? q : R - 1;
        if (!RES) {
#pragma unroll
            for (int a = 0; a < TA; ++a)
#pragma unroll
                for (int v = 0; v < M::NV; ++v) {
                    const int64_t i = i0 + 64 * a + M::row(v, lane);
                    if (i < m && q < R) out[i * R + q] = c[a][b][v];
                }
            continue;
        }
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
                if (i < m && q < R) { out[i * R + q] = y; t = dmmv_max(t, dmmv_abs(y)); }
            }
        }
        // lanes that share an instance first, then one integer maximum per instance and wavefront
        for (int off = M::COLS; off < 64; off <<= 1) t = dmmv_max(t, __shfl_xor(t, off, 64));
        if (lane < M::COLS && q < R) atomicMax(reinterpret_cast<int*>(&st[q].t), __float_as_int(t));
    }
}

}  // namespace

// out[m][R] = the product of X's n columns and V's n rows, by the tile that takes least
template <bool RES>
static dmmv_status chain_product(Ctx* c, int64_t m, int64_t n, const float* X, int64_t ldx, const float* V, float* out) {
    const int64_t R = c->p.R;
    auto launch = [&](auto kernel, int64_t rows, int64_t insts, int threads, size_t lds) -> dmmv_status {
        hipLaunchKernelGGL(kernel, dim3((unsigned)ceil_div(m, rows), (unsigned)ceil_div(R, insts)), dim3(threads), lds, c->stream,
                           m, n, R, X, ldx, V, (const float*)c->scale_dev,
                           (const float*)c->Bt, out, (InstState<float>*)c->state);
        DMMV_LAUNCH_CHECK();
        return DMMV_OK;
    };
    // The tile: an instruction's time per column is fixed, so a launch takes (columns) x (rounds of
    // workgroups over 256 compute units) x (a workgroup's time per column).  Measured on n = 4096, ns per
    // column and round: 64 x 16 per wavefront 20, 64 x 32 31 (27 are its product's), 64 x 64 59; small launches, 64 x 16 with one
    // wavefront per workgroup 18.  Total at R = 20 / 128 / 500 / 1024 / 4096 of m = 2048 (us): 73 / 78 / 96 / 146 / 512 with
    // the tile taken; before the operands of V shared their registers and the loads went out between the products
    // 95 / 98 / 147 / 201 / 578, and 1610 / 1610 / 1610 / 1744 / 2206 on the vector unit.
    // A chain of up to 256 columns ends before the deep request queues of the tiles below have paid for their start: 2048 x 64
    // with 500 instances 11.1 us by this one, 12.4 by the next; 4096 x 128 with 128 11.1 and 12.8.
    const int64_t few = ceil_div(m, 64) * ceil_div(R, 16);
    if (n <= 256 && few <= 1024) return launch(k_chain_product<Mfma16, 1, 1, 1, 1, 16, 1, RES>, 64, 16, 64, 0);
    if (few <= 512) return launch(k_chain_product<Mfma16, 1, 1, 1, 1, 48, 1, RES>, 64, 16, 64, 0);
    auto rounds = [&](int64_t rows, int64_t insts) { return ceil_div(ceil_div(m, rows) * ceil_div(R, insts), 256); };
    const int64_t t16 = 20 * rounds(64, 64), t32 = 31 * rounds(64, 128), t64 = 59 * rounds(128, 128);
    if (t16 <= t32 && t16 <= t64) return launch(k_chain_product<Mfma16, 1, 1, 1, 4, 32, 1, RES>, 64, 64, 256, 0);
    // The larger tiles ask for LDS that they do not use, for two workgroups a compute unit: where the registers let three
    // (G of the 64 x 64 tile) or five in, 1024 workgroups are 768 and then 256 of uneven distribution.  G of 2048 x 4096
    // with 4096 instances: 644 us with three, 497 with two (64 x 32: 553 with five, 504 with two).
    constexpr size_t TWO_PER_CU = 56 * 1024;
    if (t32 <= t64) return launch(k_chain_product<Mfma32, 1, 1, 1, 4, 16, 3, RES>, 64, 128, 256, TWO_PER_CU);
    return launch(k_chain_product<Mfma32, 1, 2, 2, 2, 16, 2, RES>, 128, 128, 256, TWO_PER_CU);
}

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
    return chain_product<true>(c, m, n, (const float*)c->p.A_dense, c->p.lda, V, (float*)c->r);
}

bool batched_chain_l2_applicable(const Ctx* c) {
    return c->kind == KIND_BATCHED && c->p.dtype == DMMV_F32 && c->p.m > 0 && c->p.m * c->p.n < (1ll << 30) &&
           c->p.m * c->p.R < (1ll << 30);          // 32-bit byte offsets
}

dmmv_status batched_chain_l2_g(Ctx* c) {
    return chain_product<false>(c, c->p.n, c->p.m, (const float*)c->Xt, c->p.n, (const float*)c->r, (float*)c->l2_g);
}

}  // namespace dmmv
