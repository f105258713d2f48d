// Projections of the SA layer (Appendix G.3: Q = P W_Q, K = X W_K, the history X
// itself aggregated) around the sketching kernels.
//
// The key projection is absorbed into the prototype side:
//
//   S = scale (P W_Q)(X W_K)^T = scale (P W_Q W_K^T) X^T = scale P' X^T,
//
// the reordering the paper applies to single-query STCA (Appendix G.2), so the
// per-token work is the sketching step with K = V = X and prototypes P'.  X is
// read once, no [T, d] key tensor exists, and the only added work is per head:
// two [M, d] x [d, d] products forward and four backward:
//
//   dW_K = dP'^T Q,   dQ = dP' W_K,   dW_Q = P^T dQ,   dP = dQ W_Q^T
//
// (P' = Q W_K^T, Q = P W_Q), with dP' the prototype gradient of the sketching
// backward and dX = dV + scale dS P' from its token side.
//
// This file holds the small batched product used for those six [M|d] x d
// matrices (fp32 accumulation, strided operands so that transposes are free).
#include <type_traits>

#include "sa_internal.h"
#include "tile_ops.h"

namespace sa {

namespace {

template <typename T>
__device__ inline float load_el(const T* p, int64_t i);
template <>
__device__ inline float load_el<float>(const float* p, int64_t i) { return p[i]; }
template <>
__device__ inline float load_el<uint16_t>(const uint16_t* p, int64_t i) {
    return __uint_as_float((uint32_t)p[i] << 16);
}

template <typename T>
__device__ inline void store_el(T* p, int64_t i, float v);
template <>
__device__ inline void store_el<float>(float* p, int64_t i, float v) { p[i] = v; }
template <>
__device__ inline void store_el<uint16_t>(uint16_t* p, int64_t i, float v) { p[i] = tile::to_bf16(v); }

// One operand of the product: four consecutive k of a row (column) as fp32.  With KC
// the k index is contiguous and the four come in one load (strides and base allow
// it), else one by one (lanes along the other index, which then coalesces).
template <typename T, bool KC>
__device__ inline float4 load_k4(const T* p, int64_t s_k, int k) {
    if constexpr (!KC)
        return make_float4(load_el(p, k * s_k), load_el(p, (k + 1) * s_k), load_el(p, (k + 2) * s_k), load_el(p, (k + 3) * s_k));
    else if constexpr (sizeof(T) == 4)
        return *reinterpret_cast<const float4*>(p + k);
    else {
        const uint2 v = *reinterpret_cast<const uint2*>(p + k);
        return make_float4(tile::bf16_lo(v.x), tile::bf16_hi(v.x), tile::bf16_lo(v.y), tile::bf16_hi(v.y));
    }
}
// the same where k may pass the end: zeros there
template <typename T>
__device__ inline float4 load_k4_tail(const T* p, int64_t s_k, int k, int32_t Kd) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = k + i < Kd ? load_el(p, (k + i) * s_k) : 0.f;
    return make_float4(v[0], v[1], v[2], v[3]);
}

// C[z][r][c] = alpha sum_k A[z](r, k) B[z % b_mod](k, c) (+ C with accumulate) for
// r < R, c < N, k < Kd, on the fp32 matrix cores, with A(r, k) = A[z a_h + r a_r + k a_k],
// B(k, c) = B[z' b_h + k b_k + c b_c], C[z c_h + r c_r + c].  A wave's instruction
// 32x32x2 takes one fp32 value per operand and lane: lane l holds row (column)
// l % 32, and k = 8 q + 4 (l / 32) + i at step 4 q + i.
template <typename TC>
__device__ inline void store_el32(TC* C, int64_t c_r, int row0, int col, int r, int ln, int32_t R, int32_t N, float v,
                                  float alpha, bool accumulate) {
    const int row = row0 + tile::srow(r, ln >> 5);
    if (row >= R || col >= N) return;
    const int64_t o = (int64_t)row * c_r + col;
    v *= alpha;
    store_el(C, o, accumulate ? v + load_el(C, o) : v);
}
__device__ inline void mfma_k4(tile::f32x16& acc, const float4& x, const float4& y) {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, acc, 0, 0, 0);
}

// The operands straight from L2 to registers, several steps ahead.  KSPLIT = 4: few
// tiles (64 to 1024 rows, 64 to 256 columns and k of one head), where the time is one
// wave's chain of loads and instructions: the workgroup's four waves share one 32 x 32
// tile, each a quarter of k, and add up through LDS in wave order.  KSPLIT = 1: a
// 64 x 64 tile, 32 x 32 a wave.  Measured (VALU product before -> now): M = 1024, d = 128,
// H = 1, 18-26 -> 4.9 us (about the floor of a launch); dW of M = 256, d = 64, H = 2,
// 18 -> 5.1 us.
template <typename TA, typename TB, typename TC, bool AK, bool BK, int KSPLIT>
__global__ __launch_bounds__(256) void small_gemm_kernel(const TA* __restrict__ A, int64_t a_h, int64_t a_r,
                                                         int64_t a_k, const TB* __restrict__ Bm, int64_t b_h,
                                                         int64_t b_k, int64_t b_c, int32_t b_mod,
                                                         TC* __restrict__ C, int64_t c_h, int64_t c_r, int32_t R,
                                                         int32_t N, int32_t Kd, float alpha, bool accumulate) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l32 = lane & 31, hl = lane >> 5;
    const int r0 = KSPLIT == 1 ? blockIdx.x * 64 + 32 * (w >> 1) : blockIdx.x * 32;
    const int c0 = KSPLIT == 1 ? blockIdx.y * 64 + 32 * (w & 1) : blockIdx.y * 32;
    const int64_t z = blockIdx.z;
    // rows and columns past the edge repeat the last one and are not stored
    const TA* Ap = A + z * a_h + (int64_t)min(r0 + l32, R - 1) * a_r;
    const TB* Bp = Bm + (z % b_mod) * b_h + (int64_t)min(c0 + l32, N - 1) * b_c;
    tile::f32x16 acc = {};
    // whole groups of eight k, GROUP of them loaded at a time; then the rest of k
    constexpr int GROUP = 4;
    const int nq = Kd / 8;
    int q = KSPLIT == 1 ? 0 : w;
    for (; q + (GROUP - 1) * KSPLIT < nq; q += GROUP * KSPLIT) {
        float4 x[GROUP], y[GROUP];
#pragma unroll
        for (int i = 0; i < GROUP; ++i) {
            x[i] = load_k4<TA, AK>(Ap, a_k, 8 * (q + i * KSPLIT) + 4 * hl);
            y[i] = load_k4<TB, BK>(Bp, b_k, 8 * (q + i * KSPLIT) + 4 * hl);
        }
#pragma unroll
        for (int i = 0; i < GROUP; ++i) mfma_k4(acc, x[i], y[i]);
    }
    for (; q < nq; q += KSPLIT)
        mfma_k4(acc, load_k4<TA, AK>(Ap, a_k, 8 * q + 4 * hl), load_k4<TB, BK>(Bp, b_k, 8 * q + 4 * hl));
    if (q == nq && 8 * nq < Kd)   // (one wave reaches nq)
        mfma_k4(acc, load_k4_tail(Ap, a_k, 8 * nq + 4 * hl, Kd), load_k4_tail(Bp, b_k, 8 * nq + 4 * hl, Kd));
    TC* Cz = C + z * c_h;
    if constexpr (KSPLIT == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) store_el32(Cz, c_r, r0, c0 + l32, r, lane, R, N, acc[r], alpha, accumulate);
    } else {
        __shared__ float part[4][16][64];
#pragma unroll
        for (int r = 0; r < 16; ++r) part[w][r][lane] = acc[r];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * w + i;
            store_el32(Cz, c_r, r0, c0 + l32, r, lane, R, N,
                       (part[0][r][lane] + part[1][r][lane]) + (part[2][r][lane] + part[3][r][lane]), alpha, accumulate);
        }
    }
}

// Many tiles whose operands do not come in vectors of k: 64 x 64 a workgroup, 32 x 32 a
// wave, slabs of 32 k through LDS, the next in registers.  Read from global memory along
// whichever index is contiguous and kept [row][k] in LDS (36 floats a row: 16-byte
// accesses of eight consecutive rows touch all banks once), so that strides and
// remainders of k cost nothing: from L2, one value a lane and instruction, the matrix
// cores wait for loads.  Measured (us; the VALU product before, from L2, through LDS; bf16
// operands): 512 x 1024 x 160 in 32 batches, k strided, 109, 143, 74; 160 x 500 x 1030 in
// 32, k contiguous, 208, 334, 86.  With A in vectors of k from L2 stays ahead: 512 x 1024
// x 160 in 32, B in vectors too 61 against 73, B strided 70 against 73; 512 x 512 x 40 in 64
// 23 and 26 against 37 and 42.
template <typename TA, typename TB, typename TC, bool AK, bool BK>
__global__ __launch_bounds__(256) void tiled_gemm_kernel(const TA* __restrict__ A, int64_t a_h, int64_t a_r,
                                                         int64_t a_k, const TB* __restrict__ Bm, int64_t b_h,
                                                         int64_t b_k, int64_t b_c, int32_t b_mod,
                                                         TC* __restrict__ C, int64_t c_h, int64_t c_r, int32_t R,
                                                         int32_t N, int32_t Kd, float alpha, bool accumulate) {
    constexpr int KC = 32, LD = KC + 4;
    __shared__ __attribute__((aligned(16))) float slab[2][2][64 * LD];   // [buffer][operand]
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hl = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // k offsets of strided operands in scalar registers
    const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
    const int64_t z = blockIdx.z;
    const TA* Ap = A + z * a_h;
    const TB* Bp = Bm + (z % b_mod) * b_h;
    // Eight values of a slab a thread: lanes along k (KCONT), one k of eight rows; else
    // lanes along the rows, two runs of four k of one row.  Rows past the edge repeat
    // the last one, k past the end is 0.
    auto row_of = [&](bool kcont, int i) { return kcont ? tid / 32 + 8 * i : lane; };
    auto k_of = [&](bool kcont, int i) { return kcont ? tid % 32 : 16 * (i / 4) + 4 * w + i % 4; };
    const TA* pa[AK ? 8 : 1];
    const TB* pb[BK ? 8 : 1];
#pragma unroll
    for (int i = 0; i < (AK ? 8 : 1); ++i) pa[i] = Ap + (int64_t)min(r0 + row_of(AK, i), R - 1) * a_r + k_of(AK, 0) * a_k;
#pragma unroll
    for (int i = 0; i < (BK ? 8 : 1); ++i) pb[i] = Bp + (int64_t)min(c0 + row_of(BK, i), N - 1) * b_c + k_of(BK, 0) * b_k;
    float va[8], vb[8];
    auto fetch = [&](int k0, auto tail) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int ka = k_of(AK, i), kb = k_of(BK, i);
            va[i] = !tail.value || k0 + ka < Kd ? load_el(pa[AK ? i : 0] + (k0 + ka - k_of(AK, 0)) * a_k, 0) : 0.f;
            vb[i] = !tail.value || k0 + kb < Kd ? load_el(pb[BK ? i : 0] + (k0 + kb - k_of(BK, 0)) * b_k, 0) : 0.f;
        }
    };
    auto fetch_slab = [&](int k0) __attribute__((always_inline)) {
        if (k0 + KC <= Kd) fetch(k0, std::false_type{});
        else fetch(k0, std::true_type{});
    };
    auto store = [&](float* t, auto kcont, const float (&v)[8]) __attribute__((always_inline)) {
        if constexpr (kcont.value) {
#pragma unroll
            for (int i = 0; i < 8; ++i) t[(tid / 32 + 8 * i) * LD + tid % 32] = v[i];
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i)
                *reinterpret_cast<float4*>(t + lane * LD + 16 * i + 4 * w) =
                    make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
        }
    };
    using ak = std::integral_constant<bool, AK>;
    using bk = std::integral_constant<bool, BK>;
    const int wr = 32 * (w >> 1), wc = 32 * (w & 1);
    tile::f32x16 acc = {};
    if (Kd > 0) {
        fetch_slab(0);
        store(slab[0][0], ak{}, va);
        store(slab[0][1], bk{}, vb);
    }
    __syncthreads();
    for (int k0 = 0, buf = 0; k0 < Kd; k0 += KC, buf ^= 1) {
        const bool more = k0 + KC < Kd;
        if (more) fetch_slab(k0 + KC);
#pragma unroll
        for (int q = 0; q < KC / 8; ++q)
            mfma_k4(acc, *reinterpret_cast<const float4*>(&slab[buf][0][(wr + l32) * LD + 8 * q + 4 * hl]),
                    *reinterpret_cast<const float4*>(&slab[buf][1][(wc + l32) * LD + 8 * q + 4 * hl]));
        if (more) {
            store(slab[buf ^ 1][0], ak{}, va);
            store(slab[buf ^ 1][1], bk{}, vb);
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 16; ++r)
        store_el32(C + z * c_h, c_r, r0 + wr, c0 + wc + l32, r, lane, R, N, acc[r], alpha, accumulate);
}

enum GemmKind { kSplitK, kDirect, kTiled };

template <typename TA, typename TB, typename TC, bool AK, bool BK, GemmKind KIND>
hipError_t gemm_k(const MatView& a, const MatView& b, int32_t b_mod, void* c, int64_t c_h, int64_t c_r, int32_t H,
                  int32_t R, int32_t N, int32_t Kd, float alpha, bool accumulate, hipStream_t stream) {
    const int t = KIND == kSplitK ? 32 : 64;
    const dim3 grid((unsigned)((R + t - 1) / t), (unsigned)((N + t - 1) / t), (unsigned)H);
    const auto kern = [] {
        if constexpr (KIND == kTiled) return tiled_gemm_kernel<TA, TB, TC, AK, BK>;
        else return small_gemm_kernel<TA, TB, TC, AK, BK, KIND == kSplitK ? 4 : 1>;
    }();
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, reinterpret_cast<const TA*>(a.p), a.s_h, a.s_0, a.s_1,
                       reinterpret_cast<const TB*>(b.p), b.s_h, b.s_0, b.s_1, b_mod, reinterpret_cast<TC*>(c), c_h, c_r,
                       R, N, Kd, alpha, accumulate);
    return hipGetLastError();
}

// whether four consecutive k of any row come in one aligned load: `row` and `batch`
// are the strides of the other index and of the batch
bool k_vectors(const void* p, size_t el, int64_t s_k, int64_t row, int64_t batch, int32_t Kd) {
    return s_k == 1 && row % 4 == 0 && batch % 4 == 0 && Kd % 4 == 0 && reinterpret_cast<uintptr_t>(p) % (4 * el) == 0;
}

template <typename TA, typename TB, typename TC>
hipError_t gemm_t(const MatView& a, const MatView& b, int32_t b_mod, void* c, int64_t c_h, int64_t c_r, int32_t H,
                  int32_t R, int32_t N, int32_t Kd, float alpha, bool accumulate, hipStream_t stream) {
#define SA_K(X, Y, KIND) gemm_k<TA, TB, TC, X, Y, KIND>(a, b, b_mod, c, c_h, c_r, H, R, N, Kd, alpha, accumulate, stream)
    const bool ak = k_vectors(a.p, sizeof(TA), a.s_1, a.s_0, a.s_h, Kd);
    const bool bk = k_vectors(b.p, sizeof(TB), b.s_0, b.s_1, b.s_h, Kd);
    // 64 x 64 tiles where they give every CU two workgroups
    const int64_t big = (int64_t)((R + 63) / 64) * ((N + 63) / 64) * H;
    if (big < 2 * (int64_t)device_cus()) {
        if (ak) return bk ? SA_K(true, true, kSplitK) : SA_K(true, false, kSplitK);
        return bk ? SA_K(false, true, kSplitK) : SA_K(false, false, kSplitK);
    }
    if (ak && bk) return SA_K(true, true, kDirect);
    if (ak && b.s_0 != 1) return SA_K(true, false, kDirect);
    if (a.s_1 == 1) return b.s_0 == 1 ? SA_K(true, true, kTiled) : SA_K(true, false, kTiled);
    return b.s_0 == 1 ? SA_K(false, true, kTiled) : SA_K(false, false, kTiled);
#undef SA_K
}

hipError_t small_gemm_dispatch(const MatView& a, const MatView& b, void* c, bool c_bf16, int64_t c_h, int64_t c_r,
                               int32_t H, int32_t R, int32_t N, int32_t Kd, int32_t b_mod, float alpha,
                               bool accumulate, hipStream_t stream) {
    if (H <= 0 || R <= 0 || N <= 0) return hipSuccess;
    if (H > 65535) return hipErrorInvalidValue;
#define SA_GEMM(TA, TB) \
    return c_bf16 ? gemm_t<TA, TB, uint16_t>(a, b, b_mod, c, c_h, c_r, H, R, N, Kd, alpha, accumulate, stream) \
                  : gemm_t<TA, TB, float>(a, b, b_mod, c, c_h, c_r, H, R, N, Kd, alpha, accumulate, stream)
    if (a.bf16 && b.bf16) SA_GEMM(uint16_t, uint16_t);
    if (a.bf16) SA_GEMM(uint16_t, float);
    if (b.bf16) SA_GEMM(float, uint16_t);
    SA_GEMM(float, float);
#undef SA_GEMM
}

}  // namespace

hipError_t launch_small_gemm(const MatView& a, const MatView& b, void* c, bool c_bf16, int32_t H, int32_t R,
                             int32_t N, int32_t Kd, hipStream_t stream, int32_t b_mod, bool accumulate) {
    if (b_mod <= 0) b_mod = H;
    return small_gemm_dispatch(a, b, c, c_bf16, (int64_t)R * N, N, H, R, N, Kd, b_mod, 1.0f, accumulate, stream);
}

hipError_t launch_small_gemm_general(const GemmDesc& d, hipStream_t stream) {
    return small_gemm_dispatch({d.A, d.a_bf16, d.a_z, d.a_m, d.a_k}, {d.B, d.b_bf16, d.b_z, d.b_k, d.b_n}, d.C,
                               d.c_bf16, d.c_z, d.c_m, d.batch, d.M, d.N, d.K, d.b_mod > 0 ? (int32_t)d.b_mod : d.batch,
                               d.alpha, d.accumulate, stream);
}

}  // namespace sa
