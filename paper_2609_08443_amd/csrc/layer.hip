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
// l % 32, and k = 8 q + 4 (l / 32) + i at step 4 q + i.  The products are small (64 to
// 1024 rows, 64 to 256 columns and k), so the operands go from L2 straight to
// registers, several steps ahead.  KSPLIT = 4: the workgroup's four waves share one
// 32 x 32 tile, each a quarter of k, and add up through LDS in wave order (the few
// tiles of a per-head product, whose time is one wave's chain of loads and
// instructions); KSPLIT = 1: a 64 x 64 tile, 32 x 32 a wave.  Measured (VALU product
// before -> now): M = 1024, d = 128, H = 1, 18-26 -> 4.9 us (about the floor of a launch);
// dW of M = 256, d = 64, H = 2, 18 -> 5.1 us.
template <typename TA, typename TB, typename TC, bool AK, bool BK, int KSPLIT>
__global__ __launch_bounds__(256) void small_gemm_kernel(const TA* __restrict__ A, int64_t a_h, int64_t a_r,
                                                         int64_t a_k, const TB* __restrict__ Bm, int64_t b_h,
                                                         int64_t b_k, int64_t b_c, int32_t b_mod,
                                                         TC* __restrict__ C, int64_t c_h, int64_t c_r, int32_t R,
                                                         int32_t N, int32_t Kd, float alpha, bool accumulate) {
    using tile::f32x16;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l32 = lane & 31, hl = lane >> 5;
    const int r0 = KSPLIT == 1 ? blockIdx.x * 64 + 32 * (w >> 1) : blockIdx.x * 32;
    const int c0 = KSPLIT == 1 ? blockIdx.y * 64 + 32 * (w & 1) : blockIdx.y * 32;
    const int64_t z = blockIdx.z;
    // rows and columns past the edge repeat the last one and are not stored
    const TA* Ap = A + z * a_h + (int64_t)min(r0 + l32, R - 1) * a_r;
    const TB* Bp = Bm + (z % b_mod) * b_h + (int64_t)min(c0 + l32, N - 1) * b_c;
    f32x16 acc = {};
    auto add = [&](const float4& x, const float4& y) __attribute__((always_inline)) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, y.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, y.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, y.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, y.w, acc, 0, 0, 0);
    };
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
        for (int i = 0; i < GROUP; ++i) add(x[i], y[i]);
    }
    for (; q < nq; q += KSPLIT) add(load_k4<TA, AK>(Ap, a_k, 8 * q + 4 * hl), load_k4<TB, BK>(Bp, b_k, 8 * q + 4 * hl));
    if (q == nq && 8 * nq < Kd)   // (one wave reaches nq)
        add(load_k4_tail(Ap, a_k, 8 * nq + 4 * hl, Kd), load_k4_tail(Bp, b_k, 8 * nq + 4 * hl, Kd));
    TC* Cz = C + z * c_h;
    auto put = [&](int r, int ln, float v) __attribute__((always_inline)) {
        const int row = r0 + tile::srow(r, ln >> 5), col = c0 + (ln & 31);
        if (row >= R || col >= N) return;
        const int64_t o = (int64_t)row * c_r + col;
        v *= alpha;
        store_el(Cz, o, accumulate ? v + load_el(Cz, o) : v);
    };
    if constexpr (KSPLIT == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) put(r, lane, acc[r]);
    } else {
        __shared__ float part[4][16][64];
#pragma unroll
        for (int r = 0; r < 16; ++r) part[w][r][lane] = acc[r];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * w + i;
            put(r, lane, (part[0][r][lane] + part[1][r][lane]) + (part[2][r][lane] + part[3][r][lane]));
        }
    }
}

template <typename TA, typename TB, typename TC, bool AK, bool BK>
hipError_t gemm_k(const MatView& a, const MatView& b, int32_t b_mod, void* c, int64_t c_h, int64_t c_r, int32_t H,
                  int32_t R, int32_t N, int32_t Kd, float alpha, bool accumulate, hipStream_t stream) {
    // 64 x 64 tiles where they give every CU two workgroups
    const int64_t big = (int64_t)((R + 63) / 64) * ((N + 63) / 64) * H;
    const bool split = big < 2 * (int64_t)device_cus();
    const int t = split ? 32 : 64;
    const dim3 grid((unsigned)((R + t - 1) / t), (unsigned)((N + t - 1) / t), (unsigned)H);
    auto kern = split ? small_gemm_kernel<TA, TB, TC, AK, BK, 4> : small_gemm_kernel<TA, TB, TC, AK, BK, 1>;
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
    const bool ak = k_vectors(a.p, sizeof(TA), a.s_1, a.s_0, a.s_h, Kd);
    const bool bk = k_vectors(b.p, sizeof(TB), b.s_0, b.s_1, b.s_h, Kd);
#define SA_K(X, Y) gemm_k<TA, TB, TC, X, Y>(a, b, b_mod, c, c_h, c_r, H, R, N, Kd, alpha, accumulate, stream)
    if (ak) return bk ? SA_K(true, true) : SA_K(true, false);
    return bk ? SA_K(false, true) : SA_K(false, false);
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
