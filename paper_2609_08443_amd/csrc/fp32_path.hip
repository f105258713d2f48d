// Single-precision path of the SA sketching step on the fp32 matrix cores
// (v_mfma_f32_32x32x2_f32): fp32 inputs, forward and backward, and the backward of
// bf16 inputs for prototype counts the fused kernels have no instance for.  No value
// is rounded below fp32.
//
// Forward (section 3.1), two passes over the keys as in fwd_split.hip:
//   lse_f32_kernel      lse_t = log sum_m exp(scale <K_t, P_m>)
//   agg_f32_kernel      sketch_m += exp(scale <K_t, P_m> - lse_t) V_t
// (or in the second alone, when one workgroup holds all M <= 256 prototypes)
// Backward (chain rule; the MRLB sum over R targets, section 4.2, is done first):
//   bwd_token_f32_kernel, a block of 128 tokens against all prototypes, twice:
//     sweep 1: A = exp(scale S - lse), dV = A^T dY;  then D_t = <V_t, dV_t>
//     sweep 2: dS = A (V dY^T - D_t), dK = scale dS P
//   bwd_proto_f32_kernel, 32 prototypes a wave against a token range:
//     dP = scale sum_t dS K_t
//
// Matrix instruction 32x32x2: lane l gives row (column) l % 32 at k = l / 32, and
// the result has column l % 32, rows srow(r, l / 32) = 8 (r / 4) + 4 (l / 32) + r % 4
// in register r.  The k index of an operand may be any bijection as long as both
// operands use the same one:
//   * contractions over the d features take k = 8 q + 4 (l / 32) + i at step 4 q + i,
//     so a lane reads four consecutive features (16 bytes) at a time;
//   * contractions over a result tile's rows take row srow(r, l / 32) at step r, so
//     register r of the tile is the operand of step r as it stands.
// The features of a lane under the first rule are the rows of a result tile under
// srow, so <V_t, dV_t> needs no exchange between lanes but the final half-wave sum.
//
// An instruction takes 64 cycles for 4096 FLOPs; everything else (one 4-byte or a
// quarter of a 16-byte LDS read per instruction, the exponentials) hides beside it.
// Measured (fp32 VALU path before -> now): layer forward + backward on 9,619 tokens,
// H = 2, M = 256, d = 64, 1366 -> 195 us; one user of 2,048 tokens, M = 64, d = 64,
// forward, 44 -> 15 us (18 with a log-sum-exp pass of its own); distance from float64 the same or smaller on every output.
#include <algorithm>

#include "reduce_ops.h"
#include "sa_internal.h"
#include "segments.h"
#include "tile_ops.h"

namespace sa {

namespace {

using namespace tile;

constexpr float kLn2 = 0.6931471805599453f;
constexpr float kFloatMax = 3.4028234664e38f;

__device__ inline f32x16 mfma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ inline f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

// e^x to about one unit in the last place: 2^t for the rounded t = x / ln 2, corrected
// for t's rounding error and that of the constant
__device__ inline float exp_f32(float x) {
    constexpr float kLog2eLo = 1.9259629911e-8f;   // 1 / ln 2 - kLog2e
    const float t = x * kLog2e;
    float d = __builtin_fmaf(x, kLog2eLo, __builtin_fmaf(x, kLog2e, -t));
    if (!(__builtin_fabsf(x) < 1024.f)) d = 0.f;   // infinities and NaN: 2^t as it is
    const float e = __builtin_amdgcn_exp2f(t);
    return __builtin_fmaf(e, d * kLn2, e);
}

// four consecutive values at element i of an fp32 or bf16 tensor
template <bool BF16>
__device__ inline float4 load4(const void* p, int64_t i) {
    if constexpr (BF16) {
        const uint2 v = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(p) + i);
        return make_float4(bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y));
    } else {
        return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(p) + i);
    }
}

// D features of one row as the operand of D / 2 steps: register 4 q + i holds
// feature 8 q + 4 hl + i
template <bool BF16, int D>
__device__ inline void load_operand(const void* p, int64_t row0, int hl, float (&op)[D / 2]) {
#pragma unroll
    for (int q = 0; q < D / 8; ++q) {
        const float4 v = load4<BF16>(p, row0 + 8 * q + 4 * hl);
        op[4 * q] = v.x;
        op[4 * q + 1] = v.y;
        op[4 * q + 2] = v.z;
        op[4 * q + 3] = v.w;
    }
}

// LDS tiles: 32 rows of D + 4 floats (the padding spreads 16-byte reads of 32
// consecutive rows over the banks)
template <int D>
struct Tile32 {
    static constexpr int LD = D + 4;
    static constexpr int FLOATS = 32 * LD;
    // sum over the features of row (lane % 32) times the held operand, in two chains
    // (half the rounding steps of one, and no instruction waits for the one before)
    static __device__ inline f32x16 rows_dot(const float* t, int l32, int hl, const float (&op)[D / 2]) {
        f32x16 s0 = zero16(), s1 = zero16();
#pragma unroll
        for (int q = 0; q < D / 8; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(t + l32 * LD + 8 * q + 4 * hl);
            s0 = mfma(v.x, op[4 * q], s0);
            s1 = mfma(v.y, op[4 * q + 1], s1);
            s0 = mfma(v.z, op[4 * q + 2], s0);
            s1 = mfma(v.w, op[4 * q + 3], s1);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) s0[r] += s1[r];
        return s0;
    }
    // element (row srow(r, hl), column 32 jt + lane % 32)
    static __device__ inline float at(const float* t, int r, int l32, int hl, int jt) {
        return t[srow(r, hl) * LD + 32 * jt + l32];
    }
};

// one [32][D] tile, global -> registers -> LDS by THREADS threads; row(i) gives the
// element offset of tile row i in its tensor
template <bool BF16, int D, int THREADS>
struct TileLoad {
    static constexpr int CH = 32 * D / 4;                          // 4-value pieces
    static constexpr int N = (CH + THREADS - 1) / THREADS;
    float4 r[N];
    template <typename Row>
    __device__ inline void fetch(const void* p, int tid, Row row) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int idx = (tid + i * THREADS) % CH;
            r[i] = load4<BF16>(p, row(idx / (D / 4)) + (idx % (D / 4)) * 4);
        }
    }
    // rows from `rows` on are stored as zeros
    __device__ inline void store(float* t, int tid, int rows) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int idx = tid + i * THREADS;
            if (CH % THREADS == 0 || idx < CH) {
                const int row = idx / (D / 4);
                *reinterpret_cast<float4*>(t + row * Tile32<D>::LD + (idx % (D / 4)) * 4) =
                    row < rows ? r[i] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    }
};

// ---------------------------------------------------------------- forward: log-sum-exp
// Workgroup = 4 waves; WM of them hold the same 32 tokens as operands and take every
// WM-th tile of 32 prototypes.  WM = 1: the tiles stream through LDS one at a time,
// double-buffered; WM = 4: four at a time, a wave each.  The next are in registers.  A
// token's running maximum and sum live in one lane per half-wave and wave.
template <int D, int WM>
struct LseF32Cfg {
    static constexpr int TOKENS = 128 / WM;   // per workgroup
    static constexpr int BUFS = WM == 1 ? 2 : 1;
    static constexpr size_t LDS = (size_t)BUFS * WM * Tile32<D>::FLOATS * 4 + 4 * 32 * sizeof(float2);
};
template <int D, int WM>
__global__ __launch_bounds__(256) void lse_f32_kernel(const float* __restrict__ K, const float* __restrict__ P,
                                                      const int64_t* __restrict__ off, int64_t B, int64_t T,
                                                      int32_t H, int32_t M, float scale, bool p_user,
                                                      float* __restrict__ lse) {
    using TL = Tile32<D>;
    using C = LseF32Cfg<D, WM>;
    extern __shared__ __attribute__((aligned(16))) float sm[];
    float2* stats = reinterpret_cast<float2*>(sm + C::BUFS * WM * TL::FLOATS);   // [wave][32]: maximum and sum
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l32 = lane & 31, hl = lane >> 5;
    const int wt = w / WM, wm = w % WM;
    const int64_t nblk = (T + C::TOKENS - 1) / C::TOKENS;
    const int32_t h = (int32_t)(blockIdx.x / nblk);
    const int64_t blk0 = (blockIdx.x % nblk) * C::TOKENS, blk1 = blk0 + C::TOKENS < T ? blk0 + C::TOKENS : T;
    const int64_t tok = blk0 + wt * 32 + l32;
    float kop[D / 2];
    load_operand<false, D>(K, ((tok < T ? tok : T - 1) * H + h) * D, hl, kop);
    const float ks2 = scale * kLog2e;
    const int ntiles = (M + 31) / 32;

    // with one prototype block per user, one round per user that has tokens here
    int64_t b = 0, lo = 0, hi = T;
    if (p_user) b = first_user_after(off, B, T, blk0);
    for (; p_user ? b < B : b < 1; ++b) {
        if (p_user) {
            lo = seg_clamp(off[b], T);
            hi = seg_clamp(off[b + 1], T);
            if (lo >= blk1) break;
            if (__builtin_expect(hi <= lo, 0)) {   // no tokens: past those like it
                b = next_user_after(off, b + 1, B, T, lo) - 1;
                continue;
            }
            if (hi <= blk0) continue;
        }
        const float* Pg = P + (p_user ? b * H + h : (int64_t)h) * M * D;
        TileLoad<false, D, 256> ld[WM];
        auto fetch = [&](int t) {
#pragma unroll
            for (int i = 0; i < WM; ++i)
                ld[i].fetch(Pg, tid, [=](int r) { return (int64_t)min((t + i) * 32 + r, M - 1) * D; });
        };
        auto store = [&](int buf) {
#pragma unroll
            for (int i = 0; i < WM; ++i) ld[i].store(sm + (buf * WM + i) * TL::FLOATS, tid, 32);
        };
        // log2 units; the maximum stays finite while all logits are -inf, or while a wave
        // has no tile
        float mu = -kFloatMax, z = 0.f;
        fetch(0);
        __syncthreads();   // the previous round is done with the tiles
        store(0);
        __syncthreads();
        for (int t0 = 0, buf = 0; t0 < ntiles; t0 += WM) {
            const bool more = t0 + WM < ntiles;
            if (more) fetch(t0 + WM);
            const int t = t0 + wm;
            if (t < ntiles) {
                const f32x16 s = TL::rows_dot(sm + (buf * WM + wm) * TL::FLOATS, l32, hl, kop);
                const bool ragged = t * 32 + 32 > M;   // rows past M: no part in the maximum or the sum
                float x[16], m = -kFloatMax;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    x[r] = s[r];
                    m = fmaxf(m, ragged && t * 32 + srow(r, hl) >= M ? m : x[r]);
                }
                const float mn = fmaxf(mu, m * ks2);
                z *= __builtin_amdgcn_exp2f(mu - mn);   // z is 0 on the first tile
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], ks2, -mn));
                    z += ragged && t * 32 + srow(r, hl) >= M ? 0.f : e;
                }
                mu = mn;
            }
            if constexpr (C::BUFS == 1) __syncthreads();   // every wave is done with the tiles
            else buf ^= 1;
            if (more) store(buf);
            __syncthreads();
        }
        // the two half-waves, and the waves sharing the tokens, hold the token's other
        // prototype rows
        const auto m2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mu), __float_as_uint(mu), false, false);
        const auto z2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(z), __float_as_uint(z), false, false);
        const float ma = __uint_as_float(m2[0]), mb = __uint_as_float(m2[1]);
        float mx = fmaxf(ma, mb);
        float zz = __uint_as_float(z2[0]) * __builtin_amdgcn_exp2f(ma - mx) +
                   __uint_as_float(z2[1]) * __builtin_amdgcn_exp2f(mb - mx);
        if constexpr (WM > 1) {
            if (hl == 0) stats[w * 32 + l32] = make_float2(mx, zz);
            __syncthreads();
            if (wm == 0) {
#pragma unroll
                for (int q = 1; q < WM; ++q) mx = fmaxf(mx, stats[(w + q) * 32 + l32].x);
                zz = 0.f;
#pragma unroll
                for (int q = 0; q < WM; ++q) {
                    const float2 o = stats[(w + q) * 32 + l32];
                    zz += o.y * __builtin_amdgcn_exp2f(o.x - mx);
                }
            }
        }
        if (wm == 0 && hl == 0 && tok >= lo && tok < hi)
            lse[tok * H + h] = __builtin_fmaf(mx, kLn2, __builtin_amdgcn_logf(zz) * kLn2);
    }
}

// Waves sharing a workgroup's tokens: four where workgroups of 128 tokens leave CUs idle
// (M = 4096, d = 64, one user of 64 tokens, the call: 217 us with one, 82 with four; M = 512,
// d = 128, one of 2,048: 79 and 52).
template <int D, int WM>
hipError_t launch_lse_f32(const SplitFwdArgs& f, hipStream_t stream) {
    using C = LseF32Cfg<D, WM>;
    const int64_t nblk = (f.T + C::TOKENS - 1) / C::TOKENS;
    if (nblk * f.H > 0x7fffffff) return hipErrorInvalidValue;
    auto kern = lse_f32_kernel<D, WM>;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)C::LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3((unsigned)(nblk * f.H)), dim3(256), C::LDS, stream, reinterpret_cast<const float*>(f.K),
                       reinterpret_cast<const float*>(f.P), f.offsets, f.B, f.T, f.H, f.M, f.scale, f.p_user, f.lse);
    return hipGetLastError();
}

// workgroup -> (token range, part of the prototypes), the parts of a range back to
// back on one XCD; false for the grid's padding
__device__ inline bool range_part(int64_t n_ranges, int parts, int64_t& range, int& part) {
    const int64_t xcd = blockIdx.x % 8, jx = blockIdx.x / 8;
    part = (int)(jx % parts);
    const int64_t ix = jx / parts, q8 = n_ranges / 8, r8 = n_ranges % 8;
    if (ix >= q8 + (xcd < r8 ? 1 : 0)) return false;
    range = xcd * q8 + (xcd < r8 ? xcd : r8) + ix;
    return true;
}

// acc += the product of a wave's 32 weights a lane pair with a tile's 32 token rows.
// The tile is summed on its own first: a sum over a range's thousands of tokens in one
// chain has a larger rounding error (16 users of up to 30K tokens,
// M = 256, against 64 bits: dP 7.8e-7, so summed 3.5e-7; the sketch 5.7e-7 -> 3.1e-7).
template <int D>
__device__ inline void add_tile(f32x16 (&acc)[D / 32], const float (&e)[16], const float* tile, int l32, int hl) {
    using TL = Tile32<D>;
#pragma unroll
    for (int jt = 0; jt < D / 32; ++jt) {
        f32x16 t = zero16();
#pragma unroll
        for (int r = 0; r < 16; ++r) t = mfma(e[r], TL::at(tile, r, l32, hl, jt), t);
        acc[jt] += t;
    }
}

// the wave's 32 result rows (prototypes m0 + srow(r, hl)) to out [M][D]
template <int D>
__device__ inline void store_rows(float* out, const f32x16 (&acc)[D / 32], int m0, int M, int l32, int hl, float f) {
#pragma unroll
    for (int jt = 0; jt < D / 32; ++jt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = m0 + srow(r, hl);
            if (m < M) out[(int64_t)m * D + 32 * jt + l32] = acc[jt][r] * f;
        }
}

// ---------------------------------------------------------------- forward: aggregation
struct AggF32Args {
    const float *K, *V, *P;
    const int64_t* off;
    const float* lse;
    int64_t B, T, C, n_ranges;
    int32_t H, M, parts;
    float scale;
    bool p_user;
    float* sketch;
    float* partials;
    float* lse_out;   // (ONE) [T,H], or null
};

// ONE: all M prototypes in the workgroup (one part): the log-sum-exp of a tile's
// tokens comes from its own logits, the waves' (maximum, sum) of each token combined
// through LDS, and no pass over the keys precedes (4 M d instead of 6 M d executed).
// `lse` is then an output, or null.
template <int D, int NW, bool ONE>
__global__ __launch_bounds__(NW * 64) void agg_f32_kernel(AggF32Args a) {
    using TL = Tile32<D>;
    constexpr int JT = D / 32, THREADS = NW * 64;
    extern __shared__ __attribute__((aligned(16))) float sm[];
    float* Kt = sm;                       // [2] tiles
    float* Vt = Kt + 2 * TL::FLOATS;      // [2] tiles
    float* shift = Vt + 2 * TL::FLOATS;   // [2][32]: -lse
    float2* stats = reinterpret_cast<float2*>(shift + 64);   // (ONE) [NW][32]: a wave's maximum and sum
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l32 = lane & 31, hl = lane >> 5;
    int64_t range;
    int part;
    if (!range_part(a.n_ranges, a.parts, range, part)) return;
    const int64_t MD = (int64_t)a.M * D;
    const int m0 = (part * NW + w) * 32;
    SegmentWalk walk(a.off, a.B, a.T, a.H, a.C, a.n_ranges, range);
    Segment sg;
    while (walk.next(sg)) {
        const int t0 = sg.t0, t1 = sg.t1, h = sg.h;
        float pop[D / 2];
        load_operand<false, D>(a.P, (a.p_user ? (int64_t)sg.b * a.H + h : (int64_t)h) * MD + (int64_t)min(m0 + l32, a.M - 1) * D,
                               hl, pop);
        TileLoad<false, D, THREADS> lk, lv;
        float ll;
        auto fetch = [&](int ts) {
            auto row = [&](int i) { return ((int64_t)min(ts + i, t1 - 1) * a.H + h) * D; };
            lk.fetch(a.K, tid, row);
            lv.fetch(a.V, tid, row);
            if constexpr (!ONE) ll = a.lse[(int64_t)min(ts + l32, t1 - 1) * a.H + h];
        };
        auto store = [&](int ts, int buf) {
            lk.store(Kt + buf * TL::FLOATS, tid, 32);
            lv.store(Vt + buf * TL::FLOATS, tid, t1 - ts);   // V of rows past the segment: zeros
            if constexpr (!ONE) {
                if (tid < 32) shift[buf * 32 + tid] = -ll;
            }
        };
        f32x16 acc[JT];
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) acc[jt] = zero16();
        fetch(t0);
        __syncthreads();   // the previous segment is done with the tiles
        store(t0, 0);
        __syncthreads();
        for (int ts = t0, buf = 0; ts < t1; ts += 32, buf ^= 1) {
            const bool more = ts + 32 < t1;
            if (more) fetch(ts + 32);
            f32x16 s = TL::rows_dot(Kt + buf * TL::FLOATS, l32, hl, pop);
            float e[16];
            if constexpr (ONE) {
                // per token: maximum and sum over this wave's prototypes (those past M
                // count as -inf, and a wave without any as an empty sum; the maximum
                // stays finite where all of a wave's logits are -inf)
                const bool valid = m0 + l32 < a.M;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float x = valid ? s[r] * a.scale : -INFINITY;
                    const float m = fmaxf(half_max(x), -kFloatMax);
                    const float z = half_sum(exp_f32(x - m));
                    if (l32 == 0) stats[w * 32 + srow(r, hl)] = m0 < a.M ? make_float2(m, z) : make_float2(-INFINITY, 0.f);
                }
                __syncthreads();
                if (tid < 32) {
                    float m = stats[tid].x;
#pragma unroll
                    for (int q = 1; q < NW; ++q) m = fmaxf(m, stats[q * 32 + tid].x);
                    float z = 0.f;
#pragma unroll
                    for (int q = 0; q < NW; ++q) {
                        const float2 o = stats[q * 32 + tid];
                        z += o.y == 0.f ? 0.f : o.y * exp_f32(o.x - m);
                    }
                    const float l = __builtin_fmaf(__builtin_amdgcn_logf(z), kLn2, m);
                    shift[buf * 32 + tid] = -l;
                    if (a.lse_out && ts + tid < t1) a.lse_out[(int64_t)(ts + tid) * a.H + h] = l;
                }
                __syncthreads();
            }
#pragma unroll
            for (int r = 0; r < 16; ++r)
                e[r] = exp_f32(__builtin_fmaf(s[r], a.scale, shift[buf * 32 + srow(r, hl)]));
            add_tile<D>(acc, e, Vt + buf * TL::FLOATS, l32, hl);
            if (more) store(ts + 32, buf ^ 1);
            __syncthreads();
        }
        store_rows<D>(sg.split ? a.partials + sg.slot * MD : a.sketch + ((int64_t)sg.b * a.H + h) * MD, acc, m0, a.M, l32,
                      hl, 1.0f);
    }
}

// ---------------------------------------------------------------- backward: token side
struct BwdF32Args {
    const void *K, *V, *P;
    const int64_t* off;
    const float *dY, *lse;
    int64_t B, T, C, n_ranges;
    int32_t H, M, parts;
    float scale;
    bool p_user, dx_add;
    float* Dbuf;
    float *dK, *dV, *dX;   // dX: K and V are one tensor, its gradient is written there
    float* dP;             // [H,M,d], or [B,H,M,d] with p_user
    float* partials;       // [n_ranges + H, or n_ranges + H B with p_user][M][d]
};

// Workgroup = 4 waves of 32 tokens: up to 128 tokens of one user, counted from the
// user's first, and one head; P and dY tiles of 32 prototypes stream through LDS,
// twice.  Result tiles have prototypes (or features) as rows and a token per lane.
//
// User b's blocks are numbers floor(off[b] / 128) + b on: floor(off[b+1] / 128) + b + 1
// is at least ceil(length / 128) further, so floor(T / 128) + B numbers a head hold every
// user's blocks, found by binary search.  With ranges of 128 tokens cut anywhere, the
// ranges that held two users' tokens did two passes over the prototypes one after the
// other and the launch waited for them (9,619 tokens of 8 users, H = 2, M = 256, d = 64:
// 121 us, now 68).
template <bool BF16, int D, bool XV>
__global__ __launch_bounds__(256) void bwd_token_f32_kernel(BwdF32Args a) {
    using TL = Tile32<D>;
    constexpr int JT = D / 32;
    extern __shared__ __attribute__((aligned(16))) float sm[];
    float* Pt = sm;                      // [2] tiles
    float* Yt = Pt + 2 * TL::FLOATS;     // [2] tiles
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l32 = lane & 31, hl = lane >> 5;
    const int64_t MD = (int64_t)a.M * D;
    const int ntiles = (a.M + 31) / 32;

    const int64_t nblk = a.T / 128 + a.B + 1, blk = blockIdx.x % nblk;
    const int h = (int)(blockIdx.x / nblk);
    const int64_t first = a.B > 0 ? seg_clamp(a.off[0], a.T) : 0, last = a.B > 0 ? seg_clamp(a.off[a.B], a.T) : 0;
    // tokens before the first user's and after the last one's: zero gradients
    for (int64_t t = blk; t < a.T; t += nblk) {
        if (t >= first && t < last) {
            t += (last - 1 - t) / nblk * nblk;   // this workgroup's next one is past the users'
            continue;
        }
        for (int j = tid; j < D; j += 256) {
            const int64_t o = (t * a.H + h) * D + j;
            if constexpr (XV) {
                if (!a.dx_add) a.dX[o] = 0.f;
            } else {
                a.dK[o] = 0.f;
                a.dV[o] = 0.f;
            }
            if (j == 0) a.Dbuf[t * a.H + h] = 0.f;
        }
    }
    // the last user whose first number is not past blk
    int64_t ub = 0;
    for (int64_t hi = a.B; ub + 1 < hi;) {
        const int64_t mid = (ub + hi) >> 1;
        if (seg_clamp(a.off[mid], a.T) / 128 + mid <= blk) ub = mid; else hi = mid;
    }
    if (a.B == 0) return;
    Segment sg;
    {
        const int64_t lo = seg_clamp(a.off[ub], a.T), hi = seg_clamp(a.off[ub + 1], a.T);
        const int64_t t0 = lo + (blk - lo / 128 - ub) * 128;
        if (t0 < lo || t0 >= hi) return;
        sg.b = (int32_t)ub;
        sg.t0 = (int32_t)t0;
        sg.t1 = (int32_t)(t0 + 128 < hi ? t0 + 128 : hi);
    }
    {
        const int64_t pair = (int64_t)sg.b * a.H + h;
        const int tok = sg.t0 + w * 32 + l32;
        const bool live = tok < sg.t1;
        const int64_t trow = (int64_t)min(tok, sg.t1 - 1) * a.H + h;
        float kop[D / 2], vop[XV ? 1 : D / 2];
        load_operand<BF16, D>(a.K, trow * D, hl, kop);
        if constexpr (!XV) load_operand<BF16, D>(a.V, trow * D, hl, vop);
        auto vval = [&](int i) {
            if constexpr (XV) return kop[i];
            else return vop[i];
        };
        const float shift = -a.lse[trow];
        const int64_t p0 = (a.p_user ? pair : (int64_t)h) * MD, y0 = pair * MD;
        TileLoad<BF16, D, 256> lp;
        TileLoad<false, D, 256> ly;
        auto fetch = [&](int t) {
            auto row = [&](int i) { return (int64_t)min(t * 32 + i, a.M - 1) * D; };
            lp.fetch(a.P, tid, [&](int i) { return p0 + row(i); });
            ly.fetch(a.dY, tid, [&](int i) { return y0 + row(i); });
        };
        auto store = [&](int buf) {
            lp.store(Pt + buf * TL::FLOATS, tid, 32);
            ly.store(Yt + buf * TL::FLOATS, tid, 32);
        };
        // weights of prototype tile t (0 for rows past M)
        auto weights = [&](int t, const float* P, float (&e)[16]) {
            const f32x16 s = TL::rows_dot(P, l32, hl, kop);
            const bool ragged = t * 32 + 32 > a.M;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                e[r] = exp_f32(__builtin_fmaf(s[r], a.scale, shift));
                if (ragged && t * 32 + srow(r, hl) >= a.M) e[r] = 0.f;
            }
        };
        f32x16 acc[JT], accv[XV ? JT : 1];   // accv: dV, added to dK at the end
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) acc[jt] = zero16();
        float Dt = 0.f;
        fetch(0);
        __syncthreads();   // the previous segment is done with the tiles
        store(0);
        __syncthreads();
        for (int st = 0; st < 2 * ntiles; ++st) {
            const int t = st < ntiles ? st : st - ntiles;
            const bool more = st + 1 < 2 * ntiles;
            if (more) fetch(st + 1 < ntiles ? st + 1 : st + 1 - ntiles);
            const float* P = Pt + (st & 1) * TL::FLOATS;
            const float* Y = Yt + (st & 1) * TL::FLOATS;
            float e[16];
            weights(t, P, e);
            if (st < ntiles) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
#pragma unroll
                    for (int jt = 0; jt < JT; ++jt) acc[jt] = mfma(TL::at(Y, r, l32, hl, jt), e[r], acc[jt]);
            } else {
                f32x16 g;
                if constexpr (XV) g = TL::rows_dot(Y, l32, hl, kop);
                else g = TL::rows_dot(Y, l32, hl, vop);
#pragma unroll
                for (int r = 0; r < 16; ++r) e[r] *= g[r] - Dt;
#pragma unroll
                for (int r = 0; r < 16; ++r)
#pragma unroll
                    for (int jt = 0; jt < JT; ++jt) acc[jt] = mfma(TL::at(P, r, l32, hl, jt), e[r], acc[jt]);
            }
            if (st + 1 == ntiles) {
                // dV complete: D_t = <V_t, dV_t>, both half-waves' features
                float dd = 0.f;
#pragma unroll
                for (int jt = 0; jt < JT; ++jt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) dd = __builtin_fmaf(vval(16 * jt + r), acc[jt][r], dd);
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(dd), __float_as_uint(dd), false, false);
                Dt = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
                if (live && hl == 0) a.Dbuf[trow] = Dt;
#pragma unroll
                for (int jt = 0; jt < JT; ++jt) {
                    if constexpr (XV) {
                        accv[jt] = acc[jt];
                    } else {
#pragma unroll
                        for (int g = 0; g < 4; ++g)
                            if (live)
                                *reinterpret_cast<float4*>(a.dV + trow * D + 32 * jt + 8 * g + 4 * hl) =
                                    make_float4(acc[jt][4 * g], acc[jt][4 * g + 1], acc[jt][4 * g + 2], acc[jt][4 * g + 3]);
                    }
                    acc[jt] = zero16();
                }
            }
            if (more) store((st + 1) & 1);
            __syncthreads();
        }
        if (live) {
#pragma unroll
            for (int jt = 0; jt < JT; ++jt)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float4 v = make_float4(a.scale * acc[jt][4 * g], a.scale * acc[jt][4 * g + 1],
                                           a.scale * acc[jt][4 * g + 2], a.scale * acc[jt][4 * g + 3]);
                    float4* out;
                    if constexpr (XV) {
                        v = make_float4(accv[jt][4 * g] + v.x, accv[jt][4 * g + 1] + v.y, accv[jt][4 * g + 2] + v.z,
                                        accv[jt][4 * g + 3] + v.w);
                        out = reinterpret_cast<float4*>(a.dX + trow * D + 32 * jt + 8 * g + 4 * hl);
                        if (a.dx_add) {
                            const float4 o = *out;
                            v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
                        }
                    } else {
                        out = reinterpret_cast<float4*>(a.dK + trow * D + 32 * jt + 8 * g + 4 * hl);
                    }
                    *out = v;
                }
        }
    }
}

// ---------------------------------------------------------------- backward: prototype side
// Workgroup = (token range, 32 NW prototypes), a wave = 32 prototypes with their P
// and (the segment's user's) dY rows held as operands; result tiles have tokens as
// rows and a prototype per lane.  Shared prototypes accumulate over the users of a
// head and leave one partial per (range, head); per-user ones one per segment.
template <bool BF16, int D, int NW>
__global__ __launch_bounds__(NW * 64) void bwd_proto_f32_kernel(BwdF32Args a) {
    using TL = Tile32<D>;
    constexpr int JT = D / 32, THREADS = NW * 64;
    extern __shared__ __attribute__((aligned(16))) float sm[];
    float* Kt = sm;
    float* Vt = Kt + 2 * TL::FLOATS;
    float* shift = Vt + 2 * TL::FLOATS;   // [2][32]: -lse
    float* Ds = shift + 64;               // [2][32]: D_t
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l32 = lane & 31, hl = lane >> 5;
    int64_t range;
    int part;
    if (!range_part(a.n_ranges, a.parts, range, part)) return;
    const int64_t MD = (int64_t)a.M * D;
    const int m0 = (part * NW + w) * 32, mrow = min(m0 + l32, a.M - 1);
    f32x16 acc[JT];
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) acc[jt] = zero16();
    // shared prototypes: the heads of this range up to h1, each with its sum (zero
    // where no user has tokens), to the head's slot or straight to dP
    const int64_t HT = (int64_t)a.H * a.T, g_end = min((range + 1) * a.C, HT);
    int cur_h = (int)(range * a.C / a.T);
    auto flush_to = [&](int h1) {
        for (; cur_h < h1; ++cur_h) {
            const int64_t g0 = (int64_t)cur_h * a.T, g1 = g0 + a.T - 1;
            const int64_t slot = g0 <= range * a.C ? range : a.n_ranges + cur_h;
            store_rows<D>(g0 / a.C != g1 / a.C ? a.partials + slot * MD : a.dP + cur_h * MD, acc, m0, a.M, l32, hl, a.scale);
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) acc[jt] = zero16();
        }
    };
    SegmentWalk walk(a.off, a.B, a.T, a.H, a.C, a.n_ranges, range);
    Segment sg;
    while (walk.next(sg)) {
        const int t0 = sg.t0, t1 = sg.t1, h = sg.h;
        const int64_t pair = (int64_t)sg.b * a.H + h;
        if (!a.p_user) flush_to(h);
        float pop[D / 2], yop[D / 2];
        load_operand<BF16, D>(a.P, (a.p_user ? pair : (int64_t)h) * MD + (int64_t)mrow * D, hl, pop);
        load_operand<false, D>(a.dY, pair * MD + (int64_t)mrow * D, hl, yop);
        TileLoad<BF16, D, THREADS> lk, lv;
        float ll, ld;
        auto fetch = [&](int ts) {
            auto row = [&](int i) { return ((int64_t)min(ts + i, t1 - 1) * a.H + h) * D; };
            lk.fetch(a.K, tid, row);
            lv.fetch(a.V, tid, row);
            const int64_t i = (int64_t)min(ts + l32, t1 - 1) * a.H + h;
            ll = a.lse[i];
            ld = a.Dbuf[i];
        };
        auto store = [&](int buf) {
            lk.store(Kt + buf * TL::FLOATS, tid, 32);
            lv.store(Vt + buf * TL::FLOATS, tid, 32);
            if (tid < 32) {
                shift[buf * 32 + tid] = -ll;
                Ds[buf * 32 + tid] = ld;
            }
        };
        fetch(t0);
        __syncthreads();   // the previous segment is done with the tiles
        store(0);
        __syncthreads();
        for (int ts = t0, buf = 0; ts < t1; ts += 32, buf ^= 1) {
            const bool more = ts + 32 < t1;
            if (more) fetch(ts + 32);
            const float* Kb = Kt + buf * TL::FLOATS;
            const f32x16 s = TL::rows_dot(Kb, l32, hl, pop);
            const f32x16 g = TL::rows_dot(Vt + buf * TL::FLOATS, l32, hl, yop);
            float e[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = srow(r, hl);
                e[r] = exp_f32(__builtin_fmaf(s[r], a.scale, shift[buf * 32 + row])) * (g[r] - Ds[buf * 32 + row]);
                if (ts + row >= t1) e[r] = 0.f;   // past the segment
            }
            add_tile<D>(acc, e, Kb, l32, hl);
            if (more) store(buf ^ 1);
            __syncthreads();
        }
        if (a.p_user) {
            store_rows<D>(sg.split ? a.partials + sg.slot * MD : a.dP + pair * MD, acc, m0, a.M, l32, hl, a.scale);
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) acc[jt] = zero16();
        }
    }
    if (!a.p_user) flush_to((int)((g_end - 1) / a.T) + 1);
}

// dY[b,h] = sum over the R targets of dsketch
__global__ __launch_bounds__(256) void dy_kernel(const float4* __restrict__ ds, int64_t n4, int32_t R, int64_t hmd4,
                                                 float4* __restrict__ dY) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const int64_t b = i / hmd4, rest = i % hmd4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int r = 0; r < R; ++r) {
        const float4 v = ds[(b * R + r) * hmd4 + rest];
        s = make_float4(s.x + v.x, s.y + v.y, s.z + v.z, s.w + v.w);
    }
    dY[i] = s;
}

// Waves of 32 prototypes per workgroup: as many as M fills, up to eight.  At d = 128 eight
// waves, two a SIMD with 256 registers each, spill: none on the prototype side of the
// backward, and in the forward only for M <= 256, where one pass takes all prototypes
// (61 registers spilled; in two passes with four waves 8 users of 1,200 tokens take 51
// instead of 70 us, one of 50K 118 instead of 116, but lse is 1.2 times as far from 64 bits).
// Forward with eight waves (53 spilled) / four: M = 512, 8 users of 1,200 tokens 103 / 73 us,
// one of 50K 229 / 212.  (At d = 64 the prototype side's eight waves spill 14 registers
// and are still ahead on long batches: M = 1024, 50K tokens, training step 786, with four 834.)
int part_waves(int32_t M) { return M <= 64 ? 2 : (M % 256 > 0 && M % 256 <= 128 ? 4 : 8); }
int fwd_waves(int32_t M, int32_t d) { return d == 128 && M > 256 ? 4 : part_waves(M); }
int proto_waves(int32_t M, int32_t d) { return d == 64 ? part_waves(M) : (M <= 64 ? 2 : 4); }

// ranges that give every CU its two waves per SIMD once, in at most two workgroups per
// CU; one wave (by its registers) with `one`: four waves at d = 128, any number there on
// the prototype side
int64_t ranges(int32_t M, int nw, bool one) {
    const int64_t parts = (M + 32 * nw - 1) / (32 * nw);
    return xcd_ranges(one || nw == 8 ? 1 : 2, parts);
}

template <typename Kern, typename Args>
hipError_t launch_parts(Kern kern, Args a, int nw, size_t lds, hipStream_t stream) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    a.parts = (a.M + 32 * nw - 1) / (32 * nw);
    const int64_t per_xcd = (a.n_ranges + 7) / 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * per_xcd * a.parts)), dim3(nw * 64), lds, stream, a);
    return hipGetLastError();
}

template <int D>
hipError_t fwd_impl(const SplitFwdArgs& f, hipStream_t stream) {
    const float *K = reinterpret_cast<const float*>(f.K), *V = reinterpret_cast<const float*>(f.V),
                *P = reinterpret_cast<const float*>(f.P);
    AggF32Args a{K, V, P, f.offsets, f.lse, f.B, f.T, f.C, f.n_ranges, f.H, f.M, 1, f.scale, f.p_user, f.sketch, f.partials,
                 nullptr};
    const int nw = fwd_waves(f.M, D);
    if (f.M <= 32 * nw) {   // one part: no pass for the log-sum-exp
        a.lse_out = f.lse;
        const size_t lds = (4 * Tile32<D>::FLOATS + 64 + 64 * nw) * sizeof(float);
        ProfScope ps("plain_fwd", stream);
        switch (nw) {
            case 2: return launch_parts(agg_f32_kernel<D, 2, true>, a, 2, lds, stream);
            case 4: return launch_parts(agg_f32_kernel<D, 4, true>, a, 4, lds, stream);
            default: return launch_parts(agg_f32_kernel<D, 8, true>, a, 8, lds, stream);
        }
    }
    {
        ProfScope ps("plain_lse", stream);
        const hipError_t e = (f.T + 127) / 128 * f.H < device_cus() ? launch_lse_f32<D, 4>(f, stream) : launch_lse_f32<D, 1>(f, stream);
        if (e != hipSuccess) return e;
    }
    const size_t lds = (4 * Tile32<D>::FLOATS + 64) * sizeof(float);
    ProfScope ps("plain_agg", stream);
    if constexpr (D == 64) {
        if (nw == 8) return launch_parts(agg_f32_kernel<D, 8, false>, a, 8, lds, stream);
    }
    return launch_parts(agg_f32_kernel<D, 4, false>, a, 4, lds, stream);
}

template <bool BF16, int D>
hipError_t bwd_impl(const PlainBwdArgs& f, hipStream_t stream) {
    BwdF32Args a{f.K, f.V, f.P, f.offsets, f.dY, f.lse, f.B, f.T, f.C, f.n_ranges, f.H, f.M, 1, f.scale, f.p_user, f.dx_add,
                 f.Dbuf, f.dK, f.dV, f.dX, f.dP, f.partials};
    const int64_t HT = (int64_t)f.H * f.T;
    if (HT > 0) {
        hipError_t e;
        {
            ProfScope ps("plain_bwd_token", stream);
            const size_t lds = 4 * Tile32<D>::FLOATS * sizeof(float);
            const int64_t blocks = (f.T / 128 + f.B + 1) * f.H;
            if (blocks > 0x7fffffff) return hipErrorInvalidValue;
            auto kern = f.dX ? bwd_token_f32_kernel<BF16, D, true> : bwd_token_f32_kernel<BF16, D, false>;
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), lds, stream, a);
            e = hipGetLastError();
        }
        if (e != hipSuccess) return e;
        ProfScope ps("plain_bwd_proto", stream);
        const size_t lds = (4 * Tile32<D>::FLOATS + 128) * sizeof(float);
        switch (proto_waves(f.M, D)) {
            case 2: e = launch_parts(bwd_proto_f32_kernel<BF16, D, 2>, a, 2, lds, stream); break;
            case 4: e = launch_parts(bwd_proto_f32_kernel<BF16, D, 4>, a, 4, lds, stream); break;
            default:   // (d = 64 only: at d = 128 eight waves do not fit the registers)
                if constexpr (D == 64) e = launch_parts(bwd_proto_f32_kernel<BF16, D, 8>, a, 8, lds, stream);
                else e = hipErrorInvalidValue;
        }
        if (e != hipSuccess) return e;
    }
    // shared prototypes: each head's T tokens are one run of ranges
    ProfScope ps("plain_dp_sum", stream);
    return launch_merge_ranges(f.p_user ? f.offsets : nullptr, f.p_user ? f.B : 1, f.T, f.H, f.C, f.n_ranges, f.partials,
                               (int64_t)f.M * D, f.dP, stream);
}

}  // namespace

int64_t plain_fwd_ranges(int32_t M, int32_t d) {
    return ranges(M, fwd_waves(M, d), d == 128 && fwd_waves(M, d) == 4);
}
int64_t plain_bwd_ranges(int32_t M, int32_t d) { return ranges(M, proto_waves(M, d), d == 128); }

hipError_t launch_plain_fwd(const SplitFwdArgs& f, hipStream_t stream) {
    if (f.T == 0) return hipSuccess;
    return f.d == 64 ? fwd_impl<64>(f, stream) : fwd_impl<128>(f, stream);
}

hipError_t launch_dy_reduce(const float* dsketch, int64_t B, int32_t R, int32_t H, int64_t MD, float* dY,
                            hipStream_t stream) {
    const int64_t n4 = B * H * MD / 4;   // MD is a multiple of 4 (d is 64 or 128)
    if (n4 == 0) return hipSuccess;
    hipLaunchKernelGGL(dy_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, stream,
                       reinterpret_cast<const float4*>(dsketch), n4, R, H * MD / 4, reinterpret_cast<float4*>(dY));
    return hipGetLastError();
}

hipError_t launch_plain_bwd(const PlainBwdArgs& f, bool bf16, hipStream_t stream) {
    if (f.d == 64) return bf16 ? bwd_impl<true, 64>(f, stream) : bwd_impl<false, 64>(f, stream);
    return bf16 ? bwd_impl<true, 128>(f, stream) : bwd_impl<false, 128>(f, stream);
}

}  // namespace sa
