// Two-pass forward of the SA sketching step on bf16 inputs.  It runs the shapes the
// one-pass fused kernel (fwd_fused.hip) has no instance for: M x d too large for one
// workgroup's registers (d = 128 above 512 prototypes, d = 64 above 1024), or M
// not a multiple of 128; there the weights keep their fp32 precision.  And it runs
// short batches of the one-pass shapes, with that kernel's bf16 weights.
//
// Two passes over the keys:
//
//   lse_tokens_kernel  lse_t = log sum_m exp(scale <K_t, P_m>)
//   agg_split_kernel   A = exp(scale <K_t, P_m> - lse_t);  sketch_m += A V_t
//
// so that a workgroup of the second pass needs only its own prototypes (section
// 3.1: the softmax of a token couples all M prototypes through lse_t alone) and
// the M x d accumulator is spread over workgroups.
//
// Products of bf16 inputs are exact in the matrix cores' fp32 accumulation, so
// the logits are single-precision sums.  fp32 weights A: each is cut into
// three bf16 parts of eight mantissa bits, A = hi + mid + lo exactly (truncation,
// each remainder is exact), and the three products with the bf16 V accumulate in
// fp32.  Against float64 the sketch is then as close as a plain fp32 evaluation
// (5.3e-7 relative, 2-norm, at M = 1024, d = 128; the fp32 VALU path had 5.9e-7).
//
// Executed matrix work is (2 + 2 + 6) M d per token against 4 M d algorithmic;
// the aggregation is bound by its matrix instructions (32 of them per 32 x 32
// logits tile at d = 128) beside about 11 VALU instructions per weight.
// Measured on 100K tokens, H = 1, M = 1024, d = 128: lse 45 us, aggregation 118 us
// (890 TFLOP/s executed, against 1200 for a large library product), merge 7 us; the
// fp32 VALU path took 2.8 ms, 3.2 ms and 86 us.
#include <algorithm>
#include <type_traits>
#include "reduce_ops.h"
#include "sa_internal.h"
#include "segments.h"
#include "tile_ops.h"

namespace sa {

namespace {

using namespace tile;

constexpr float kLn2 = 0.6931471805599453f;
constexpr float kLog2eLo = 1.9259629911e-8f;   // 1 / ln 2 - kLog2e

// ---------------------------------------------------------------- log-sum-exp
// Workgroup = 4 waves; a wave holds 64 tokens of one head as B operands (two
// 32-token tiles share each prototype operand read from LDS), WM waves share the
// same tokens and take every WM-th 32 prototypes.  The prototypes stream through
// LDS ROWS at a time (double-buffered, the next tile in registers).  The logits
// tile has prototypes as rows and a token per lane, so the running maximum and sum
// of a token live in one lane per half-wave and wave: no cross-lane work until the
// end.
template <int D, int WM>
struct LseCfg {
    static constexpr int TT = 2;
    static constexpr int KS = D / 16;
    static constexpr int KCH = D / 8;
    static constexpr int ROWS = WM == 4 ? 128 : 64;       // prototypes per LDS tile
    static constexpr int SUB = ROWS / (32 * WM);          // 32-prototype tiles per wave and LDS tile
    static constexpr int NLD = ROWS * KCH / 256;          // 16-byte chunks per thread
    static constexpr int TILE = ROWS * D * 2;
    static constexpr int TOKENS = 4 / WM * 32 * TT;       // tokens per workgroup
};

// PU: P is [B,H,M,d], one prototype block per user: a round for every user with tokens here
// (an instance of its own: the walk over users in the other's code cost 2 of 45 us).
template <int D, int WM, bool PU>
__global__ __launch_bounds__(256, 2) void lse_tokens_kernel(const uint16_t* __restrict__ K,
                                                            const uint16_t* __restrict__ P,
                                                            const int64_t* __restrict__ off, int64_t B, int64_t T,
                                                            int32_t H, int32_t M, float scale,
                                                            float* __restrict__ lse) {
    using C = LseCfg<D, WM>;
    constexpr int KS = C::KS, TT = C::TT;
    __shared__ __attribute__((aligned(16))) uint8_t smem[2 * C::TILE];
    __shared__ float2 stats[WM > 1 ? 4 : 1][TT * 32];   // (maximum, sum) of each wave's tokens
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int l32 = lane & 31, hl = lane >> 5;
    const int wt = w / WM, wm = w % WM;
    const int64_t nblk = (T + C::TOKENS - 1) / C::TOKENS;
    const int32_t h = (int32_t)(blockIdx.x / nblk);
    const int64_t blk0 = (blockIdx.x % nblk) * C::TOKENS;          // the workgroup's first token
    const int64_t blk1 = blk0 + C::TOKENS < T ? blk0 + C::TOKENS : T;

    int64_t tok[TT];
    bf16x8 kop[TT][KS];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        tok[tt] = blk0 + (wt * TT + tt) * 32 + l32;
        const int64_t row = tok[tt] < T ? tok[tt] : T - 1;
        const uint16_t* src = K + (row * H + h) * D + 8 * hl;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
            kop[tt][kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + 16 * kk));
    }
    const float ks2 = scale * kLog2e;
    const int ntiles = (M + C::ROWS - 1) / C::ROWS;

    int64_t b = 0, lo = 0, hi = T;
    if constexpr (PU) b = first_user_after(off, B, T, blk0);
    for (; PU ? b < B : b < 1; ++b) {
        if constexpr (PU) {
            lo = seg_clamp(off[b], T);
            hi = seg_clamp(off[b + 1], T);
            if (lo >= blk1) break;
            if (__builtin_expect(hi <= lo, 0)) {   // no tokens: past those like it
                b = next_user_after(off, b + 1, B, T, lo) - 1;
                continue;
            }
            if (hi <= blk0) continue;
        }
        const uint16_t* Pg = P + (PU ? b * H + h : (int64_t)h) * M * D;
        u32x4 reg[C::NLD];
        auto fetch = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < C::NLD; ++i) {
                const int idx = tid + i * 256;
                const int row = min(tile * C::ROWS + idx / C::KCH, M - 1);
                reg[i] = *reinterpret_cast<const u32x4*>(Pg + (uint32_t)(row * D + (idx % C::KCH) * 8));
            }
        };
        auto store = [&](int buf) __attribute__((always_inline)) {
            uint16_t* dst = reinterpret_cast<uint16_t*>(smem + buf * C::TILE);
#pragma unroll
            for (int i = 0; i < C::NLD; ++i) {
                const int idx = tid + i * 256;
                *reinterpret_cast<u32x4*>(dst + swz<D>(idx / C::KCH, idx % C::KCH)) = reg[i];
            }
        };
        // log2 units; the maximum starts at the lowest finite value, so that it stays
        // finite while a lane has seen only masked rows (which the scale may take to
        // -inf) or logits of -inf, and no difference of two maxima is a NaN
        float mu[TT], z[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            mu[tt] = -3.4028234664e38f;
            z[tt] = 0.f;
        }
        // a logits tile into the running maximum and sum; in the ragged one, rows past
        // M have no part in either
        auto add_tile = [&](f32x16 (&s)[TT], int row0, auto ragged) __attribute__((always_inline)) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                if constexpr (ragged.value) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (row0 + srow(r, hl) >= M) s[tt][r] = -3.4028234664e38f;
                }
                float t = s[tt][0];
#pragma unroll
                for (int r = 1; r < 16; ++r) t = fmaxf(t, s[tt][r]);
                const float mn = fmaxf(mu[tt], t * ks2);
                z[tt] *= __builtin_amdgcn_exp2f(mu[tt] - mn);   // z is 0 on the first tile
                float sum[2] = {0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float e = __builtin_amdgcn_exp2f(__builtin_fmaf(s[tt][r], ks2, -mn));
                    if constexpr (ragged.value) {
                        if (row0 + srow(r, hl) >= M) e = 0.f;
                    }
                    sum[r & 1] += e;
                }
                z[tt] += sum[0] + sum[1];
                mu[tt] = mn;
            }
        };
        fetch(0);
        __syncthreads();   // the previous round is done with the tiles
        store(0);
        __syncthreads();
        for (int tile = 0; tile < ntiles; ++tile) {
            const bool more = tile + 1 < ntiles;
            if (more) fetch(tile + 1);
            const uint16_t* Ps = reinterpret_cast<const uint16_t*>(smem + (tile & 1) * C::TILE);
#pragma unroll
            for (int sub = 0; sub < C::SUB; ++sub) {
                const int r32 = (sub * WM + wm) * 32, row0 = tile * C::ROWS + r32;
                if (row0 >= M) break;
                f32x16 s[TT];
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[tt][r] = 0.f;
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) {
                    const bf16x8 pop = lds_b128(Ps, swz<D>(r32 + l32, 2 * kk + hl));
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt)
                        s[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pop, kop[tt][kk], s[tt], 0, 0, 0);
                }
                if (row0 + 32 <= M) add_tile(s, M, std::false_type{});
                else add_tile(s, row0, std::true_type{});
            }
            if (more) store((tile + 1) & 1);
            __syncthreads();
        }
        // the half-waves, and the waves sharing the tokens, hold a token's other
        // prototypes; every wave has a row of the last tile unless M ends before it
        auto merge = [](float ma, float za, float mb, float zb, float& m, float& z) {
            m = fmaxf(ma, mb);
            z = (za > 0.f || za != za ? za * __builtin_amdgcn_exp2f(ma - m) : 0.f) +
                (zb > 0.f || zb != zb ? zb * __builtin_amdgcn_exp2f(mb - m) : 0.f);
        };
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            const auto m2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mu[tt]), __float_as_uint(mu[tt]), false, false);
            const auto z2 = __builtin_amdgcn_permlane32_swap(__float_as_uint(z[tt]), __float_as_uint(z[tt]), false, false);
            merge(__uint_as_float(m2[0]), __uint_as_float(z2[0]), __uint_as_float(m2[1]), __uint_as_float(z2[1]), mu[tt], z[tt]);
            if constexpr (WM > 1) {
                if (hl == 0) stats[w][tt * 32 + l32] = make_float2(mu[tt], z[tt]);
            }
        }
        if constexpr (WM > 1) __syncthreads();
        if (wm == 0) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
                for (int q = 1; q < WM; ++q) {
                    const float2 o = stats[w + q][tt * 32 + l32];
                    merge(mu[tt], z[tt], o.x, o.y, mu[tt], z[tt]);
                }
                if (hl == 0 && tok[tt] >= lo && tok[tt] < hi)
                    lse[tok[tt] * H + h] = __builtin_fmaf(mu[tt], kLn2, __builtin_amdgcn_logf(z[tt]) * kLn2);
            }
        }
    }
}

// ---------------------------------------------------------------- aggregation
// Workgroup = (token range, 32 NW prototypes), a wave = 32 prototypes held in
// registers as B operands for the whole segment; token tiles of 32 double-buffered
// in LDS, fetched two tiles ahead into alternating register sets.  The logits tile
// has tokens as rows and a prototype per lane, which is the A operand layout of the
// aggregation (V read with the transposing LDS load).
template <int D, int NW>
struct AggCfg {
    static constexpr int THREADS = NW * 64;
    static constexpr int MP = 32 * NW;
    static constexpr int KS = D / 16;
    static constexpr int JT = D / 32;
    static constexpr int KCH = D / 8;
    static constexpr int LD_CHUNKS = 32 * KCH;
    static constexpr int NCH = (LD_CHUNKS + THREADS - 1) / THREADS;
    static constexpr int TILE = 32 * D * 2;
    static constexpr int OFF_K = 0;                    // 2 x [32][D] K tiles
    static constexpr int OFF_V = OFF_K + 2 * TILE;     // 2 x [32][D] V tiles
    static constexpr int OFF_L = OFF_V + 2 * TILE;     // 2 x [2][32] token shifts (see `shift`)
    static constexpr int OFF_F = OFF_L + 4 * 32 * 4;   // [2] first token + 1 of a tile with infinite or NaN V
    static constexpr int LDS = OFF_F + 16;
};

struct AggArgs {
    const uint16_t* K;
    const uint16_t* V;
    const uint16_t* P;
    const int64_t* off;
    const float* lse;
    int64_t B, T, C, n_ranges;
    int32_t H, M, parts;
    float scale;
    bool p_user;
    float* sketch;
    float* partials;
};

// whether any of eight bf16 values is infinite or NaN
__device__ inline bool nonfinite8(u32x4 v) {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    u16x2 m = __builtin_bit_cast(u16x2, v[0] & 0x7fff7fffu);
#pragma unroll
    for (int i = 1; i < 4; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, v[i] & 0x7fff7fffu));
    return m[0] >= 0x7f80 || m[1] >= 0x7f80;
}
__device__ inline uint32_t finite_or_zero(uint32_t w) {
    if ((w & 0x7f80u) == 0x7f80u) w &= 0xffff0000u;
    if ((w & 0x7f800000u) == 0x7f800000u) w &= 0xffffu;
    return w;
}

template <int D, int NW, int PARTS>
__global__ __launch_bounds__(NW * 64, 1) __attribute__((amdgpu_waves_per_eu(2, 2))) void agg_split_kernel(AggArgs a) {
    using C = AggCfg<D, NW>;
    constexpr int KS = C::KS, JT = C::JT;
    __shared__ __attribute__((aligned(16))) uint8_t smem[C::LDS];
    // The exponent of a weight is s ks2 - lse / ln 2: its second term rounded to
    // fp32 is added after the product, the rounding error (the same for all of a
    // token's weights) enters as the score chain's initial value.
    float* shift = reinterpret_cast<float*>(smem + C::OFF_L);
    volatile int* flag = reinterpret_cast<volatile int*>(smem + C::OFF_F);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int l32 = lane & 31, hl = lane >> 5;

    // workgroup -> (range, part): the parts of a range read the same tokens, so
    // they sit back to back on one XCD
    const int64_t xcd = blockIdx.x % 8, jx = blockIdx.x / 8;
    const int part = (int)(jx % a.parts);
    const int64_t ix = jx / a.parts;
    const int64_t q8 = a.n_ranges / 8, r8 = a.n_ranges % 8;
    if (ix >= q8 + (xcd < r8 ? 1 : 0)) return;
    const int64_t range = xcd * q8 + (xcd < r8 ? xcd : r8) + ix;

    const float ks2 = a.scale * kLog2e;
    const float rks2 = ks2 > 1e-37f ? 1.0f / ks2 : 0.f;   // (finite; below that the logits are zero)
    const int64_t MD = (int64_t)a.M * D;
    const int64_t row_stride = (int64_t)a.H * D;
    const int m0 = part * C::MP + w * 32;            // the wave's first prototype
    const int prow = min(m0 + l32, a.M - 1);         // this lane's (rows past M repeat the last)

    SegmentWalk walk(a.off, a.B, a.T, a.H, a.C, a.n_ranges, range);
    Segment sg;
    while (walk.next(sg)) {
        const int b = sg.b, h = sg.h, t0 = sg.t0, t1 = sg.t1;
        bf16x8 pop[KS];
        {
            const uint16_t* Pg = a.P + (a.p_user ? (int64_t)b * a.H + h : (int64_t)h) * MD + (int64_t)prow * D;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
                pop[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(Pg + 16 * kk + 8 * hl));
        }
        // Every fetch issues the same loads (rows past the segment read its last
        // token), so the wait before a store counts exactly the newer set's loads.
        struct Regs { u32x4 k[C::NCH], v[C::NCH]; float l; };
        Regs ra, rb;
        // Rows are addressed in 64 bits: with many prototype parts the ranges are few and a
        // segment may span more than 4 GB of K (one user of 1M tokens, 16 heads, d = 128).
        auto fetch = [&](int ts, Regs& r) __attribute__((always_inline)) {
            const int64_t tb = __builtin_amdgcn_readfirstlane(min(ts, t1 - 1));
            const int last = t1 - 1 - (int)tb;
            const int64_t base = (tb * a.H + h) * D;
#pragma unroll
            for (int c = 0; c < C::NCH; ++c) {
                const int idx = (tid + c * C::THREADS) % C::LD_CHUNKS;
                const int64_t o = base + min(idx / C::KCH, last) * row_stride + (idx % C::KCH) * 8;
                r.k[c] = *reinterpret_cast<const u32x4*>(a.K + o);
                r.v[c] = *reinterpret_cast<const u32x4*>(a.V + o);
            }
            r.l = a.lse[(tb + min(l32, last)) * a.H + h];
        };
        auto store = [&](int ts, int buf, const Regs& r) __attribute__((always_inline)) {
            uint16_t* Kd = reinterpret_cast<uint16_t*>(smem + C::OFF_K + buf * C::TILE);
            uint16_t* Vd = reinterpret_cast<uint16_t*>(smem + C::OFF_V + buf * C::TILE);
            bool bad = false;
#pragma unroll
            for (int c = 0; c < C::NCH; ++c) {
                const int idx = tid + c * C::THREADS;
                if (C::LD_CHUNKS % C::THREADS == 0 || idx < C::LD_CHUNKS) {
                    u32x4 v = r.v[c];
                    if (ts + idx / C::KCH >= t1) v = (u32x4){0, 0, 0, 0};   // V of rows past the segment
                    *reinterpret_cast<u32x4*>(Kd + swz<D>(idx / C::KCH, idx % C::KCH)) = r.k[c];
                    *reinterpret_cast<u32x4*>(Vd + swz<D>(idx / C::KCH, idx % C::KCH)) = v;
                    if constexpr (PARTS == 3) bad |= nonfinite8(v);
                }
            }
            if (w == 0 && hl == 0) {
                const float l2 = -r.l * kLog2e;
                const float lo = __builtin_fmaf(-r.l, kLog2eLo, __builtin_fmaf(-r.l, kLog2e, -l2));
                shift[buf * 64 + l32] = l2;
                shift[buf * 64 + 32 + l32] = __builtin_fabsf(r.l) < 1e30f ? lo * rks2 : 0.f;
            }
            if (bad) flag[buf] = ts + 1;
        };
        fetch(t0, ra);
        fetch(t0 + 32, rb);
        __syncthreads();   // the previous segment is done with every LDS buffer
        store(t0, 0, ra);
        __syncthreads();

        f32x16 acc[JT];
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[jt][r] = 0.f;
        // wait for the held operands here, so that the waits inside the loop count
        // the token fetches alone
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) asm volatile("" ::"v"(pop[kk]));

        auto step = [&](int ts, int buf, Regs& far, const Regs& nxt) __attribute__((always_inline)) {
            const bool more = ts + 32 < t1;
            fetch(ts + 64, far);
            const uint16_t* Ks = reinterpret_cast<const uint16_t*>(smem + C::OFF_K + buf * C::TILE);
            uint16_t* Vs = reinterpret_cast<uint16_t*>(smem + C::OFF_V + buf * C::TILE);
            f32x16 s;
            float sh[16];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 q = *reinterpret_cast<const float4*>(shift + buf * 64 + 8 * g + 4 * hl);
                const float4 c = *reinterpret_cast<const float4*>(shift + buf * 64 + 32 + 8 * g + 4 * hl);
                sh[4 * g] = q.x;
                sh[4 * g + 1] = q.y;
                sh[4 * g + 2] = q.z;
                sh[4 * g + 3] = q.w;
                s[4 * g] = c.x;
                s[4 * g + 1] = c.y;
                s[4 * g + 2] = c.z;
                s[4 * g + 3] = c.w;
            }
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_b128(Ks, swz<D>(l32, 2 * kk + hl)), pop[kk], s, 0, 0, 0);
            if constexpr (PARTS == 1) {
                float e[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) e[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], ks2, sh[r]));
                const bf16x8 e0 = pack8(e), e1 = pack8(e + 8);
#pragma unroll
                for (int jt = 0; jt < JT; ++jt) {
                    acc[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(e0, lds_tr_tokens<D>(Vs, lane, jt, 0), acc[jt], 0, 0, 0);
                    acc[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(e1, lds_tr_tokens<D>(Vs, lane, jt, 1), acc[jt], 0, 0, 0);
                }
            } else {
                // weights and their three bf16 parts (parts[p][i]: two tokens' values)
                uint32_t parts[3][8];
    #pragma unroll
                for (int i = 0; i < 8; ++i) {
                    float e[2], r1[2], r2[2];
    #pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        e[q] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * i + q], ks2, sh[2 * i + q]));
                        r1[q] = e[q] - bf16_hi(__float_as_uint(e[q]));
                        r2[q] = r1[q] - bf16_hi(__float_as_uint(r1[q]));
                    }
                    // the upper halves of two values, the first in the low half
                    parts[0][i] = __builtin_amdgcn_perm(__float_as_uint(e[1]), __float_as_uint(e[0]), 0x07060302u);
                    parts[1][i] = __builtin_amdgcn_perm(__float_as_uint(r1[1]), __float_as_uint(r1[0]), 0x07060302u);
                    parts[2][i] = __builtin_amdgcn_perm(__float_as_uint(r2[1]), __float_as_uint(r2[0]), 0x07060302u);
                }
                auto op = [&](int p, int h2) __attribute__((always_inline)) {
                    return __builtin_bit_cast(bf16x8, (u32x4){parts[p][4 * h2], parts[p][4 * h2 + 1], parts[p][4 * h2 + 2],
                                                              parts[p][4 * h2 + 3]});
                };
                if (__builtin_expect(flag[buf] != ts + 1, 1)) {
                    // a tile's products sum up on their own, the smallest parts first, and
                    // are added to the running sum once (one rounding at its magnitude per
                    // 32 tokens instead of six)
    #pragma unroll
                    for (int jt = 0; jt < JT; ++jt) {
                        const bf16x8 v0 = lds_tr_tokens<D>(Vs, lane, jt, 0), v1 = lds_tr_tokens<D>(Vs, lane, jt, 1);
                        f32x16 t = {};
    #pragma unroll
                        for (int p = 2; p >= 0; --p) {
                            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op(p, 0), v0, t, 0, 0, 0);
                            t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op(p, 1), v1, t, 0, 0, 0);
                        }
    #pragma unroll
                        for (int r = 0; r < 16; ++r) acc[jt][r] += t[r];
                    }
                } else {
                    // an infinite V times a weight's zero lower part would be NaN: the
                    // upper parts see V as it is, the others its finite values only
                    // (uniform over the workgroup: every thread reads the same flag)
                    auto add = [&](int p) __attribute__((always_inline)) {
    #pragma unroll
                        for (int jt = 0; jt < JT; ++jt)
    #pragma unroll
                            for (int h2 = 0; h2 < 2; ++h2)
                                acc[jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op(p, h2), lds_tr_tokens<D>(Vs, lane, jt, h2),
                                                                                  acc[jt], 0, 0, 0);
                    };
                    add(0);
                    __syncthreads();
                    for (int idx = tid; idx < C::LD_CHUNKS * 4; idx += C::THREADS) {
                        uint32_t* q = reinterpret_cast<uint32_t*>(Vs) + idx;
                        *q = finite_or_zero(*q);
                    }
                    __syncthreads();
                    add(1);
                    add(2);
                }
            }
            if (more) store(ts + 32, buf ^ 1, nxt);
            __syncthreads();
        };
        for (int ts = t0;; ts += 64) {
            step(ts, 0, ra, rb);
            if (ts + 32 >= t1) break;
            step(ts + 32, 1, rb, ra);
            if (ts + 64 >= t1) break;
        }
        // rows of this wave: prototypes m0 + srow(r, hl), columns jt*32 + l32
        float* out = sg.split ? a.partials + sg.slot * MD : a.sketch + ((int64_t)b * a.H + h) * MD;
        uint32_t lane_off = (uint32_t)((m0 + 4 * hl) * D + l32);
        asm volatile("" : "+v"(lane_off));
        if (m0 + 32 <= a.M) {
#pragma unroll
            for (int jt = 0; jt < JT; ++jt)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    out[lane_off + (uint32_t)((8 * (r >> 2) + (r & 3)) * D + jt * 32)] = acc[jt][r];
        } else {
#pragma unroll
            for (int jt = 0; jt < JT; ++jt)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (m0 + srow(r, hl) < a.M)
                        out[lane_off + (uint32_t)((8 * (r >> 2) + (r & 3)) * D + jt * 32)] = acc[jt][r];
        }
    }
}

template <int D, int NW, int PARTS>
hipError_t launch_agg(AggArgs a, hipStream_t stream) {
    a.parts = (a.M + 32 * NW - 1) / (32 * NW);
    const int64_t per_xcd = (a.n_ranges + 7) / 8;
    hipLaunchKernelGGL((agg_split_kernel<D, NW, PARTS>), dim3((unsigned)(8 * per_xcd * a.parts)), dim3(NW * 64), 0, stream, a);
    return hipGetLastError();
}

template <int D, int WM>
hipError_t launch_lse_inst(const SplitFwdArgs& f, hipStream_t stream) {
    const int64_t nblk = (f.T + LseCfg<D, WM>::TOKENS - 1) / LseCfg<D, WM>::TOKENS;
    if (nblk * f.H > 0x7fffffff) return hipErrorInvalidValue;
    auto kern = f.p_user ? lse_tokens_kernel<D, WM, true> : lse_tokens_kernel<D, WM, false>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(nblk * f.H)), dim3(256), 0, stream, f.K, f.P, f.offsets, f.B, f.T, f.H, f.M,
                       f.scale, f.lse);
    return hipGetLastError();
}
// Waves sharing a workgroup's tokens: none while 256-token workgroups give every CU
// one (each prototype operand then serves the most tokens), two or four below that.
// Measured (us; sharing 1 / 2 / 4 waves): M = 1024, d = 128, 100K tokens (391 workgroups
// of 256) 45 / 52 / 59; M = 2048, d = 128, 15K tokens (59 of 256) 50 / 33 / 23.
template <int D>
hipError_t launch_lse(const SplitFwdArgs& f, hipStream_t stream) {
    const int64_t n256 = (f.T + 255) / 256 * f.H;
    if (n256 >= device_cus()) return launch_lse_inst<D, 1>(f, stream);
    if (2 * n256 >= device_cus()) return launch_lse_inst<D, 2>(f, stream);
    return launch_lse_inst<D, 4>(f, stream);
}

// Waves (of 32 prototypes) per aggregation workgroup: eight, or four where eight
// would leave at least half a workgroup without prototypes, two for M <= 64.
int agg_waves(int32_t M) {
    if (M <= 64) return 2;
    const int rest = M % 256;
    return rest > 0 && rest <= 128 ? 4 : 8;
}

}  // namespace

int64_t split_fwd_ranges(int32_t M, bool bf16_weights, int64_t HT, int64_t pairs) {
    // two waves per SIMD of every CU in one round of workgroups, at most two
    // workgroups per CU and as many ranges on every XCD (256 / 3 ranges of three parts
    // are 33 workgroups for some XCD's 32 CUs, a second round: 65 us against 49 at
    // M = 768, d = 64, 16 users of 4K tokens); ranges of at least 128 (bf16 weights) or 64 tokens, below
    // which a range's partial costs more than its tiles (M = 512, d = 128, 2K tokens,
    // us: 16 ranges 23, 32 25, 63 27).  Shorter ones, down to a tile, where the mean user
    // is shorter: a range's users are done one after the other, a tile or more each
    // (512 users of 8 tokens, M = 256, d = 128: ranges of 128 93 us, of 32 45; 64 users of
    // 64: 128 23, 64 18).
    const int nw = agg_waves(M);
    const int64_t parts = (M + 32 * nw - 1) / (32 * nw);
    const int64_t least = std::clamp<int64_t>(HT / std::max<int64_t>(pairs, 1), kTileTokens, bf16_weights ? 128 : 64);
    return std::min(xcd_ranges(nw == 8 ? 1 : 2, parts), std::max<int64_t>(1, (HT + least - 1) / least));
}

hipError_t launch_split_fwd(const SplitFwdArgs& f, hipStream_t stream) {
    if (f.T == 0) return hipSuccess;
    hipError_t e;
    {
        ProfScope ps("split_lse", stream);
        e = f.d == 64 ? launch_lse<64>(f, stream) : launch_lse<128>(f, stream);
    }
    if (e != hipSuccess) return e;
    AggArgs a{f.K, f.V, f.P, f.offsets, f.lse, f.B, f.T, f.C, f.n_ranges, f.H, f.M, 1, f.scale, f.p_user, f.sketch,
              f.partials};
    ProfScope ps("split_agg", stream);
    const bool d64 = f.d == 64;
    if (f.bf16_weights) {
        if (agg_waves(f.M) == 4) return d64 ? launch_agg<64, 4, 1>(a, stream) : launch_agg<128, 4, 1>(a, stream);
        return d64 ? launch_agg<64, 8, 1>(a, stream) : launch_agg<128, 8, 1>(a, stream);
    }
    switch (agg_waves(f.M)) {
        case 2: return d64 ? launch_agg<64, 2, 3>(a, stream) : launch_agg<128, 2, 3>(a, stream);
        case 4: return d64 ? launch_agg<64, 4, 3>(a, stream) : launch_agg<128, 4, 3>(a, stream);
        default: return d64 ? launch_agg<64, 8, 3>(a, stream) : launch_agg<128, 8, 3>(a, stream);
    }
}

}  // namespace sa
