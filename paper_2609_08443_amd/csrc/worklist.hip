// Ragged scheduling: the work list of (user, head, token range) segments and
// the split-L merge of partial sketches.
//
// Users are ragged (section 4.4: fused kernel under ragged batching).  The
// (head, token) pairs are laid out head-major in one index space of length
// H*T and cut into equal ranges of C tokens, one range per workgroup, so every
// workgroup gets the same number of tokens whatever the length mix.  A (user,
// head) pair is cut at range boundaries into segments.  Because the softmax is
// taken over prototypes for each token separately (section 3.1, A sums to 1
// over prototypes), the sketch of a user is a plain sum over its tokens, so
// the partial sketches of a user cut across ranges merge by addition; there is
// no rescaling step as in a token-wise softmax.
#include <algorithm>
#include <type_traits>

#include "sa_internal.h"
#include "segments.h"

namespace sa {

namespace {

__device__ inline int64_t clamp64(int64_t x, int64_t lo, int64_t hi) {
    return x < lo ? lo : (x > hi ? hi : x);
}

// One workgroup: per 1024 pairs, their segment counts are scanned (wave shuffles, then
// the 16 wave totals), then all threads share the segments, each finding its
// segment's pair by binary search among the scanned starts.  With one thread writing
// all segments of a pair, a single user's list took up to 100 us (200 segments: 21).
__global__ __launch_bounds__(kWorklistThreads) void worklist_kernel(
    const int64_t* __restrict__ offsets, int64_t B, int64_t T, int32_t H, int64_t C,
    int64_t n_ranges, int32_t* __restrict__ items, int64_t max_items,
    int32_t* __restrict__ wg_start, int32_t* __restrict__ pair_start,
    int64_t* __restrict__ n_items) {
    constexpr int kWaves = kWorklistThreads / 64;
    __shared__ int64_t starts[kWorklistThreads + 1], wave_total[kWaves];
    __shared__ int32_t los[kWorklistThreads], his[kWorklistThreads];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (wg_start) {
        for (int64_t i = tid; i <= n_ranges; i += kWorklistThreads) wg_start[i] = -1;
    }
    const int64_t npairs = (int64_t)H * B;
    int64_t carry = 0;
    for (int64_t base = 0; base < npairs; base += kWorklistThreads) {
        const int64_t p = base + tid;
        int64_t n = 0, lo = 0, hi = 0;
        if (p < npairs) {
            const int64_t h = p / B, b = p % B;
            lo = clamp64(offsets[b], 0, T);
            hi = clamp64(offsets[b + 1], 0, T);
            if (hi > lo) n = (h * T + hi - 1) / C - (h * T + lo) / C + 1;
        }
        int64_t incl = n;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t v = __shfl_up((long long)incl, o, 64);
            if (lane >= o) incl += v;
        }
        if (lane == 63) wave_total[w] = incl;
        __syncthreads();   // (also: wg_start is cleared)
        for (int i = 0; i < w; ++i) incl += wave_total[i];
        starts[tid + 1] = incl;
        if (tid == 0) starts[0] = 0;
        los[tid] = (int32_t)lo;
        his[tid] = (int32_t)hi;
        if (p < npairs && pair_start) pair_start[p] = (int32_t)(carry + incl - n < max_items ? carry + incl - n : max_items);
        __syncthreads();
        const int64_t total = starts[kWorklistThreads];
        const int64_t here = total < max_items - carry ? total : max_items - carry;
        for (int64_t j = tid; j < here; j += kWorklistThreads) {
            int a = 0, z = kWorklistThreads - 1;   // the last pair with starts[pair] <= j
            while (a < z) {
                const int mid = (a + z + 1) >> 1;
                if (starts[mid] <= j) a = mid; else z = mid - 1;
            }
            const int64_t h = (base + a) / B, b = (base + a) % B, hT = h * T;
            const int64_t plo = los[a], phi = his[a], r = (hT + plo) / C + (j - starts[a]);
            const int64_t t0 = plo > r * C - hT ? plo : r * C - hT;
            const int64_t t1 = phi < (r + 1) * C - hT ? phi : (r + 1) * C - hT;
            const int64_t k = carry + j;
            int32_t* it = items + k * IT_WORDS;
            it[IT_B] = (int32_t)b;
            it[IT_H] = (int32_t)h;
            it[IT_T0] = (int32_t)t0;
            it[IT_T1] = (int32_t)t1;
            it[IT_RANGE] = (int32_t)r;
            it[IT_SPLIT] = starts[a + 1] - starts[a] > 1 ? 1 : 0;
            it[IT_PAIR_FIRST] = (int32_t)(carry + starts[a]);
            it[7] = 0;
            if (wg_start && r < n_ranges && hT + t0 == r * C) wg_start[r] = (int32_t)k;
        }
        carry += total;
        if (carry > max_items) carry = max_items;
        __syncthreads();   // the next pairs overwrite the scan
    }
    if (tid == 0) {
        if (pair_start) pair_start[npairs] = (int32_t)carry;
        if (wg_start) wg_start[n_ranges] = (int32_t)carry;
        *n_items = carry;
    }
}

// ---------------------------------------------------------------- split-L merge
// sketch[b,h] = the sum of a split pair's partials; zero for an empty one; a pair
// held by one range is written by its own workgroup.  Without offsets there is one
// user, of all T tokens.  A workgroup takes 1024 / G columns at a time: G groups of
// threads add G consecutive parts of the segments in token order, INFLIGHT loads in
// flight, and the groups' sums are added in order.
template <int G, int INFLIGHT>
__global__ __launch_bounds__(256) void merge_ranges_kernel(const int64_t* __restrict__ off, int64_t B, int64_t T,
                                                           int32_t H, int64_t C, int64_t n_ranges,
                                                           const float* __restrict__ partials, int64_t MD,
                                                           float* __restrict__ sketch) {
    constexpr int COLS = 256 / G;
    __shared__ float4 part[G > 1 ? 256 : 1];
    const int64_t h = blockIdx.x / B, b = blockIdx.x % B;
    const PairSlots ps(off ? seg_clamp(off[b], T) : 0, off ? seg_clamp(off[b + 1], T) : T, b, h, B, T, C, n_ranges);
    if (ps.count == 1) return;
    const int g = threadIdx.x / COLS;
    const int64_t per = (ps.count + G - 1) / G;
    const int64_t i1 = min((g + 1) * per, ps.count);
    for (int64_t c0 = (int64_t)blockIdx.y * 4 * COLS; c0 < MD; c0 += (int64_t)gridDim.y * 4 * COLS) {
        const int64_t idx = c0 + threadIdx.x % COLS * 4;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (idx < MD) {
            const float* p0 = partials + ps.first * MD + idx;   // slot 0; slot i at p + i MD
            const float* p = partials + ps.rest * MD + idx;
            auto add = [&](int64_t i, int n, auto whole) __attribute__((always_inline)) {
                const float* q = p + i * MD;
                float4 v[INFLIGHT];
#pragma unroll
                for (int u = 0; u < INFLIGHT; ++u)   // (past the end: the last again, not added)
                    v[u] = *reinterpret_cast<const float4*>(u == 0 && i == 0 ? p0 : q + (whole.value ? u : min(u, n - 1)) * MD);
#pragma unroll
                for (int u = 0; u < INFLIGHT; ++u) {
                    if (whole.value || u < n) {
                        acc.x += v[u].x;
                        acc.y += v[u].y;
                        acc.z += v[u].z;
                        acc.w += v[u].w;
                    }
                }
            };
            int64_t i = g * per;
            for (; i + INFLIGHT <= i1; i += INFLIGHT) add(i, INFLIGHT, std::true_type{});
            if (i < i1) add(i, (int)(i1 - i), std::false_type{});
        }
        if constexpr (G > 1) {
            __syncthreads();   // the previous columns are added up
            part[threadIdx.x] = acc;
            __syncthreads();
            if (g > 0) continue;
#pragma unroll
            for (int q = 1; q < G; ++q) {
                const float4 v = part[q * COLS + threadIdx.x];
                acc.x += v.x;
                acc.y += v.y;
                acc.z += v.z;
                acc.w += v.w;
            }
        }
        if (idx < MD) *reinterpret_cast<float4*>(sketch + (b * H + h) * MD + idx) = acc;
    }
}

}  // namespace

hipError_t launch_worklist(const int64_t* offsets, int64_t B, int64_t T, int32_t H, int64_t C,
                           int64_t n_ranges, int32_t* items, int64_t max_items,
                           int32_t* wg_start, int32_t* pair_start, int64_t* n_items,
                           hipStream_t stream) {
    hipLaunchKernelGGL(worklist_kernel, dim3(1), dim3(kWorklistThreads), 0, stream, offsets, B,
                       T, H, C, n_ranges, items, max_items, wg_start, pair_start, n_items);
    return hipGetLastError();
}

hipError_t launch_merge_ranges(const int64_t* offsets, int64_t B, int64_t T, int32_t H, int64_t C, int64_t n_ranges,
                               const float* partials, int64_t MD, float* sketch, hipStream_t stream) {
    const int64_t pairs = (int64_t)H * B;
    if (pairs == 0) return hipSuccess;
    // Eight groups where pairs have many segments (a column's loads then spread over
    // eight threads; one user of 2K tokens in 63 segments, M = 512, d = 128: the call 30.5
    // -> 27 us), one with fewer (64 pairs in 500 ranges: 94.5 us with one group, 97.5 with
    // eight: more workgroups, most of whose threads add one segment)
    // MD is a multiple of 4.
    const bool many = n_ranges >= 16 * pairs;
    const int64_t cols = many ? 128 : 1024;
    // A workgroup works out its pair's slots before, with many pairs, it mostly finds
    // nothing to add: about a microsecond, on 2,000 of them at once.  From 8K workgroups on
    // a pair's columns are dealt to fewer (2,048 users of 16 tokens, M = 512, d = 64: merge
    // with 65,536 workgroups 49 us, with 16,384 15, with 8,192 9), but not to less than
    // four, or the pairs with many segments wait for theirs (8 users of 90 - 2,500 tokens
    // and 16,000 of none, M = 128: the call 135 us, 199 with one).
    const int64_t most = std::max<int64_t>(4, kMergeWgs / pairs);
    const dim3 grid((unsigned)pairs, (unsigned)std::min<int64_t>((MD + cols - 1) / cols, most));
    // eight loads in flight a thread, three where four workgroups a CU have eight groups
    // each (one user of 100K tokens in 64 segments: M = 1024, d = 128, 1,024 workgroups, with
    // eight 11.7 us, with three 9.9; M = 128, d = 64, 64 of them, the call 26.8, with three 31.7)
    auto kern = !many ? merge_ranges_kernel<1, 8>
                : (int64_t)grid.x * grid.y >= 4 * (int64_t)device_cus() ? merge_ranges_kernel<8, 3> : merge_ranges_kernel<8, 8>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, offsets, B, T, H, C, n_ranges, partials, MD, sketch);
    return hipGetLastError();
}

}  // namespace sa
