// Top-k of a few long rows of scores, split over many workgroups (Sec. 3.3.2: the hidden-state eviction
// keeps the layer's highest-scoring tokens out of one row of N scores per batch entry, far fewer rows than
// the chip has CUs; Sec. 3.3.3 defines the per-row selection).  Same result as select_kernel: the k largest
// scores, ties at the threshold by position, indices ascending, then the w window positions.
//
// A row is cut into chunks of 2048 positions, one workgroup each, and the exact k-th largest key is found by a
// most-significant-digit radix select on the order-preserving 32-bit image of the float with digits of 11, 11 and 10 bits at
// fixed positions.  Workgroups only meet between kernels:
//   zero     clears the three histograms of every row;
//   digit<p> resolves the histogram of digit p-1 (every workgroup for itself, workgroup 0 records the result), then counts
//            digit p of its chunk's keys that match the digits found so far in LDS and adds the non-empty counters to the
//            row's histogram;
//   count    resolves the last digit: threshold and number of equal keys to take; counts the chunk's keys above / equal to it;
//   write    sums the counts of the chunks before its own and writes its kept positions in order.
// Integer atomics only: the result does not depend on the order in which workgroups run.
//
// Six launches of 3 to 4 us each, whatever the scores: 8 rows of 40009 scores 21 us, 22 to 24 where they are all but an outlier
// within 1/50 of an octave, mostly zero or all equal; 131008 scores 22 to 31, one row of a million 28 to 43.  (Three launches,
// with bins that cut a known range of the keys and a list of the keys of the threshold's bin, took 18 us where 40009 scores are
// spread and 140 to 160 where they crowd into one bin: then every workgroup searched the row.  With the bin cut once more by
// the chunks' workgroups that was 38.  Four launches with a histogram per chunk instead of atomics took 22.)
#include "common.h"
#include "device_utils.h"

namespace uncomp {

namespace {

constexpr int kWThreads = 256;
constexpr int kWPer = 8;                         // consecutive positions per thread
constexpr int kWStep = kWThreads * kWPer;        // positions per workgroup: its chunk
constexpr int kWBins = 2048;                     // eight per thread
constexpr int kWStates = 4;                      // state after resolving 0, 1, 2, 3 digits

struct WideState {
    uint32_t prefix;         // digits found so far (in place)
    uint32_t remaining;      // rank of the wanted key among the keys that share the prefix (1 = largest)
};

struct WideSmem {
    uint32_t hist[kWBins];
    uint32_t wsum[kWThreads / 64];
    uint32_t bcast[2];
};

__device__ __forceinline__ int digit_shift(int pass) { return pass == 0 ? 21 : (pass == 1 ? 10 : 0); }
// mask of the digits above digit `pass`
__device__ __forceinline__ uint32_t prefix_mask(int pass) { return pass == 0 ? 0u : (pass == 1 ? 0xffe00000u : 0xfffffc00u); }

__device__ __forceinline__ uint32_t wide_wave_incl_scan(uint32_t v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t n = __shfl_up(v, o, 64);
        if (lane >= o) v += n;
    }
    return v;
}

// exclusive prefix over the workgroup and the total; ends with a barrier
__device__ __forceinline__ uint32_t wide_excl_scan(uint32_t v, WideSmem& sm, uint32_t* total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t inc = wide_wave_incl_scan(v, lane);
    if (lane == 63) sm.wsum[wv] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kWThreads / 64; ++i) {
        const uint32_t s = sm.wsum[i];
        if (i < wv) base += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

// the row's budget as the number of prefix positions to keep
__device__ __forceinline__ int prefix_budget(const int32_t* budget, int budget_stride, int g, int N, int w, int cap,
                                             int* bud_out) {
    int bud = budget[(int64_t)g * budget_stride];
    const int hi = N < cap ? N : cap;
    bud = bud < w ? w : bud;
    bud = bud > hi ? hi : bud;
    *bud_out = bud;
    return bud - w;
}

// keys of this thread's kWPer consecutive positions (0 past the end of the row: callers skip those)
__device__ __forceinline__ void load_keys(const float* sc, int P, int j0, uint32_t (&key)[kWPer]) {
    typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));     // rows start on any float
    if (j0 + kWPer <= P) {
        const f32x4u_t a = *reinterpret_cast<const f32x4u_t*>(sc + j0), b = *reinterpret_cast<const f32x4u_t*>(sc + j0 + 4);
        key[0] = order_key(a.x); key[1] = order_key(a.y); key[2] = order_key(a.z); key[3] = order_key(a.w);
        key[4] = order_key(b.x); key[5] = order_key(b.y); key[6] = order_key(b.z); key[7] = order_key(b.w);
    } else {
#pragma unroll
        for (int e = 0; e < kWPer; ++e) key[e] = j0 + e < P ? order_key(sc[j0 + e]) : 0u;
    }
}

// The bin (0 .. kWBins - 1) that holds the `remaining`-th largest key, given this thread's counts c[u] of bins
// kWBins - 1 - 8 tid - u; the rank inside it comes back in *rank_in.  Every thread gets the same answers.
__device__ __forceinline__ uint32_t pick_bin(const uint32_t (&c)[8], uint32_t remaining, WideSmem& sm, uint32_t* rank_in) {
    const int tid = threadIdx.x;
    uint32_t mine = 0, total;
#pragma unroll
    for (int u = 0; u < 8; ++u) mine += c[u];
    if (tid == 0) {                                                // what a rank beyond the keys counted would leave behind
        sm.bcast[0] = 0u;
        sm.bcast[1] = 1u;
    }
    uint32_t before = wide_excl_scan(mine, sm, &total);            // keys in higher bins
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if (before < remaining && remaining <= before + c[u]) {
            sm.bcast[0] = (uint32_t)(kWBins - 1 - 8 * tid - u);
            sm.bcast[1] = remaining - before;
        }
        before += c[u];
    }
    __syncthreads();
    const uint32_t bin = sm.bcast[0];
    *rank_in = sm.bcast[1];
    __syncthreads();
    return bin;
}

// bit e of x: position j0 + e has a key above the threshold; of y: equal to it
__device__ __forceinline__ uint2 compare_keys(const uint32_t (&key)[kWPer], int j0, int P, uint32_t thr) {
    uint32_t above = 0, equal = 0;
#pragma unroll
    for (int e = 0; e < kWPer; ++e) {
        if (j0 + e < P) {
            above |= key[e] > thr ? 1u << e : 0u;
            equal |= key[e] == thr ? 1u << e : 0u;
        }
    }
    return make_uint2(above, equal);
}
// both counts in one word: at most 2048 of either in a workgroup, no carry between the halves
__device__ __forceinline__ uint32_t both_counts(uint2 m) { return (uint32_t)__builtin_popcount(m.x) << 16 | (uint32_t)__builtin_popcount(m.y); }

// The kept ones of this thread's positions: all above the threshold and the first need_eq equal ones; g_before / e_before: above
// and equal ones before the thread's first position.  Writes stay inside the k slots.
__device__ __forceinline__ void place_keys(uint2 m, uint32_t g_before, uint32_t e_before, uint32_t need_eq, int k,
                                           int j0, int32_t* idx) {
#pragma unroll
    for (int e = 0; e < kWPer; ++e) {
        if (m.x & (1u << e)) {
            const uint32_t pos = g_before + (e_before < need_eq ? e_before : need_eq);
            if (pos < (uint32_t)k) idx[pos] = j0 + e;
            ++g_before;
        } else if (m.y & (1u << e)) {
            const uint32_t pos = g_before + e_before;
            if (e_before < need_eq && pos < (uint32_t)k) idx[pos] = j0 + e;
            ++e_before;
        }
    }
}

struct WideBufs {
    uint32_t* hist;          // [n_groups][3][kWBins]
    WideState* state;        // [n_groups][kWStates]
    uint32_t* counts;        // [n_groups][n_wg][2]
    size_t bytes;
};

__host__ __device__ inline WideBufs wide_bufs(char* ws, int n_groups, int n_wg) {
    WideBufs b;
    b.hist = reinterpret_cast<uint32_t*>(ws);
    b.state = reinterpret_cast<WideState*>(b.hist + (size_t)n_groups * 3 * kWBins);
    b.counts = reinterpret_cast<uint32_t*>(b.state + (size_t)n_groups * kWStates);
    b.bytes = reinterpret_cast<char*>(b.counts + (size_t)n_groups * n_wg * 2) - ws;
    return b;
}

// the state after digit `pass`, from its finished histogram (the last digit's upper half stays empty)
__device__ __forceinline__ WideState resolve_digit(const uint32_t* __restrict__ hist, int pass, WideState st, WideSmem& sm) {
    uint32_t c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) c[u] = hist[kWBins - 1 - 8 * threadIdx.x - u];
    st.prefix |= pick_bin(c, st.remaining, sm, &st.remaining) << digit_shift(pass);
    return st;
}

}  // namespace

__global__ __launch_bounds__(kWThreads) void selw_zero_kernel(uint32_t* __restrict__ hist, int n) {
    const int i = blockIdx.x * kWThreads + threadIdx.x;
    if (i < n) hist[i] = 0u;
}

template <int PASS>
__global__ __launch_bounds__(kWThreads) void selw_digit_kernel(const float* __restrict__ score,
                                                               const int32_t* __restrict__ budget, int budget_stride, int N,
                                                               int w, int cap, char* __restrict__ ws) {
    __shared__ WideSmem sm;
    const int g = blockIdx.y, wg = blockIdx.x, tid = threadIdx.x, P = N - w, j0 = wg * kWStep + tid * kWPer;
    const WideBufs b = wide_bufs(ws, gridDim.y, gridDim.x);
    uint32_t* hist = b.hist + (size_t)g * 3 * kWBins;
    WideState* state = b.state + (size_t)g * kWStates;
    int bud;
    const int k = prefix_budget(budget, budget_stride, g, N, w, cap, &bud);
    if (k <= 0 || k >= P) return;                                  // nothing to search for: the write kernel handles it
    uint32_t key[kWPer];                                           // on their way while the digit before is found
    load_keys(score + (int64_t)g * P, P, j0, key);
    WideState st{0u, (uint32_t)k};
    if (PASS > 0) st = resolve_digit(hist + (PASS - 1) * kWBins, PASS - 1, state[PASS - 1], sm);
    if (wg == 0 && tid == 0) state[PASS] = st;
    for (int i = tid; i < kWBins; i += kWThreads) sm.hist[i] = 0u;
    __syncthreads();
    const uint32_t pm = prefix_mask(PASS), digits = PASS == 2 ? 1023u : 2047u;
#pragma unroll
    for (int e = 0; e < kWPer; ++e)
        if (j0 + e < P && (key[e] & pm) == (st.prefix & pm)) atomicAdd(&sm.hist[(key[e] >> digit_shift(PASS)) & digits], 1u);
    __syncthreads();
    for (int i = tid; i <= (int)digits; i += kWThreads) {
        const uint32_t c = sm.hist[i];
        if (c != 0u) atomicAdd(&hist[PASS * kWBins + i], c);
    }
}

__global__ __launch_bounds__(kWThreads) void selw_count_kernel(const float* __restrict__ score,
                                                               const int32_t* __restrict__ budget, int budget_stride, int N,
                                                               int w, int cap, char* __restrict__ ws) {
    __shared__ WideSmem sm;
    const int g = blockIdx.y, wg = blockIdx.x, tid = threadIdx.x, P = N - w, j0 = wg * kWStep + tid * kWPer;
    const WideBufs b = wide_bufs(ws, gridDim.y, gridDim.x);
    WideState* state = b.state + (size_t)g * kWStates;
    int bud;
    const int k = prefix_budget(budget, budget_stride, g, N, w, cap, &bud);
    if (k <= 0 || k >= P) return;
    uint32_t key[kWPer], total;
    load_keys(score + (int64_t)g * P, P, j0, key);
    const WideState st = resolve_digit(b.hist + ((size_t)g * 3 + 2) * kWBins, 2, state[2], sm);
    if (wg == 0 && tid == 0) state[3] = st;                        // prefix = the threshold key, remaining = equal keys to take
    wide_excl_scan(both_counts(compare_keys(key, j0, P, st.prefix)), sm, &total);
    if (tid == 0) {
        b.counts[((size_t)g * gridDim.x + wg) * 2] = total >> 16;
        b.counts[((size_t)g * gridDim.x + wg) * 2 + 1] = total & 0xffffu;
    }
}

__global__ __launch_bounds__(kWThreads) void selw_write_kernel(const float* __restrict__ score,
                                                               const int32_t* __restrict__ budget, int budget_stride, int N,
                                                               int w, int cap, char* __restrict__ ws,
                                                               int32_t* __restrict__ idx_out, int32_t* __restrict__ len_out) {
    __shared__ WideSmem sm;
    const int g = blockIdx.y, wg = blockIdx.x, tid = threadIdx.x, P = N - w, j0 = wg * kWStep + tid * kWPer;
    const WideBufs b = wide_bufs(ws, gridDim.y, gridDim.x);
    int32_t* idx = idx_out + (int64_t)g * cap;
    int bud;
    const int k = prefix_budget(budget, budget_stride, g, N, w, cap, &bud);
    if (wg == 0) {
        for (int i = tid; i < w; i += kWThreads) idx[k + i] = P + i;
        if (tid == 0) len_out[g] = bud;
    }
    if (k <= 0) return;
    if (k >= P) {                                                 // every prefix position is kept
#pragma unroll
        for (int e = 0; e < kWPer; ++e)
            if (j0 + e < P) idx[j0 + e] = j0 + e;
        return;
    }
    uint32_t key[kWPer], g_tot, e_tot, total;
    load_keys(score + (int64_t)g * P, P, j0, key);
    const WideState st = b.state[(size_t)g * kWStates + 3];
    uint32_t gsum = 0, esum = 0;                                   // kept / equal keys in the chunks before this one
    for (int i = tid; i < wg; i += kWThreads) {
        gsum += b.counts[((size_t)g * gridDim.x + i) * 2];
        esum += b.counts[((size_t)g * gridDim.x + i) * 2 + 1];
    }
    wide_excl_scan(gsum, sm, &g_tot);
    wide_excl_scan(esum, sm, &e_tot);
    const uint2 kept = compare_keys(key, j0, P, st.prefix);
    const uint32_t ex = wide_excl_scan(both_counts(kept), sm, &total);
    place_keys(kept, g_tot + (ex >> 16), e_tot + (ex & 0xffffu), st.remaining, k, j0, idx);
}

SelectWidePlan plan_select_wide(int n_groups, int N, int w) {
    SelectWidePlan p;
    const int64_t P = N - w > 0 ? N - w : 1;
    p.n_wg = (int)((P + kWStep - 1) / kWStep);
    p.bytes = align_up(wide_bufs(nullptr, n_groups, p.n_wg).bytes, 256);
    return p;
}

hipError_t launch_select_rows_wide(const float* score, const int32_t* budget, int budget_stride, int n_groups, int N,
                                   int w, int cap, const SelectWidePlan& p, char* ws, int32_t* idx_out, int32_t* len_out,
                                   const Env& env) {
    hipStream_t s = env.s;
    const dim3 grid((unsigned)p.n_wg, (unsigned)n_groups), block(kWThreads);
    const int n_hist = n_groups * 3 * kWBins;
    env.begin("select");
    selw_zero_kernel<<<dim3((unsigned)((n_hist + kWThreads - 1) / kWThreads)), block, 0, s>>>(reinterpret_cast<uint32_t*>(ws), n_hist);
    selw_digit_kernel<0><<<grid, block, 0, s>>>(score, budget, budget_stride, N, w, cap, ws);
    selw_digit_kernel<1><<<grid, block, 0, s>>>(score, budget, budget_stride, N, w, cap, ws);
    selw_digit_kernel<2><<<grid, block, 0, s>>>(score, budget, budget_stride, N, w, cap, ws);
    selw_count_kernel<<<grid, block, 0, s>>>(score, budget, budget_stride, N, w, cap, ws);
    selw_write_kernel<<<grid, block, 0, s>>>(score, budget, budget_stride, N, w, cap, ws, idx_out, len_out);
    env.end();
    return hipGetLastError();
}

}  // namespace uncomp
