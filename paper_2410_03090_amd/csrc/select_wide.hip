// Top-k of a few long rows of scores, split over many workgroups (Sec. 3.3.2: the hidden-state eviction
// keeps the layer's highest-scoring tokens out of one row of N scores per batch entry, far fewer rows than
// the chip has CUs; Sec. 3.3.3 defines the per-row selection).  Same result as select_kernel: the k largest
// scores, ties at the threshold by position, indices ascending, then the w window positions.
//
// A row is cut into at most 256 chunks of whole 2048 positions, one workgroup each.  What a call costs is its number of
// dependent launches (4 us each before anything is in them), so there are three:
//   hist   counts the chunk's keys in 2048 bins that cut the row's range of keys (order-preserving 32-bit images of the
//          scores) into equal pieces, and leaves them as the chunk's own histogram;
//   list   adds up the row's histograms (every workgroup for itself) and finds the bin that holds the k-th largest key;
//          counts the chunk's keys in higher bins and lists its keys in that bin, a few dozen in a row;
//   write  collects the row's lists, finds the exact threshold among them and the chunk's place in the output, and
//          writes the chunk's kept positions in order.
// The range comes from the kernel that wrote the scores; where it is not known a fourth launch finds it.  Bins only have
// to rise with the key, so a range that does not fit the scores costs time, not results.  A chunk's list holds a quarter
// of its positions: with more keys in the bin (thousands of equal scores) the write kernel searches the row itself.
// 8 rows of 40009 scores: 5 + 7 + 7 us (30 with six launches: three digits, each a histogram with global atomics).
// The result does not depend on the order in which workgroups run.
#include "common.h"
#include "device_utils.h"

namespace uncomp {

namespace {

constexpr int kWThreads = 256;
constexpr int kWPer = 8;                         // consecutive positions per thread and step
constexpr int kWStep = kWThreads * kWPer;        // positions per workgroup and step
constexpr int kWBins = 2048;                     // eight per thread
constexpr int kWMaxChunks = kWThreads;           // a thread per chunk of the row
constexpr int kWCand = 4096;                     // keys of the threshold's bin that the write kernel holds in LDS
constexpr int kWRankAll = 1024;                  // up to so many are ranked by comparing each with all

struct WideState {           // what the list kernel found out about a row
    uint32_t lo;             // bin of a key: (key - lo) >> shift, clamped
    int32_t shift;
    uint32_t bin;            // the bin of the k-th largest key
    uint32_t remaining;      // its rank among the keys of that bin (1 = largest)
};

struct WideSmem {
    uint32_t hist[kWBins];
    uint32_t wsum[kWThreads / 64];
    uint32_t bcast[2];
};

__device__ __forceinline__ uint32_t bin_of(uint32_t key, uint32_t lo, int shift) {
    const uint32_t b = key > lo ? (key - lo) >> shift : 0u;
    return b < (uint32_t)kWBins ? b : (uint32_t)(kWBins - 1);
}

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

// keys of this thread's kWPer consecutive positions (0 past `end`: callers skip those)
__device__ __forceinline__ void load_keys(const float* sc, int P, int end, int j0, uint32_t (&key)[kWPer]) {
    const bool aligned = (P & 3) == 0 && (reinterpret_cast<uintptr_t>(sc) & 15u) == 0;   // every row then starts on 16 bytes
    if (aligned && j0 + kWPer <= end) {
        const float4 a = *reinterpret_cast<const float4*>(sc + j0);
        const float4 b = *reinterpret_cast<const float4*>(sc + j0 + 4);
        key[0] = order_key(a.x); key[1] = order_key(a.y); key[2] = order_key(a.z); key[3] = order_key(a.w);
        key[4] = order_key(b.x); key[5] = order_key(b.y); key[6] = order_key(b.z); key[7] = order_key(b.w);
    } else {
#pragma unroll
        for (int e = 0; e < kWPer; ++e) key[e] = j0 + e < end ? order_key(sc[j0 + e]) : 0u;
    }
}

// f(position, key) for the positions [begin, end) of a row, in no order; first: this thread's keys of the first step
template <typename F>
__device__ __forceinline__ void each_key(const float* sc, int P, int begin, int end, const uint32_t (&first)[kWPer], F&& f) {
    int j0 = begin + threadIdx.x * kWPer;
#pragma unroll
    for (int e = 0; e < kWPer; ++e)
        if (j0 + e < end) f(j0 + e, first[e]);
    for (j0 += kWStep; j0 < end; j0 += kWStep) {
        uint32_t key[kWPer];
        load_keys(sc, P, end, j0, key);
#pragma unroll
        for (int e = 0; e < kWPer; ++e)
            if (j0 + e < end) f(j0 + e, key[e]);
    }
}
template <typename F>
__device__ __forceinline__ void each_key(const float* sc, int P, int begin, int end, F&& f) {
    uint32_t first[kWPer];
    load_keys(sc, P, end, begin + threadIdx.x * kWPer, first);
    each_key(sc, P, begin, end, first, f);
}

// The bin (0 .. kWBins - 1) that holds the `remaining`-th largest key, given this thread's eight counts c[u] of bins
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

struct WideBufs {
    uint32_t* range;         // [n_groups][n_wg][2], for rows whose range is not known
    uint16_t* hist;          // [n_groups][n_wg][kWBins]
    uint32_t* list;          // [n_groups][n_wg][list_cap]
    uint32_t* info;          // [n_groups][n_wg][2]: keys in higher bins, keys in the bin
    WideState* state;        // [n_groups]
    size_t bytes;
};

__host__ __device__ inline WideBufs wide_bufs(char* ws, int n_groups, int n_wg, int list_cap) {
    WideBufs b;
    const size_t n = (size_t)n_groups * n_wg;
    b.hist = reinterpret_cast<uint16_t*>(ws);
    b.state = reinterpret_cast<WideState*>(ws + n * kWBins * sizeof(uint16_t));
    b.range = reinterpret_cast<uint32_t*>(b.state + n_groups);
    b.info = b.range + 2 * n;
    b.list = b.info + 2 * n;
    b.bytes = reinterpret_cast<char*>(b.list + n * list_cap) - ws;
    return b;
}

}  // namespace

// smallest and largest key of every chunk
__global__ __launch_bounds__(kWThreads) void selw_range_kernel(const float* __restrict__ score, int P, int chunk,
                                                               uint32_t* __restrict__ range) {
    __shared__ uint32_t part[kWThreads / 64][2];
    const int g = blockIdx.y, wg = blockIdx.x, tid = threadIdx.x;
    uint32_t lo = 0xffffffffu, hi = 0u;
    each_key(score + (int64_t)g * P, P, wg * chunk, min(P, (wg + 1) * chunk), [&](int, uint32_t key) {
        lo = min(lo, key);
        hi = max(hi, key);
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor(lo, o, 64));
        hi = max(hi, (uint32_t)__shfl_xor(hi, o, 64));
    }
    if ((tid & 63) == 0) {
        part[tid >> 6][0] = lo;
        part[tid >> 6][1] = hi;
    }
    __syncthreads();
    if (tid == 0) {
        for (int i = 1; i < kWThreads / 64; ++i) {
            lo = min(lo, part[i][0]);
            hi = max(hi, part[i][1]);
        }
        uint32_t* out = range + ((int64_t)g * gridDim.x + wg) * 2;
        out[0] = lo;
        out[1] = hi;
    }
}

// range: n_range pairs (smallest, largest key) per row that together cover it
__global__ __launch_bounds__(kWThreads) void selw_hist_kernel(const float* __restrict__ score,
                                                              const int32_t* __restrict__ budget, int budget_stride, int N,
                                                              int w, int cap, int chunk, int list_cap,
                                                              const uint32_t* __restrict__ range, int n_range,
                                                              char* __restrict__ ws) {
    __shared__ __align__(16) WideSmem sm;
    __shared__ uint32_t part[kWThreads / 64][2];
    const int g = blockIdx.y, wg = blockIdx.x, tid = threadIdx.x;
    const int P = N - w, begin = wg * chunk, end = min(P, begin + chunk);
    const WideBufs b = wide_bufs(ws, gridDim.y, gridDim.x, list_cap);
    int bud;
    const int k = prefix_budget(budget, budget_stride, g, N, w, cap, &bud);
    if (k <= 0 || k >= P) return;                                  // nothing to search for: the write kernel handles it
    uint32_t first[kWPer];                                         // on their way while the range is found
    load_keys(score + (int64_t)g * P, P, end, begin + tid * kWPer, first);
    uint32_t lo = 0xffffffffu, hi = 0u;
    const uint2* rg = reinterpret_cast<const uint2*>(range) + (int64_t)g * n_range;
    for (int i = tid; i < n_range; i += kWThreads) {
        const uint2 r = rg[i];
        lo = min(lo, r.x);
        hi = max(hi, r.y);
    }
    for (int i = tid; i < kWBins; i += kWThreads) sm.hist[i] = 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor(lo, o, 64));
        hi = max(hi, (uint32_t)__shfl_xor(hi, o, 64));
    }
    if ((tid & 63) == 0) {
        part[tid >> 6][0] = lo;
        part[tid >> 6][1] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kWThreads / 64; ++i) {
        lo = min(lo, part[i][0]);
        hi = max(hi, part[i][1]);
    }
    const uint32_t span = hi > lo ? hi - lo : 0u;
    const int shift = max(0, 32 - (span ? __clz(span) : 32) - 11);
    if (wg == 0 && tid == 0) {
        b.state[g].lo = lo;
        b.state[g].shift = shift;
    }
    each_key(score + (int64_t)g * P, P, begin, end, first, [&](int, uint32_t key) { atomicAdd(&sm.hist[bin_of(key, lo, shift)], 1u); });
    __syncthreads();
    uint32_t pk[4];                                                // a chunk has fewer than 65536 positions
#pragma unroll
    for (int u = 0; u < 4; ++u) pk[u] = sm.hist[8 * tid + 2 * u] | (sm.hist[8 * tid + 2 * u + 1] << 16);
    *reinterpret_cast<uint4*>(b.hist + ((int64_t)g * gridDim.x + wg) * kWBins + 8 * tid) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
}

__global__ __launch_bounds__(kWThreads) void selw_list_kernel(const float* __restrict__ score,
                                                              const int32_t* __restrict__ budget, int budget_stride, int N,
                                                              int w, int cap, int chunk, int list_cap, char* __restrict__ ws) {
    __shared__ WideSmem sm;
    __shared__ uint32_t n_list;
    const int g = blockIdx.y, wg = blockIdx.x, tid = threadIdx.x, n_wg = gridDim.x;
    const int P = N - w, begin = wg * chunk, end = min(P, begin + chunk);
    const WideBufs b = wide_bufs(ws, gridDim.y, n_wg, list_cap);
    int bud;
    const int k = prefix_budget(budget, budget_stride, g, N, w, cap, &bud);
    if (k <= 0 || k >= P) return;
    uint32_t first[kWPer];                                         // on their way while the bin is found
    load_keys(score + (int64_t)g * P, P, end, begin + tid * kWPer, first);
    const uint32_t lo = b.state[g].lo;
    const int shift = b.state[g].shift;
    uint32_t c[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};              // bins kWBins - 1 - 8 tid and down
    const uint16_t* hg = b.hist + (int64_t)g * n_wg * kWBins + (kWBins - 8 - 8 * tid);
    constexpr int kLoads = 16;
    for (int x0 = 0; x0 < n_wg; x0 += kLoads) {
        uint4 v[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; ++u) v[u] = *reinterpret_cast<const uint4*>(hg + (int64_t)min(x0 + u, n_wg - 1) * kWBins);
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            if (x0 + u < n_wg) {
                c[7] += v[u].x & 0xffffu; c[6] += v[u].x >> 16;
                c[5] += v[u].y & 0xffffu; c[4] += v[u].y >> 16;
                c[3] += v[u].z & 0xffffu; c[2] += v[u].z >> 16;
                c[1] += v[u].w & 0xffffu; c[0] += v[u].w >> 16;
            }
        }
    }
    if (tid == 0) n_list = 0u;
    uint32_t rank;
    const uint32_t bin = pick_bin(c, (uint32_t)k, sm, &rank);
    if (wg == 0 && tid == 0) {
        b.state[g].bin = bin;
        b.state[g].remaining = rank;
    }
    uint32_t above = 0;
    uint32_t* list = b.list + ((int64_t)g * n_wg + wg) * list_cap;
    each_key(score + (int64_t)g * P, P, begin, end, first, [&](int, uint32_t key) {
        const uint32_t kb = bin_of(key, lo, shift);
        above += kb > bin ? 1u : 0u;
        if (kb == bin) {
            const uint32_t at = atomicAdd(&n_list, 1u);
            if (at < (uint32_t)list_cap) list[at] = key;
        }
    });
    uint32_t total;
    wide_excl_scan(above, sm, &total);
    if (tid == 0) {
        uint32_t* info = b.info + ((int64_t)g * n_wg + wg) * 2;
        info[0] = total;
        info[1] = n_list;
    }
}

__global__ __launch_bounds__(kWThreads) void selw_write_kernel(const float* __restrict__ score,
                                                               const int32_t* __restrict__ budget, int budget_stride, int N,
                                                               int w, int cap, int chunk, int list_cap, char* __restrict__ ws,
                                                               int32_t* __restrict__ idx_out, int32_t* __restrict__ len_out) {
    __shared__ WideSmem sm;
    __shared__ __align__(16) uint32_t cand[kWCand];
    __shared__ uint32_t at_s[kWMaxChunks + 1], thr_s[2];
    const int g = blockIdx.y, wg = blockIdx.x, tid = threadIdx.x, n_wg = gridDim.x;
    const int P = N - w, begin = wg * chunk, end = min(P, begin + chunk);
    const WideBufs b = wide_bufs(ws, gridDim.y, n_wg, list_cap);
    const float* sc = score + (int64_t)g * P;
    int32_t* idx = idx_out + (int64_t)g * cap;
    int bud;
    const int k = prefix_budget(budget, budget_stride, g, N, w, cap, &bud);
    if (wg == 0) {
        for (int i = tid; i < w; i += kWThreads) idx[k + i] = P + i;
        if (tid == 0) len_out[g] = bud;
    }
    if (k <= 0) return;
    if (k >= P) {                                                 // every prefix position is kept
        for (int j = begin + tid; j < end; j += kWThreads) idx[j] = j;
        return;
    }
    uint32_t key[kWPer];                                           // on their way while the threshold is found
    load_keys(sc, P, end, begin + tid * kWPer, key);
    const WideState st = b.state[g];
    // Where the chunks' lists start and what is kept before this chunk: every wave for itself, four chunks a lane.
    const int lane = tid & 63;
    uint32_t at[4], n_cand = 0, n_above = 0;
    bool over = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int c = 4 * lane + u;
        at[u] = n_cand;
        if (c < n_wg) {
            const uint2 v = reinterpret_cast<const uint2*>(b.info)[(int64_t)g * n_wg + c];
            n_cand += v.y;
            n_above += c < wg ? v.x : 0u;
            over |= v.y > (uint32_t)list_cap;
        }
    }
    const uint32_t incl = wide_wave_incl_scan(n_cand, lane), before_me = incl - n_cand;
    n_cand = __builtin_amdgcn_readlane(incl, 63);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n_above += __shfl_xor(n_above, o, 64);
    const bool listed = !__any(over) && n_cand <= (uint32_t)kWCand;
    auto in_bin = [&](uint32_t key) { return bin_of(key, st.lo, st.shift) == st.bin; };
    uint32_t thr, need_eq;                                         // threshold, equal keys to take
    if (listed) {
        if (tid < 64) {
#pragma unroll
            for (int u = 0; u < 4; ++u) at_s[4 * lane + u] = before_me + at[u];
            if (tid == 0) at_s[kWMaxChunks] = n_cand;
        }
        __syncthreads();
        for (int c = tid >> 3; c < n_wg; c += kWThreads / 8) {     // eight threads per list
            const uint32_t a0 = at_s[c], n = at_s[c + 1] - a0;
            const uint32_t* list = b.list + ((int64_t)g * n_wg + c) * list_cap;
            for (uint32_t i = tid & 7; i < n; i += 8) cand[a0 + i] = list[i];
        }
        const uint32_t n4 = (n_cand + 3u) & ~3u;
        if (tid < (int)(n4 - n_cand)) cand[n_cand + tid] = 0u;
        __syncthreads();
    }
    if (listed && n_cand <= (uint32_t)kWRankAll) {
        const uint32_t n4 = (n_cand + 3u) & ~3u;
        for (uint32_t i = tid; i < n_cand; i += kWThreads) {
            const uint32_t mine = cand[i];
            uint32_t gt = 0, ge = 0;
            for (uint32_t j = 0; j < n4; j += 4) {
                const uint4 v = *reinterpret_cast<const uint4*>(&cand[j]);
                gt += (v.x > mine ? 1u : 0u) + (v.y > mine ? 1u : 0u) + (v.z > mine ? 1u : 0u) + (v.w > mine ? 1u : 0u);
                ge += (v.x >= mine ? 1u : 0u) + (v.y >= mine ? 1u : 0u) + (v.z >= mine ? 1u : 0u) + (v.w >= mine ? 1u : 0u);
            }
            if (mine == 0u) ge -= n4 - n_cand;                     // the padding
            if (gt < st.remaining && st.remaining <= ge) {         // all that find this hold the same key
                thr_s[0] = mine;
                thr_s[1] = st.remaining - gt;
            }
        }
        __syncthreads();
        thr = thr_s[0];
        need_eq = thr_s[1];
    } else {
        // three digits of 11, 11 and 10 bits from the top, over the lists or over the whole row
        uint32_t prefix = 0u, remaining = st.remaining;
        for (int pass = 0; pass < 3; ++pass) {
            const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
            const uint32_t mask = pass == 0 ? 0u : (pass == 1 ? 0xffe00000u : 0xfffffc00u), digits = pass == 2 ? 1023u : 2047u;
            for (int i = tid; i < kWBins; i += kWThreads) sm.hist[i] = 0u;
            __syncthreads();
            auto count = [&](int, uint32_t key) {
                if (((key ^ prefix) & mask) == 0u) atomicAdd(&sm.hist[(key >> shift) & digits], 1u);
            };
            if (listed) {
                for (uint32_t i = tid; i < n_cand; i += kWThreads) count(0, cand[i]);
            } else {
                each_key(sc, P, 0, P, [&](int j, uint32_t key) {
                    if (in_bin(key)) count(j, key);
                });
            }
            __syncthreads();
            uint32_t c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = sm.hist[kWBins - 1 - 8 * tid - u];
            prefix |= pick_bin(c, remaining, sm, &remaining) << shift;
        }
        thr = prefix;
        need_eq = remaining;
    }
    uint32_t g_before, e_before;                                   // above / equal to the threshold before this chunk
    if (listed) {
        uint32_t both = 0;                                         // at most 4096 of either
        for (uint32_t i = tid; i < at_s[wg]; i += kWThreads) both += cand[i] > thr ? 0x10000u : (cand[i] == thr ? 1u : 0u);
        wide_excl_scan(both, sm, &both);
        g_before = both >> 16;
        e_before = both & 0xffffu;
    } else {
        uint32_t gsum = 0, esum = 0;
        each_key(sc, P, 0, begin, [&](int, uint32_t x) {
            gsum += in_bin(x) && x > thr ? 1u : 0u;
            esum += x == thr ? 1u : 0u;
        });
        wide_excl_scan(gsum, sm, &g_before);
        wide_excl_scan(esum, sm, &e_before);
    }
    g_before += n_above;
    for (int base = begin; base < end; base += kWStep) {
        const int j0 = base + tid * kWPer;
        if (base > begin) load_keys(sc, P, end, j0, key);
        uint32_t gtm = 0, eqm = 0;
#pragma unroll
        for (int e = 0; e < kWPer; ++e) {
            if (j0 + e < end) {
                if (key[e] > thr) gtm |= 1u << e;
                else if (key[e] == thr) eqm |= 1u << e;
            }
        }
        uint32_t total;                                            // at most 2048 of either: no carry between the halves
        const uint32_t ex = wide_excl_scan(((uint32_t)__builtin_popcount(gtm) << 16) | (uint32_t)__builtin_popcount(eqm), sm, &total);
        uint32_t gb = g_before + (ex >> 16), eb = e_before + (ex & 0xffffu);
        // everything above the threshold and the first need_eq equal keys; writes stay inside the k slots
#pragma unroll
        for (int e = 0; e < kWPer; ++e) {
            if (gtm & (1u << e)) {
                const uint32_t pos = gb + (eb < need_eq ? eb : need_eq);
                if (pos < (uint32_t)k) idx[pos] = j0 + e;
                ++gb;
            } else if (eqm & (1u << e)) {
                const uint32_t pos = gb + eb;
                if (eb < need_eq && pos < (uint32_t)k) idx[pos] = j0 + e;
                ++eb;
            }
        }
        g_before += total >> 16;
        e_before += total & 0xffffu;
    }
}

// Chunks of 2048 positions up to 32 of them, then as many steps longer as keep to 32, so that the list kernel adds up no more
// than 32 histograms; beyond 28 steps (histograms of 16 bits) the chunks become more again.
SelectWidePlan plan_select_wide(int n_groups, int N, int w) {
    SelectWidePlan p;
    constexpr int kMaxSteps = 28;
    const int64_t P = N - w > 0 ? N - w : 1, steps = (P + kWStep - 1) / kWStep;
    int64_t per = (steps + 31) / 32;
    if (per > kMaxSteps) per = kMaxSteps;
    p.chunk = (int)per * kWStep;
    p.list_cap = p.chunk / 4;
    const int64_t n_wg = (steps + per - 1) / per;
    p.fits = n_wg <= kWMaxChunks;
    p.n_wg = p.fits ? (int)n_wg : 0;
    p.bytes = align_up(wide_bufs(nullptr, n_groups, p.n_wg, p.list_cap).bytes, 256);
    return p;
}

hipError_t launch_select_rows_wide(const float* score, const int32_t* budget, int budget_stride, int n_groups, int N,
                                   int w, int cap, const SelectWidePlan& p, char* ws, const uint32_t* range, int n_range,
                                   int32_t* idx_out, int32_t* len_out, const Env& env) {
    hipStream_t s = env.s;
    const dim3 grid((unsigned)p.n_wg, (unsigned)n_groups), block(kWThreads);
    env.begin("select");
    if (range == nullptr) {
        uint32_t* own = wide_bufs(ws, n_groups, p.n_wg, p.list_cap).range;
        selw_range_kernel<<<grid, block, 0, s>>>(score, N - w, p.chunk, own);
        range = own;
        n_range = p.n_wg;
    }
    selw_hist_kernel<<<grid, block, 0, s>>>(score, budget, budget_stride, N, w, cap, p.chunk, p.list_cap, range, n_range, ws);
    selw_list_kernel<<<grid, block, 0, s>>>(score, budget, budget_stride, N, w, cap, p.chunk, p.list_cap, ws);
    selw_write_kernel<<<grid, block, 0, s>>>(score, budget, budget_stride, N, w, cap, p.chunk, p.list_cap, ws, idx_out, len_out);
    env.end();
    return hipGetLastError();
}

}  // namespace uncomp
