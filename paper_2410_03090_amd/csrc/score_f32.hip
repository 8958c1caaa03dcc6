// Both scoring passes with fp32 logits on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 FMA sums, so
// nothing is rounded that the plain-arithmetic kernels keep): fp32 inputs, and bf16 ones whose window has no cut into
// 16-row blocks.  See score.hip for the two passes.
//
// What bounds them: the matrix instruction, 32 cycles each for 2048 flops (157 TFLOP/s over the chip).  A wave keeps 32
// tokens of keys in registers, in operand layout, and walks over the query rows in blocks of 16: 64 instructions, some
// 2000 cycles, per 8 KB of queries, which therefore come straight from the caches, one block ahead, without LDS.
// Contraction order: lane group kq holds features 16 s + 4 kq + e, so a 16-byte load is the operand of four instructions.
// Few heads are spread over the chip by their query rows (blockIdx), not by shorter token chunks: the partials of a
// chunk fill a region whose size callers have planned for.
// 8 heads of 1024 fp32 tokens, 128 rows: statistics 9 us and votes 7 us; 174 and 148 in the plain-arithmetic kernels.
#include "common.h"
#include "device_utils.h"
#include "score_stats_body.h"

namespace uncomp {

namespace {

constexpr int kWaveTokens = 32, kWgTokens = 4 * kWaveTokens;

__device__ __forceinline__ f32x4_t load4(const float* p) { return *reinterpret_cast<const f32x4_t*>(p); }
__device__ __forceinline__ f32x4_t load4(const bf16_bits* p) {
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    return f32x4_t{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                   __uint_as_float(v.y & 0xffff0000u)};
}

// a row's 16-byte pieces for lane group kq
template <typename T, int DD>
__device__ __forceinline__ void load_row(f32x4_t (&dst)[DD / 16], const T* row, int kq) {
#pragma unroll
    for (int s = 0; s < DD / 16; ++s) dst[s] = load4(row + 16 * s + 4 * kq);
}

template <int S>
__device__ __forceinline__ f32x4_t dot_block(const f32x4_t (&a)[S], const f32x4_t (&b)[S]) {
    f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][e], b[s][e], c, 0, 0, 0);
    return c;
}

}  // namespace

// Pass 1.  Workgroup: one token chunk and `blocks_per` 16-row blocks of one KV head; its four waves take 32 tokens in
// turn.  Keys are operand A, queries operand B: a lane holds query row lane%16 and tokens 4 kq + v.  The running
// (maximum, sum) of the rows live in LDS, a set per wave (all lanes of a row write the same pair), folded at the end.
template <typename T, int DD>
__global__ __launch_bounds__(256) void score_stats_f32_kernel(const T* __restrict__ Q, const T* __restrict__ K, int H,
                                                              int R, int N, int w, int64_t ks_b, int64_t ks_h,
                                                              int64_t ks_t, int n_chunks, int chunk, int n_split,
                                                              int blocks_per, float2* __restrict__ stats) {
    constexpr int S = DD / 16;
    extern __shared__ float2 run[];                                 // [4 waves][16 * blocks_per]
    const int sp = blockIdx.x % n_split, bc = blockIdx.x / n_split;
    const int bh = bc / n_chunks, c = bc % n_chunks;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, n = lane & 15, kq = lane >> 4;
    const int row0 = 16 * blocks_per * sp, n_rows = min(16 * blocks_per, R - row0), n_blk = (n_rows + 15) / 16;
    const T* Kh = K + (bh / H) * ks_b + (bh % H) * ks_h;
    const T* Qh = Q + ((int64_t)bh * R + row0) * DD;
    const float scale2 = kLog2e * rsqrtf((float)DD);
    const int P = N - w;
    float2* mine = run + wv * 16 * blocks_per;
    for (int i = lane; i < 16 * blocks_per; i += 64) run[wv * 16 * blocks_per + i] = make_float2(kNoLogit, 0.f);
    __syncthreads();
    const int t_end = min(N, (c + 1) * chunk);
    for (int t0 = c * chunk + kWaveTokens * wv; t0 < t_end; t0 += kWgTokens) {
        f32x4_t k0[S], k1[S], qa[S], qb[S];
        load_row<T, DD>(k0, Kh + (int64_t)min(t0 + n, N - 1) * ks_t, kq);
        load_row<T, DD>(k1, Kh + (int64_t)min(t0 + 16 + n, N - 1) * ks_t, kq);
        auto load_q = [&](f32x4_t (&q)[S], int blk) {               // clamped: rows past the end are never stored
            load_row<T, DD>(q, Qh + (int64_t)min(16 * blk + n, n_rows - 1) * DD, kq);
        };
        auto body = [&](const f32x4_t (&q)[S], int blk) {
            const f32x4_t c0 = dot_block<S>(k0, q), c1 = dot_block<S>(k1, q);
            const int last = min(t_end - 1, P + (row0 + 16 * blk + n) % w);      // last token of this tile's chunk that the row sees
            float s[8], mx = -INFINITY;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const int t = t0 + 16 * (v >> 2) + 4 * kq + (v & 3);
                s[v] = t <= last ? (v < 4 ? c0[v & 3] : c1[v & 3]) * scale2 : -INFINITY;
                mx = fmaxf(mx, s[v]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float2 old = mine[16 * blk + n];
            const float m = fmaxf(old.x, mx);
            float sum = 0.f;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                const int t = t0 + 16 * (v >> 2) + 4 * kq + (v & 3);
                sum += t <= last ? exp2f(s[v] - m) : 0.f;
            }
            sum += __shfl_xor(sum, 16, 64);
            sum += __shfl_xor(sum, 32, 64);
            if (t0 <= last) mine[16 * blk + n] = make_float2(m, old.y * (old.y == 0.f ? 0.f : exp2f(old.x - m)) + sum);
        };
        load_q(qa, 0);
        for (int blk = 0; blk < n_blk; blk += 2) {
            load_q(qb, blk + 1);
            body(qa, blk);
            if (blk + 1 < n_blk) {
                load_q(qa, blk + 2);
                body(qb, blk + 1);
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < n_rows; i += 256) {
        float m = -INFINITY, l = 0.f;
        for (int x = 0; x < 4; ++x) m = fmaxf(m, run[x * 16 * blocks_per + i].x);
        for (int x = 0; x < 4; ++x) {
            const float2 v = run[x * 16 * blocks_per + i];
            if (v.y != 0.f) l += v.y * exp2f(v.x - m);               // a wave without a token for this row holds a sum of zero
        }
        stats[((int64_t)bh * n_chunks + c) * R + row0 + i] = make_float2(m, l);
    }
}

// Pass 2.  Workgroup: 128 prefix tokens and `g_per` query heads (of w rows) of one KV head; waves run on their own.
// Queries are operand A, keys operand B: a lane holds token lane%16 and rows 4 kq + v, so the sum over a head's rows is
// additions within the lane and two exchanges at the end.  pair: windows of eight, where a 16-row block is two heads
// (G and w are then given as G / 2 and 16) and one exchange completes each.
template <typename T, int DD>
__global__ __launch_bounds__(256) void score_vote_f32_kernel(const T* __restrict__ Q, const T* __restrict__ K,
                                                             const float* __restrict__ lse, int H, int G, int P, int w,
                                                             int pair, int64_t ks_b, int64_t ks_h, int64_t ks_t,
                                                             int n_tiles, int n_split, int g_per,
                                                             float* __restrict__ vote) {
    constexpr int S = DD / 16;
    const int sp = blockIdx.x % n_split, bt = blockIdx.x / n_split;
    const int bh = bt / n_tiles, tile = bt % n_tiles;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, n = lane & 15, kq = lane >> 4;
    const int t0 = tile * kWgTokens + kWaveTokens * wv;
    if (t0 >= P) return;                                            // no barrier below
    const int g0 = sp * g_per, n_g = min(g_per, G - g0), nb = (w + 15) / 16, n_it = n_g * nb;
    const T* Kh = K + (bh / H) * ks_b + (bh % H) * ks_h;
    const T* Qh = Q + ((int64_t)bh * G + g0) * w * DD;
    const float* lh = lse + ((int64_t)bh * G + g0) * w;
    const float scale2 = kLog2e * rsqrtf((float)DD);
    f32x4_t k0[S], k1[S], qa[S], qb[S], la, lb;
    load_row<T, DD>(k0, Kh + (int64_t)min(t0 + n, P - 1) * ks_t, kq);
    load_row<T, DD>(k1, Kh + (int64_t)min(t0 + 16 + n, P - 1) * ks_t, kq);
    float v0 = 0.f, v1 = 0.f;
    int g_load = 0, b_load = 0, g_use = 0, b_use = 0;               // head and block of the next load and the next product
    auto load_q = [&](f32x4_t (&q)[S], f32x4_t& l) {
        const int g = min(g_load, n_g - 1);                          // past the last head: loaded once more, never used
        load_row<T, DD>(q, Qh + ((int64_t)g * w + min(16 * b_load + n, w - 1)) * DD, kq);
#pragma unroll
        for (int v = 0; v < 4; ++v) l[v] = lh[g * w + min(16 * b_load + 4 * kq + v, w - 1)];
        if (++b_load == nb) {
            b_load = 0;
            ++g_load;
        }
    };
    auto body = [&](const f32x4_t (&q)[S], const f32x4_t& l) {
        const f32x4_t c0 = dot_block<S>(q, k0), c1 = dot_block<S>(q, k1);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool live = 16 * b_use + 4 * kq + v < w;           // rows past the head's last one
            const float p0 = exp2f(fmaf(c0[v], scale2, -l[v])), p1 = exp2f(fmaf(c1[v], scale2, -l[v]));
            v0 += live ? p0 : 0.f;
            v1 += live ? p1 : 0.f;
        }
        if (++b_use == nb) {
            v0 += __shfl_xor(v0, 16, 64);
            v1 += __shfl_xor(v1, 16, 64);
            if (!pair) {
                v0 += __shfl_xor(v0, 32, 64);
                v1 += __shfl_xor(v1, 32, 64);
            }
            const int g = g0 + g_use, G_out = pair ? 2 * G : G, g_out = pair ? 2 * g + (kq >> 1) : g;
            if (kq == 0 || (pair && kq == 2)) {
                float* o = vote + ((int64_t)bh * G_out + g_out) * P + t0 + n;
                if (t0 + n < P) o[0] = v0;
                if (t0 + 16 + n < P) o[16] = v1;
            }
            v0 = v1 = 0.f;
            b_use = 0;
            ++g_use;
        }
    };
    load_q(qa, la);
    for (int it = 0; it < n_it; it += 2) {
        load_q(qb, lb);
        body(qa, la);
        if (it + 1 < n_it) {
            load_q(qa, la);
            body(qb, lb);
        }
    }
}

// Workgroups that the row split aims at: two per CU.  8 heads of 1024 tokens, 128 rows make 32 workgroups of the
// statistics and 64 of the votes without it.
constexpr int64_t kF32Workgroups = 512;

// stats[(bh, chunk)][R]; returns the number of chunks in *n_parts, at most max_parts.
template <typename T>
hipError_t launch_stats_f32(const T* Q, const T* K, int BH, int H, int R, int N, int w, const int64_t ks[3], int max_parts,
                            float2* stats, int* n_parts, hipStream_t s, int D) {
    int nc = (N + kWgTokens - 1) / kWgTokens;
    if (nc > max_parts) nc = max_parts;
    const int chunk = ((N + nc - 1) / nc + kWgTokens - 1) / kWgTokens * kWgTokens;
    nc = (N + chunk - 1) / chunk;
    const int n_blk = (R + 15) / 16;
    int64_t split = (kF32Workgroups + (int64_t)BH * nc - 1) / ((int64_t)BH * nc);
    if (split > n_blk) split = n_blk;
    const int per = (n_blk + (int)split - 1) / (int)split, n_split = (n_blk + per - 1) / per;
    auto kern = D == 64 ? score_stats_f32_kernel<T, 64> : score_stats_f32_kernel<T, kD>;
    kern<<<dim3((unsigned)((int64_t)BH * nc * n_split)), dim3(256), (size_t)4 * 16 * per * sizeof(float2), s>>>(
        Q, K, H, R, N, w, ks[0], ks[1], ks[2], nc, chunk, n_split, per, stats);
    *n_parts = nc;
    return hipGetLastError();
}

template <typename T>
hipError_t launch_vote_f32(const T* Q, const T* K, const float* lse, int BH, int H, int G, int N, int w, const int64_t ks[3],
                           float* vote, hipStream_t s, int D) {
    const int P = N - w, n_tiles = (P + kWgTokens - 1) / kWgTokens;
    const int pair = w == 8 && G % 2 == 0;
    const int Ge = pair ? G / 2 : G, we = pair ? 16 : w;
    int64_t split = (kF32Workgroups + (int64_t)BH * n_tiles - 1) / ((int64_t)BH * n_tiles);
    if (split > Ge) split = Ge;
    const int per = (Ge + (int)split - 1) / (int)split, n_split = (Ge + per - 1) / per;
    auto kern = D == 64 ? score_vote_f32_kernel<T, 64> : score_vote_f32_kernel<T, kD>;
    kern<<<dim3((unsigned)((int64_t)BH * n_tiles * n_split)), dim3(256), 0, s>>>(
        Q, K, lse, H, Ge, P, we, pair, ks[0], ks[1], ks[2], n_tiles, n_split, per, vote);
    return hipGetLastError();
}

#define UNCOMP_SCORE_F32(T)                                                                                               \
    template hipError_t launch_stats_f32<T>(const T*, const T*, int, int, int, int, int, const int64_t[3], int, float2*, \
                                            int*, hipStream_t, int);                                                     \
    template hipError_t launch_vote_f32<T>(const T*, const T*, const float*, int, int, int, int, int, const int64_t[3],  \
                                           float*, hipStream_t, int)
UNCOMP_SCORE_F32(float);
UNCOMP_SCORE_F32(bf16_bits);
#undef UNCOMP_SCORE_F32

}  // namespace uncomp
