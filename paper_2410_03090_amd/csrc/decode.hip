// Decode-time eviction (Sec. 3.3.3 "Dynamic KV Cache Eviction", last sentence; Alg. 2
// "Decoding").  One generated token per call: the token joins every head's compacted cache,
// the head's G query rows attend to the joined cache, every entry's cumulative score grows
// by the attention it received, and a head that is over its budget gives up its
// lowest-scoring entry outside the recent window.
//
// The evicted entry's slot receives the new token, so nothing is moved: slot order is free,
// idx names each slot.
//
// bf16 caches of many heads take decode_head_kernel, one workgroup per head, and so do fewer heads of short caches.  A few
// heads of long caches take decode_split_kernel: several workgroups per head, the last of which merges.  The rest (heads
// between the two, more than 8 query heads per KV head, caches whose probabilities do not fit in LDS) takes two kernels.
// decode_attend_wave_kernel: every wave
// owns 64, 128 or 256 consecutive rows of one head and runs on its own (no workgroup barrier): keys stream straight into
// MFMA operand layout, the logits stay in registers, the wave's softmax (its own maximum and sum) goes through LDS to
// the lanes that stream the value rows, and the wave leaves (maximum, sum, unnormalised output, unnormalised
// probabilities) in the workspace.
// decode_update_kernel: one workgroup per head merges the waves' partials into the output,
// turns the stored probabilities into each row's share, updates the cumulative scores,
// finds the row to give up and places the new token.
//
// fp32 caches (and the plain-ALU switch) take decode_step_kernel: one workgroup per head
// does all of it with the step's probabilities held in LDS, rows read 16 lanes to a row.
#include "common.h"
#include "device_utils.h"

namespace uncomp {

namespace {

constexpr int kDecodeThreads = 512;
constexpr int kRowsInFlight = 4;

// Sum over the 16 lanes of a DPP row; every lane of the row receives the total.
__device__ __forceinline__ float row16_sum(float v) {
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x128, 0xF, 0xF, false));  // row_ror:8
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x124, 0xF, 0xF, false));  // row_ror:4
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x122, 0xF, 0xF, false));  // row_ror:2
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x121, 0xF, 0xF, false));  // row_ror:1
    return v;
}

// Monotone map of a float onto unsigned integers (smaller float -> smaller key).
__device__ __forceinline__ uint32_t ascending_key(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Four floats at any float's address: the caller's attention output need not be aligned to more than a float.
typedef float f32x4_any_t __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        unsigned long long other = __shfl_xor(v, o, 64);
        v = other < v ? other : v;
    }
    return v;
}

__device__ __forceinline__ void copy8(const bf16_bits* src, bf16_bits* dst) {
    *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
}
__device__ __forceinline__ void copy8(const float* src, float* dst) {
    reinterpret_cast<uint4*>(dst)[0] = reinterpret_cast<const uint4*>(src)[0];
    reinterpret_cast<uint4*>(dst)[1] = reinterpret_cast<const uint4*>(src)[1];
}

}  // namespace

__global__ __launch_bounds__(256) void decode_init_kernel(const float* __restrict__ score,
                                                          const int32_t* __restrict__ idx,
                                                          const int32_t* __restrict__ len, int n_heads,
                                                          int P, int cap, float* __restrict__ cum) {
    const int64_t total = (int64_t)n_heads * cap;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int h = (int)(e / cap), r = (int)(e - (int64_t)h * cap);
        float c = 0.f;
        if (r < len[h]) {
            const int j = idx[e];
            if (j >= 0 && j < P) c = score[(int64_t)h * P + j];
        }
        cum[e] = c;
    }
}

// GT: compile-time bound on the query heads per KV head (G <= GT).  S: row stride of the
// probability table in LDS (floats), S >= cap + 1.
template <typename T, int GT>
__global__ __launch_bounds__(kDecodeThreads) void decode_step_kernel(
    const T* __restrict__ q, const T* __restrict__ k_new, const T* __restrict__ v_new, int G,
    const int32_t* __restrict__ pos, const int32_t* __restrict__ budget, int w, int cap, T* Kc, T* Vc,
    int32_t* idx, float* cum, int32_t* len, float* __restrict__ out, int32_t* __restrict__ evicted, int S) {
    constexpr int NT = kDecodeThreads, NW = NT / 64, RPI = NT / 16, U = kRowsInFlight;
    extern __shared__ float dyn[];                  // prob[G][S]; later the per-wave output partials
    __shared__ float red[NW][GT];
    __shared__ unsigned long long wave_best[NW];
    __shared__ int victim_slot;
    __shared__ float new_cum_s;

    const int h = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sub = lane & 15, rg = tid >> 4;
    int n = len[h];
    n = n < 0 ? 0 : (n > cap ? cap : n);
    const int n1 = n + 1;                           // entries the queries attend to
    T* Kh = Kc + (int64_t)h * cap * kD;
    T* Vh = Vc + (int64_t)h * cap * kD;
    int32_t* idxh = idx + (int64_t)h * cap;
    float* cumh = cum + (int64_t)h * cap;
    const T* kn = k_new + (int64_t)h * kD;
    const T* vn = v_new + (int64_t)h * kD;
    if (tid == 0) victim_slot = -1;

    // ---- logits in the exp2 domain: s_gr = (q_g . k_r) / sqrt(D) * log2(e) -----------------
    {
        float qf[GT][8];
        const float qs = 0.08838834764831845f * 1.4426950408889634f;
#pragma unroll
        for (int g = 0; g < GT; ++g) {
            if (g < G) {
                load8(q + ((int64_t)h * G + g) * kD + 8 * sub, qf[g]);
#pragma unroll
                for (int e = 0; e < 8; ++e) qf[g][e] *= qs;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) qf[g][e] = 0.f;
            }
        }
        for (int r0 = 0; r0 < n1; r0 += RPI * U) {
            float kv[U][8];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = r0 + u * RPI + rg;
                const int rc = r < n ? r : n;       // rows past the end re-read the new token
                const T* src = rc < n ? Kh + (int64_t)rc * kD : kn;
                load8(src + 8 * sub, kv[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = r0 + u * RPI + rg;
#pragma unroll
                for (int g = 0; g < GT; ++g) {
                    float d = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) d = fmaf(qf[g][e], kv[u][e], d);
                    d = row16_sum(d);
                    if (sub == 0 && r < n1 && g < G) dyn[g * S + r] = d;
                }
            }
        }
    }
    __syncthreads();

    // ---- softmax over the n1 entries, per query head ---------------------------------------
    float m[GT], inv[GT];
    {
#pragma unroll
        for (int g = 0; g < GT; ++g) m[g] = -INFINITY;
        for (int r = tid; r < n1; r += NT)
#pragma unroll
            for (int g = 0; g < GT; ++g)
                if (g < G) m[g] = fmaxf(m[g], dyn[g * S + r]);
#pragma unroll
        for (int g = 0; g < GT; ++g) {
            float v = wave_max(m[g]);
            if (lane == 0) red[wave][g] = v;
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < GT; ++g) {
            float v = red[0][g];
#pragma unroll
            for (int x = 1; x < NW; ++x) v = fmaxf(v, red[x][g]);
            m[g] = v;
        }
        __syncthreads();
        float l[GT];
#pragma unroll
        for (int g = 0; g < GT; ++g) l[g] = 0.f;
        for (int r = tid; r < n1; r += NT)
#pragma unroll
            for (int g = 0; g < GT; ++g)
                if (g < G) {
                    const float e = exp2f(dyn[g * S + r] - m[g]);
                    dyn[g * S + r] = e;
                    l[g] += e;
                }
#pragma unroll
        for (int g = 0; g < GT; ++g) {
            float v = wave_sum(l[g]);
            if (lane == 0) red[wave][g] = v;
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < GT; ++g) {
            float v = red[0][g];
#pragma unroll
            for (int x = 1; x < NW; ++x) v += red[x][g];
            inv[g] = 1.0f / v;
        }
    }

    // ---- cumulative scores, candidate for eviction -------------------------------------------
    const int posh = pos[h];
    int b = budget[h];
    b = b < w ? w : b;
    b = b > cap ? cap : b;
    const bool over = n1 > b;
    unsigned long long best = ~0ull;
    for (int r = tid; r < n1; r += NT) {
        float inc = 0.f;
#pragma unroll
        for (int g = 0; g < GT; ++g)
            if (g < G) {
                const float pr = dyn[g * S + r] * inv[g];
                dyn[g * S + r] = pr;
                inc += pr;
            }
        if (r < n) {
            const float c = cumh[r] + inc;
            cumh[r] = c;
            const int id = idxh[r];
            if (id <= posh - w) {
                const unsigned long long key = ((unsigned long long)ascending_key(c) << 32) | (uint32_t)id;
                best = key < best ? key : best;
            }
        } else {
            new_cum_s = inc;
        }
    }
    best = wave_min_u64(best);
    if (lane == 0) wave_best[wave] = best;
    __syncthreads();
    best = wave_best[0];
#pragma unroll
    for (int x = 1; x < NW; ++x) best = wave_best[x] < best ? wave_best[x] : best;
    if (over && best != ~0ull) {
        const int want = (int)(uint32_t)(best & 0xffffffffull);
        for (int r = tid; r < n; r += NT)
            if (idxh[r] == want) victim_slot = r;
    }

    // ---- attention output: out_g = sum_r p_gr v_r ---------------------------------------------
    float acc[GT][8];
#pragma unroll
    for (int g = 0; g < GT; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
    for (int r0 = 0; r0 < n1; r0 += RPI * U) {
        float vv[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * RPI + rg;
            const int rc = r < n ? r : n;
            const T* src = rc < n ? Vh + (int64_t)rc * kD : vn;
            load8(src + 8 * sub, vv[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * RPI + rg;
            const int rc = r < n ? r : n;
            const float live = r < n1 ? 1.f : 0.f;
#pragma unroll
            for (int g = 0; g < GT; ++g) {
                if (g < G) {
                    const float pr = dyn[g * S + rc] * live;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[g][e] = fmaf(pr, vv[u][e], acc[g][e]);
                }
            }
        }
    }
#pragma unroll
    for (int g = 0; g < GT; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float v = acc[g][e];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            acc[g][e] = v;
        }
    __syncthreads();                                // every wave is done with the probabilities
    if (lane < 16) {
#pragma unroll
        for (int g = 0; g < GT; ++g)
            if (g < G) {
#pragma unroll
                for (int e = 0; e < 8; ++e) dyn[(wave * G + g) * kD + 8 * sub + e] = acc[g][e];
            }
    }
    __syncthreads();
    for (int o = tid; o < G * kD; o += NT) {
        float v = 0.f;
#pragma unroll
        for (int x = 0; x < NW; ++x) v += dyn[x * G * kD + o];
        out[(int64_t)h * G * kD + o] = v;
    }

    // ---- the new token takes the freed slot, or the next free one --------------------------
    int slot = n, ev = -1;
    if (over) {
        slot = victim_slot;
        if (slot >= 0) {
            ev = idxh[slot];
        } else if (n < cap) {
            slot = n;                               // nothing may leave: grow if there is room
        } else {
            ev = -2;                                // no room and nothing may leave: token dropped
        }
    }
    __syncthreads();                                // idxh[slot] read by all before it is replaced
    if (slot >= 0) {
        if (tid < 16) copy8(kn + 8 * tid, Kh + (int64_t)slot * kD + 8 * tid);
        else if (tid < 32) copy8(vn + 8 * (tid - 16), Vh + (int64_t)slot * kD + 8 * (tid - 16));
        else if (tid == 32) {
            idxh[slot] = posh;
            cumh[slot] = new_cum_s;
        }
    }
    if (tid == 0) {
        len[h] = (slot == n) ? n + 1 : n;
        if (evicted != nullptr) evicted[h] = ev;
    }
}


// ---- bf16: wave-per-part attention pass ---------------------------------------------------
// A wave owns WR = 64, 128 or 256 consecutive rows of one head: the fewer, the fewer waves the launch would otherwise
// have for the chip; 256 when there are plenty (half the partial results to write and merge).

// Workspace per head: prob [s_rows][GT] (unnormalised, relative to the owning wave's maximum),
// ml [np_max][GT][2] (maximum in the exp2 domain, sum), acc [np_max][GT][128].
template <int GT, int WR>
__global__ __launch_bounds__(256) void decode_attend_wave_kernel(
    const bf16_bits* __restrict__ q, const bf16_bits* __restrict__ k_new, const bf16_bits* __restrict__ v_new,
    int n_heads, int G, int cap, const bf16_bits* __restrict__ Kc, const bf16_bits* __restrict__ Vc,
    const int32_t* __restrict__ len, int np_max, int s_rows, float* __restrict__ ws_p, float* __restrict__ ws_ml,
    float* __restrict__ ws_acc) {
    constexpr int kTiles = WR / 16;
    extern __shared__ __align__(16) float pl_all[];                 // [4 waves][WR][GT]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int c16 = lane & 15, j = lane >> 4;
    const int wid = blockIdx.x * 4 + wv;
    const int h = wid / np_max, part = wid - h * np_max;
    if (h >= n_heads) return;
    int n = len[h];
    n = n < 0 ? 0 : (n > cap ? cap : n);
    const int n1 = n + 1;
    const int row0 = part * WR;
    if (row0 >= n1) return;                                         // waves run on their own: no barrier below
    const int n_t = min(kTiles, (n1 - row0 + 15) >> 4);
    float* pl = pl_all + wv * WR * GT;
    const bf16_bits* Kh = Kc + (int64_t)h * cap * kD;
    const bf16_bits* Vh = Vc + (int64_t)h * cap * kD;
    const bf16_bits* kn = k_new + (int64_t)h * kD;
    const bf16_bits* vn = v_new + (int64_t)h * kD;

    // queries as the B operand: column c16 = query head, zero beyond G
    bf16x8_t qb[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (c16 < G) v = *reinterpret_cast<const uint4*>(q + ((int64_t)h * G + c16) * kD + 32 * ks + 8 * j);
        qb[ks] = __builtin_bit_cast(bf16x8_t, v);
    }
    // rows past the end re-read the new token (clamped, never predicated: straight-line loads
    // keep exact counts of the loads in flight); what they produce is masked below
    auto load_k = [&](uint4 (&dst)[4], int t) {
        const int r = row0 + 16 * t + c16;
        const bf16_bits* src = (r < n ? Kh + (int64_t)r * kD : kn) + 8 * j;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dst[ks] = *reinterpret_cast<const uint4*>(src + 32 * ks);
    };
    auto load_v = [&](uint4 (&dst)[4], int t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = row0 + 16 * t + 4 * u + j;
            const bf16_bits* src = (r < n ? Vh + (int64_t)r * kD : vn) + 8 * c16;
            dst[u] = *reinterpret_cast<const uint4*>(src);
        }
    };

    // ---- pass 1: logits of the wave's rows; lane holds query head c16, rows 16t + 4j + v ----
    // Short waves (kAll) have all their keys and values in flight at once: with few waves on the chip their time is
    // that of the round trips to memory (8 heads of 2048 rows: 8.4 us, two tiles ahead 9.6).
    constexpr bool kAll = WR == 64 && GT <= 8;
    constexpr int kSlots = kAll ? kTiles : 2;
    f32x4_t s[kTiles];
    uint4 kt[kSlots][4], vt[kSlots][4];
    auto dots = [&](const uint4 (&x)[4], int t) {
        f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x[ks]), qb[ks], c, 0, 0, 0);
        s[t] = c;
    };
    if constexpr (kAll) {
#pragma unroll
        for (int t = 0; t < kTiles; ++t) load_k(kt[t], t);
#pragma unroll
        for (int t = 0; t < kTiles; ++t) load_v(vt[t], t);
#pragma unroll
        for (int t = 0; t < kTiles; ++t) dots(kt[t], t);
    } else {
        load_k(kt[0], 0);
#pragma unroll
        for (int t = 0; t < kTiles; t += 2) {
            if (t < n_t) {
                load_k(kt[1], t + 1);
                dots(kt[0], t);
            }
            if (t + 1 < n_t) {
                load_k(kt[0], t + 2);
                dots(kt[1], t + 1);
            }
        }
        load_v(vt[0], 0);                                           // under way during the softmax arithmetic
    }

    const float qs = 0.08838834764831845f * 1.4426950408889634f;    // 1/sqrt(128) * log2(e)
    float mx = -INFINITY;
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
        if (t < n_t) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const bool live = row0 + 16 * t + 4 * j + v < n1;
                s[t][v] = live ? s[t][v] * qs : -INFINITY;
                mx = fmaxf(mx, s[t][v]);
            }
        }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));                         // row0 < n1: at least one live row
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < kTiles; ++t)
        if (t < n_t) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float e = exp2f(s[t][v] - mx);
                sum += e;
                if (c16 < GT) pl[(16 * t + 4 * j + v) * GT + c16] = e;
            }
        }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    const int64_t hp = (int64_t)h * np_max + part;
    if (j == 0 && c16 < G) {
        ws_ml[(hp * GT + c16) * 2 + 0] = mx;
        ws_ml[(hp * GT + c16) * 2 + 1] = sum;
    }
    // LDS traffic of one wave is processed in issue order; the fences keep the compiler from
    // moving the reads below over the writes above
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    // the wave's probabilities go to the workspace as they lie in LDS (rows of GT floats)
    {
        float* dst = ws_p + ((int64_t)h * s_rows + row0) * GT;
        const int n_f4 = n_t * 16 * GT / 4;
        for (int i = lane; i < n_f4; i += 64)
            reinterpret_cast<float4*>(dst)[i] = reinterpret_cast<const float4*>(pl)[i];
    }

    // ---- pass 2: unnormalised output; lane holds features 8*c16.., rows 16t + 4u + j -----------
    float acc[GT][8];
#pragma unroll
    for (int g = 0; g < GT; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
    auto weigh = [&](const uint4 (&vt)[4], int t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float vf[8];
            const uint32_t wds[4] = {vt[u].x, vt[u].y, vt[u].z, vt[u].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                vf[2 * i] = __uint_as_float(wds[i] << 16);
                vf[2 * i + 1] = __uint_as_float(wds[i] & 0xffff0000u);
            }
            const float* prow = pl + (16 * t + 4 * u + j) * GT;
#pragma unroll
            for (int g4 = 0; g4 < GT; g4 += 4) {
                const float4 pr = *reinterpret_cast<const float4*>(prow + g4);
                const float prs[4] = {pr.x, pr.y, pr.z, pr.w};
#pragma unroll
                for (int gg = 0; gg < 4; ++gg)
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[g4 + gg][e] = fmaf(prs[gg], vf[e], acc[g4 + gg][e]);
            }
        }
    };
    if constexpr (kAll) {
#pragma unroll
        for (int t = 0; t < kTiles; ++t)
            if (t < n_t) weigh(vt[t], t);
    } else {
#pragma unroll
        for (int t = 0; t < kTiles; t += 2) {
            if (t < n_t) {
                load_v(vt[1], t + 1);
                weigh(vt[0], t);
            }
            if (t + 1 < n_t) {
                load_v(vt[0], t + 2);
                weigh(vt[1], t + 1);
            }
        }
    }
    // sum over the four lane rows; lane row j keeps query head g4 + {0,2,1,3}[j]
    const int gsel = ((j & 1) << 1) | (j >> 1);
#pragma unroll
    for (int g4 = 0; g4 < GT; g4 += 4) {
        float tot[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            tot[e] = reduce4_over_rows(acc[g4][e], acc[g4 + 1][e], acc[g4 + 2][e], acc[g4 + 3][e]);
        float* dst = ws_acc + (hp * GT + g4 + gsel) * kD + 8 * c16;
        reinterpret_cast<float4*>(dst)[0] = make_float4(tot[0], tot[1], tot[2], tot[3]);
        reinterpret_cast<float4*>(dst)[1] = make_float4(tot[4], tot[5], tot[6], tot[7]);
    }
}

// The new token takes the slot of the entry that leaves, or the next free one.  Called by the whole workgroup.
// victim: slot of the entry outside the window with the lowest score, -1 if none; victim_id: its position.
__device__ __forceinline__ void place_token(const bf16_bits* kn, const bf16_bits* vn, bf16_bits* Kh, bf16_bits* Vh,
                                            int32_t* idxh, float* cumh, int32_t* len, int32_t* evicted, int tid, int n,
                                            int cap, bool over, int victim, int victim_id, int posh, float new_cum) {
    int slot = n, ev = -1;
    if (over) {
        slot = victim;
        if (slot >= 0) {
            ev = victim_id;
        } else if (n < cap) {
            slot = n;                               // nothing may leave: grow if there is room
        } else {
            ev = -2;                                // no room and nothing may leave: token dropped
        }
    }
    if (slot >= 0) {
        if (tid < 16) copy8(kn + 8 * tid, Kh + (int64_t)slot * kD + 8 * tid);
        else if (tid < 32) copy8(vn + 8 * (tid - 16), Vh + (int64_t)slot * kD + 8 * (tid - 16));
        else if (tid == 32) {
            idxh[slot] = posh;
            cumh[slot] = new_cum;
        }
    }
    if (tid == 0) {
        *len = (slot == n) ? n + 1 : n;
        if (evicted != nullptr) *evicted = ev;
    }
}

// kEarly (a few heads): bound by the chain of memory round trips, their tables being a few hundred KB: the rows'
// probabilities, scores and positions are requested before the parts' maxima are known, a wave per query head walks the
// parts, their outputs are requested eight at a time.  8 heads of 2048 rows: 10.0 -> 8.4 us.
// Otherwise the work per head counts, which other heads' round trips hide or many query heads make plenty: a thread per
// query head walks the parts, a thread per output adds them.
template <int GT, int NT, bool kEarly>
__global__ __launch_bounds__(NT) void decode_update_kernel(
    const bf16_bits* __restrict__ k_new, const bf16_bits* __restrict__ v_new, int G,
    const int32_t* __restrict__ pos, const int32_t* __restrict__ budget, int w, int cap, bf16_bits* Kc,
    bf16_bits* Vc, int32_t* idx, float* cum, int32_t* len, float* __restrict__ out,
    int32_t* __restrict__ evicted, int wave_rows, int np_max, int s_rows, const float* __restrict__ ws_p,
    const float* __restrict__ ws_ml, const float* __restrict__ ws_acc) {
    constexpr int NW = NT / 64, U = kEarly ? 4 : 2;
    extern __shared__ __align__(16) float coef[];                   // [np_max][GT]: exp2(m_part - m) / sum
    __shared__ __align__(16) float4 part_out[kEarly ? NT : 1];
    __shared__ float head_m[GT], head_inv[GT];
    __shared__ unsigned long long wave_best[NW];
    __shared__ int victim_slot;
    __shared__ float new_cum_s;
    const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int n = len[h];
    n = n < 0 ? 0 : (n > cap ? cap : n);
    const int n1 = n + 1;
    const int np = (n1 + wave_rows - 1) / wave_rows;
    bf16_bits* Kh = Kc + (int64_t)h * cap * kD;
    bf16_bits* Vh = Vc + (int64_t)h * cap * kD;
    int32_t* idxh = idx + (int64_t)h * cap;
    float* cumh = cum + (int64_t)h * cap;
    const float2* ml = reinterpret_cast<const float2*>(ws_ml) + (int64_t)h * np_max * GT;
    const float* ph = ws_p + (int64_t)h * s_rows * GT;
    const int posh = pos[h];
    int b = budget[h];
    b = b < w ? w : b;
    b = b > cap ? cap : b;
    const bool over = n1 > b;
    if (tid == 0) victim_slot = -1;
    float4 pr[U][GT / 4];
    float c_in[U];
    int id_in[U];
    auto load_rows = [&](int r0) {                                  // clamped; skipped where no thread has a row
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kEarly && u > 0 && r0 - tid + u * NT > n) continue;
            const int r = min(r0 + u * NT, n), rc = min(r, cap - 1);
#pragma unroll
            for (int g4 = 0; g4 < GT / 4; ++g4) pr[u][g4] = *reinterpret_cast<const float4*>(ph + (int64_t)r * GT + 4 * g4);
            c_in[u] = cumh[rc];
            id_in[u] = idxh[rc];
        }
    };
    if constexpr (kEarly) load_rows(tid);
    if constexpr (!kEarly) {
        float* pm = coef + np_max * GT;                             // the parts' maxima and sums
        float* pl = coef + 2 * np_max * GT;
        for (int i = tid; i < np * GT; i += NT) {
            float2 v = make_float2(0.f, 0.f);
            if ((i % GT) < G) v = ml[i];                            // columns beyond G were never written
            pm[i] = v.x;
            pl[i] = v.y;
        }
        __syncthreads();
        if (tid < GT) {
            float m = -INFINITY, l = 0.f;
            for (int x = 0; x < np; ++x) m = fmaxf(m, pm[x * GT + tid]);
            for (int x = 0; x < np; ++x) l += pl[x * GT + tid] * exp2f(pm[x * GT + tid] - m);
            head_m[tid] = m;
            head_inv[tid] = tid < G ? 1.0f / l : 0.f;
        }
        __syncthreads();
        for (int i = tid; i < np * GT; i += NT) coef[i] = exp2f(pm[i] - head_m[i % GT]) * head_inv[i % GT];
    }
    // a wave per query head: maximum and sum over the parts
    for (int g = kEarly ? wave : GT; g < GT; g += NW) {
        if (g < G) {                                                 // columns beyond G were never written
            float m = -INFINITY, l = 0.f;
            for (int x = lane; x < np; x += 64) m = fmaxf(m, ml[x * GT + g].x);
            m = wave_max(m);
            for (int x = lane; x < np; x += 64) {
                const float2 v = ml[x * GT + g];
                l += v.y * exp2f(v.x - m);
            }
            const float inv = 1.0f / wave_sum(l);
            for (int x = lane; x < np; x += 64) coef[x * GT + g] = exp2f(ml[x * GT + g].x - m) * inv;
        } else {
            for (int x = lane; x < np; x += 64) coef[x * GT + g] = 0.f;
        }
    }
    __syncthreads();
    // attention output: the parts' unnormalised sums, rescaled to the head's maximum.  kEarly: 128 threads per four
    // heads' outputs (four features each), four groups of them share the parts.
    const float* acch = ws_acc + (int64_t)h * np_max * GT * kD;
    if constexpr (!kEarly) {
        for (int o = tid; o < G * kD; o += NT) {
            const int g = o >> 7, f = o & (kD - 1);
            float v = 0.f;
            for (int x = 0; x < np; ++x) v = fmaf(acch[((int64_t)x * GT + g) * kD + f], coef[x * GT + g], v);
            out[(int64_t)h * G * kD + o] = v;
        }
    }
    for (int g4 = kEarly ? 0 : GT; g4 < GT; g4 += 4) {
        const int o = tid & 127, grp = tid >> 7, g = g4 + (o >> 5), f = 4 * (o & 31);
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int x0 = grp; x0 < np; x0 += 32) {
            float4 a[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                a[e] = *reinterpret_cast<const float4*>(acch + ((int64_t)min(x0 + 4 * e, np - 1) * GT + g) * kD + f);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (x0 + 4 * e < np) {
                    const float cf = coef[(x0 + 4 * e) * GT + g];
                    v.x = fmaf(a[e].x, cf, v.x);
                    v.y = fmaf(a[e].y, cf, v.y);
                    v.z = fmaf(a[e].z, cf, v.z);
                    v.w = fmaf(a[e].w, cf, v.w);
                }
            }
        }
        if (g4 > 0) __syncthreads();                                 // the previous heads' sums have been read
        part_out[tid] = v;
        __syncthreads();
        if (grp == 0 && g < G) {
#pragma unroll
            for (int x = 1; x < 4; ++x) {
                const float4 t = part_out[o + 128 * x];
                v.x += t.x;
                v.y += t.y;
                v.z += t.z;
                v.w += t.w;
            }
            const f32x4_any_t o4 = {v.x, v.y, v.z, v.w};
            *reinterpret_cast<f32x4_any_t*>(out + ((int64_t)h * G + g) * kD + f) = o4;
        }
    }
    // cumulative scores and the candidate for eviction
    unsigned long long best = ~0ull;
    int best_r = -1;
    for (int r0 = tid; r0 < n1; r0 += U * NT) {
        if (!kEarly || r0 != tid) load_rows(r0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * NT;
            if (r < n1) {
                const float* cf = coef + (r / wave_rows) * GT;
                float inc = 0.f;                                     // sum over the query heads of p_gr
#pragma unroll
                for (int g4 = 0; g4 < GT / 4; ++g4) {
                    const float4 cc = *reinterpret_cast<const float4*>(cf + 4 * g4);
                    inc += pr[u][g4].x * cc.x;
                    inc += pr[u][g4].y * cc.y;
                    inc += pr[u][g4].z * cc.z;
                    inc += pr[u][g4].w * cc.w;
                }
                if (r < n) {
                    const float c = c_in[u] + inc;
                    cumh[r] = c;
                    if (id_in[u] <= posh - w) {
                        const unsigned long long key = ((unsigned long long)ascending_key(c) << 32) | (uint32_t)id_in[u];
                        if (key < best) {
                            best = key;
                            best_r = r;
                        }
                    }
                } else {
                    new_cum_s = inc;
                }
            }
        }
    }
    const unsigned long long mine = best;
    best = wave_min_u64(best);
    if (lane == 0) wave_best[wave] = best;
    __syncthreads();
    best = wave_best[0];
#pragma unroll
    for (int x = 1; x < NW; ++x) best = wave_best[x] < best ? wave_best[x] : best;
    if (over && best_r >= 0 && mine == best) victim_slot = best_r;
    __syncthreads();
    place_token(k_new + (int64_t)h * kD, v_new + (int64_t)h * kD, Kh, Vh, idxh, cumh, len + h,
                evicted != nullptr ? evicted + h : nullptr, tid, n, cap, over, victim_slot, (int)(uint32_t)best, posh, new_cum_s);
}

// ---- bf16, enough heads to fill the chip: one workgroup per head does the whole step ------------------------------
// The two kernels above write every probability and every part's output to memory and read them back, a fifth of the
// traffic of the step at 8 query heads; here they stay in LDS.  Bound by the key and value stream.  Waves take 16-row
// tiles in turn, key and value rows of the next tile in flight under the arithmetic of this one; probabilities are kept
// against a reference per wave, the maximum of its first tile, which is raised (and everything rescaled) only when a
// probability would exceed 2^40: fp32 holds the products of that range without loss.
// 5120 heads of 768 rows on average, 8 query heads: 453 + 69 us in two kernels, 405 here; 256 heads of 2048 rows: 58 + 12, 55.
constexpr float kRefSlack = 40.f;

// Head of workgroup b.  Workgroups go to the eight XCDs in turn, and lengths often repeat with the head's number (the
// budgets of a layer's eight heads): in order, one XCD would get all the long ones.  Every eight heads are turned by
// another amount instead (1000 heads of 1450 rows, every sixteenth full and the others an eighth: 65 -> 42 us).
__device__ __forceinline__ int spread_head(unsigned b, unsigned n) {
    const unsigned o = b >> 3;
    return b < (n & ~7u) ? 8 * o + ((b + o + (o >> 1) + (o >> 2) + (o >> 3)) & 7) : b;
}

template <int GT, int NW>
__global__ __launch_bounds__(64 * NW, 2) void decode_head_kernel(
    const bf16_bits* __restrict__ q, const bf16_bits* __restrict__ k_new, const bf16_bits* __restrict__ v_new, int G,
    const int32_t* __restrict__ pos, const int32_t* __restrict__ budget, int w, int cap, bf16_bits* Kc, bf16_bits* Vc,
    int32_t* idx, float* cum, int32_t* len, float* __restrict__ out, int32_t* __restrict__ evicted, int s_rows) {
    constexpr int NT = 64 * NW;
    extern __shared__ __align__(16) float dynh[];
    float* prob = dynh;                                              // [s_rows][GT]
    float* accs = dynh + s_rows * GT;                                // [NW][GT][128]
    __shared__ float wave_m[NW][GT], wave_l[NW][GT];
    __shared__ __align__(16) float coef[NW * GT];                    // exp2(m_wave - m) / sum
    __shared__ unsigned long long wave_best[NW];
    __shared__ int victim_slot;
    __shared__ float new_cum_s;
    const int h = spread_head(blockIdx.x, gridDim.x), tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, j = lane >> 4;
    int n = len[h];
    n = n < 0 ? 0 : (n > cap ? cap : n);
    const int n1 = n + 1, n_t = (n1 + 15) >> 4;                      // 16 n_t <= s_rows
    bf16_bits* Kh = Kc + (int64_t)h * cap * kD;
    bf16_bits* Vh = Vc + (int64_t)h * cap * kD;
    int32_t* idxh = idx + (int64_t)h * cap;
    float* cumh = cum + (int64_t)h * cap;
    const bf16_bits* kn = k_new + (int64_t)h * kD;
    const bf16_bits* vn = v_new + (int64_t)h * kD;
    const int posh = pos[h];
    int b = budget[h];
    b = b < w ? w : b;
    b = b > cap ? cap : b;
    const bool over = n1 > b;
    if (tid == 0) victim_slot = -1;

    bf16x8_t qb[4];                                                  // column c16 = query head, zero beyond G
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (c16 < G) v = *reinterpret_cast<const uint4*>(q + ((int64_t)h * G + c16) * kD + 32 * ks + 8 * j);
        qb[ks] = __builtin_bit_cast(bf16x8_t, v);
    }
    auto load_k = [&](uint4 (&dst)[4], int t) {                      // rows past the end re-read the new token
        const int r = 16 * t + c16;
        const bf16_bits* src = (r < n ? Kh + (int64_t)r * kD : kn) + 8 * j;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dst[ks] = *reinterpret_cast<const uint4*>(src + 32 * ks);
    };
    auto load_v = [&](uint4 (&dst)[4], int t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = 16 * t + 4 * u + j;
            const bf16_bits* src = (r < n ? Vh + (int64_t)r * kD : vn) + 8 * c16;
            dst[u] = *reinterpret_cast<const uint4*>(src);
        }
    };
    const float qs = 0.08838834764831845f * 1.4426950408889634f;     // 1/sqrt(128) * log2(e)
    // Reference before the first row: finite, so that logits of -inf give zeros and not NaN, and below every finite logit.
    constexpr float kNoRow = -3.402823466e38f;
    float ref = kNoRow, sum = 0.f;                                   // of column c16; sum over this lane's rows
    float acc[GT][8];
#pragma unroll
    for (int g = 0; g < GT; ++g)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
    auto column_max = [&](const f32x4_t& s) {
        float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        return fmaxf(mx, __shfl_xor(mx, 32, 64));
    };
    auto tile = [&](const uint4 (&kt)[4], const uint4 (&vt)[4], int t) {
        f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kt[ks]), qb[ks], s, 0, 0, 0);
        bool above = false;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            s[v] = 16 * t + 4 * j + v < n1 ? s[v] * qs : -INFINITY;
            above |= s[v] > ref + kRefSlack;
        }
        if (__any(above)) {                                          // the first tile (t = wave), hardly ever later
            const float m = fmaxf(ref, column_max(s)), f = exp2f(ref - m);
            sum *= f;
#pragma unroll
            for (int g = 0; g < GT; ++g) {
                const float fg = __shfl(f, g, 64);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[g][e] *= fg;
            }
            if (c16 < GT)
                for (int u = wave; u < t; u += NW)                   // the entries this lane has written
                    for (int v = 0; v < 4; ++v) prob[(16 * u + 4 * j + v) * GT + c16] *= f;
            ref = m;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float e = exp2f(s[v] - ref);
            sum += e;
            if (c16 < GT) prob[(16 * t + 4 * j + v) * GT + c16] = e;
        }
        // LDS traffic of one wave is processed in issue order; the fences keep the compiler from moving the reads
        // below over the writes above
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float vf[8];
            const uint32_t wds[4] = {vt[u].x, vt[u].y, vt[u].z, vt[u].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                vf[2 * i] = __uint_as_float(wds[i] << 16);
                vf[2 * i + 1] = __uint_as_float(wds[i] & 0xffff0000u);
            }
            const float* prow = prob + (16 * t + 4 * u + j) * GT;
#pragma unroll
            for (int g4 = 0; g4 < GT; g4 += 4) {
                const float4 pr = *reinterpret_cast<const float4*>(prow + g4);
                const float prs[4] = {pr.x, pr.y, pr.z, pr.w};
#pragma unroll
                for (int gg = 0; gg < 4; ++gg)
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[g4 + gg][e] = fmaf(prs[gg], vf[e], acc[g4 + gg][e]);
            }
        }
    };
    uint4 ka[4], va[4], kb[4], vb[4];
    load_k(ka, wave);
    load_v(va, wave);
    for (int t = wave; t < n_t; t += 2 * NW) {
        load_k(kb, t + NW);
        load_v(vb, t + NW);
        tile(ka, va, t);
        if (t + NW < n_t) {
            load_k(ka, t + 2 * NW);
            load_v(va, t + 2 * NW);
            tile(kb, vb, t + NW);
        }
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if (j == 0 && c16 < GT) {
        wave_m[wave][c16] = ref;
        wave_l[wave][c16] = sum;
    }
    // sum over the four lane rows; lane row j keeps query head g4 + {0,2,1,3}[j]
    const int gsel = ((j & 1) << 1) | (j >> 1);
#pragma unroll
    for (int g4 = 0; g4 < GT; g4 += 4) {
        float tot[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            tot[e] = reduce4_over_rows(acc[g4][e], acc[g4 + 1][e], acc[g4 + 2][e], acc[g4 + 3][e]);
        float* dst = accs + (wave * GT + g4 + gsel) * kD + 8 * c16;
        reinterpret_cast<float4*>(dst)[0] = make_float4(tot[0], tot[1], tot[2], tot[3]);
        reinterpret_cast<float4*>(dst)[1] = make_float4(tot[4], tot[5], tot[6], tot[7]);
    }
    __syncthreads();
    if (tid < GT) {
        float m = wave_m[0][tid], l = 0.f;
#pragma unroll
        for (int x = 1; x < NW; ++x) m = fmaxf(m, wave_m[x][tid]);
#pragma unroll
        for (int x = 0; x < NW; ++x) l += wave_l[x][tid] * exp2f(wave_m[x][tid] - m);
        const float inv = tid < G ? 1.0f / l : 0.f;
#pragma unroll
        for (int x = 0; x < NW; ++x) coef[x * GT + tid] = exp2f(wave_m[x][tid] - m) * inv;
    }
    __syncthreads();
    for (int o = tid; o < G * kD; o += NT) {
        const int g = o >> 7;
        float v = 0.f;
#pragma unroll
        for (int x = 0; x < NW; ++x) v = fmaf(accs[x * GT * kD + o], coef[x * GT + g], v);
        out[(int64_t)h * G * kD + o] = v;
    }
    // cumulative scores and the candidate for eviction
    unsigned long long best = ~0ull;
    int best_r = -1;
    constexpr int U = 4;
    for (int r0 = tid; r0 < n1; r0 += U * NT) {
        float c_in[U];
        int id_in[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int rc = min(r0 + u * NT, cap - 1);
            c_in[u] = cumh[rc];
            id_in[u] = idxh[rc];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * NT;
            if (r < n1) {
                const float* cf = coef + ((r >> 4) % NW) * GT;
                float inc = 0.f;                                     // sum over the query heads of p_gr
#pragma unroll
                for (int g4 = 0; g4 < GT; g4 += 4) {
                    const float4 pr = *reinterpret_cast<const float4*>(prob + r * GT + g4);
                    const float4 cc = *reinterpret_cast<const float4*>(cf + g4);
                    inc += pr.x * cc.x;
                    inc += pr.y * cc.y;
                    inc += pr.z * cc.z;
                    inc += pr.w * cc.w;
                }
                if (r < n) {
                    const float c = c_in[u] + inc;
                    cumh[r] = c;
                    if (id_in[u] <= posh - w) {
                        const unsigned long long key = ((unsigned long long)ascending_key(c) << 32) | (uint32_t)id_in[u];
                        if (key < best) {
                            best = key;
                            best_r = r;
                        }
                    }
                } else {
                    new_cum_s = inc;
                }
            }
        }
    }
    const unsigned long long mine = best;
    best = wave_min_u64(best);
    if (lane == 0) wave_best[wave] = best;
    __syncthreads();
    best = wave_best[0];
#pragma unroll
    for (int x = 1; x < NW; ++x) best = wave_best[x] < best ? wave_best[x] : best;
    if (over && best_r >= 0 && mine == best) victim_slot = best_r;
    __syncthreads();
    place_token(kn, vn, Kh, Vh, idxh, cumh, len + h, evicted != nullptr ? evicted + h : nullptr, tid, n, cap, over,
                victim_slot, (int)(uint32_t)best, posh, new_cum_s);
}

// Floats that another workgroup of the same launch writes or reads.  The accesses carry the agent scope (sc1): they go past
// the caches that workgroups on different XCDs do not share, so that no fence has to write back or invalidate a whole L2 (a
// fence of that scope per workgroup: 92 us for 8 heads of 8000 rows).  A store is where others can read it once the wave has
// waited for it.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
constexpr int kAgentScope = 16;                                     // the sc1 bit of a buffer access
__device__ __forceinline__ __amdgpu_buffer_rsrc_t shared_floats(float* p, int n) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, n * (int)sizeof(float), 0x00027000);
}
__device__ __forceinline__ void put4(__amdgpu_buffer_rsrc_t b, int i, float4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)}, b,
                                           i * (int)sizeof(float), 0, kAgentScope);
}
__device__ __forceinline__ float4 get4(__amdgpu_buffer_rsrc_t b, int i) {
    const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(b, i * (int)sizeof(float), 0, kAgentScope);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void put2(__amdgpu_buffer_rsrc_t b, int i, float2 v) {
    __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{__float_as_uint(v.x), __float_as_uint(v.y)}, b, i * (int)sizeof(float), 0, kAgentScope);
}
__device__ __forceinline__ float2 get2(__amdgpu_buffer_rsrc_t b, int i) {
    const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(b, i * (int)sizeof(float), 0, kAgentScope);
    return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
}

// One launch for few heads whose rows are spread over several workgroups: eight waves of WR rows each, every load of a wave
// requested before the first is needed.  A workgroup leaves its probabilities, its output and their maximum and sum in the
// workspace and counts itself; the last one of a head merges them and makes the step's update (what decode_update_kernel does
// in a launch of its own).  Nothing waits for another workgroup.  All workgroups of a head count, also those without rows:
// the last one changes the length that they all read.  The counters are zero before and after every call.
template <int GT, int WR>
__global__ __launch_bounds__(kSplitThreads) void decode_split_kernel(
    const bf16_bits* __restrict__ q, const bf16_bits* __restrict__ k_new, const bf16_bits* __restrict__ v_new, int G,
    const int32_t* __restrict__ pos, const int32_t* __restrict__ budget, int w, int cap, bf16_bits* Kc, bf16_bits* Vc,
    int32_t* idx, float* cum, int32_t* len, float* __restrict__ out, int32_t* __restrict__ evicted, int s_rows, float* ws_p,
    float* ws_ml, float* ws_acc, uint32_t* counters) {
    constexpr int NT = kSplitThreads, NW = NT / 64, kTiles = WR / 16, kRows = NW * WR;
    __shared__ __align__(16) float prob[kRows * GT];
    __shared__ __align__(16) float accs[NW * GT * kD];
    __shared__ float wave_m[NW][GT], wave_l[NW][GT];
    __shared__ __align__(16) float wave_f[NW * GT];                 // exp2(m_wave - m)
    __shared__ unsigned long long wave_best[NW];
    __shared__ int victim_slot, is_last;
    __shared__ float new_cum_s;
    const int part = blockIdx.x, np_max = gridDim.x, h = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c16 = lane & 15, j = lane >> 4;
    int n = len[h];
    n = n < 0 ? 0 : (n > cap ? cap : n);
    const int n1 = n + 1, row0 = part * kRows, wave0 = row0 + wave * WR;
    bf16_bits* Kh = Kc + (int64_t)h * cap * kD;
    bf16_bits* Vh = Vc + (int64_t)h * cap * kD;
    int32_t* idxh = idx + (int64_t)h * cap;
    float* cumh = cum + (int64_t)h * cap;
    const bf16_bits* kn = k_new + (int64_t)h * kD;
    const bf16_bits* vn = v_new + (int64_t)h * kD;
    const auto ph = shared_floats(ws_p + (int64_t)h * s_rows * GT, s_rows * GT);
    const auto mlh = shared_floats(ws_ml + (int64_t)h * np_max * GT * 2, np_max * GT * 2);
    const auto acch = shared_floats(ws_acc + (int64_t)h * np_max * GT * kD, np_max * GT * kD);
    if (row0 < n1) {
        uint4 kt[kTiles][4], vt[kTiles][4];
#pragma unroll
        for (int t = 0; t < kTiles; ++t) {                          // rows past the end re-read the new token
            const int r = wave0 + 16 * t + c16;
            const bf16_bits* src = (r < n ? Kh + (int64_t)r * kD : kn) + 8 * j;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) kt[t][ks] = *reinterpret_cast<const uint4*>(src + 32 * ks);
        }
        bf16x8_t qb[4];                                              // column c16 = query head, zero beyond G
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (c16 < G) v = *reinterpret_cast<const uint4*>(q + ((int64_t)h * G + c16) * kD + 32 * ks + 8 * j);
            qb[ks] = __builtin_bit_cast(bf16x8_t, v);
        }
#pragma unroll
        for (int t = 0; t < kTiles; ++t)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int r = wave0 + 16 * t + 4 * u + j;
                const bf16_bits* src = (r < n ? Vh + (int64_t)r * kD : vn) + 8 * c16;
                vt[t][u] = *reinterpret_cast<const uint4*>(src);
            }
        __builtin_amdgcn_sched_barrier(0);                           // everything is on its way
        const float qs = 0.08838834764831845f * 1.4426950408889634f; // 1/sqrt(128) * log2(e)
        f32x4_t s[kTiles];
        float mx = -3.402823466e38f, sum = 0.f;                      // finite: logits of -inf weigh nothing
#pragma unroll
        for (int t = 0; t < kTiles; ++t) {
            f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kt[t][ks]), qb[ks], c, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                s[t][v] = wave0 + 16 * t + 4 * j + v < n1 ? c[v] * qs : -INFINITY;
                mx = fmaxf(mx, s[t][v]);
            }
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        float* pl = prob + wave * WR * GT;
#pragma unroll
        for (int t = 0; t < kTiles; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float e = exp2f(s[t][v] - mx);
                sum += e;
                if (c16 < GT) pl[(16 * t + 4 * j + v) * GT + c16] = e;
            }
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        if (j == 0 && c16 < GT) {
            wave_m[wave][c16] = mx;
            wave_l[wave][c16] = sum;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");       // the wave's own probabilities
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        float acc[GT][8];
#pragma unroll
        for (int g = 0; g < GT; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
#pragma unroll
        for (int t = 0; t < kTiles; ++t)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float vf[8];
                const uint32_t wds[4] = {vt[t][u].x, vt[t][u].y, vt[t][u].z, vt[t][u].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    vf[2 * i] = __uint_as_float(wds[i] << 16);
                    vf[2 * i + 1] = __uint_as_float(wds[i] & 0xffff0000u);
                }
                const float* prow = pl + (16 * t + 4 * u + j) * GT;
#pragma unroll
                for (int g4 = 0; g4 < GT; g4 += 4) {
                    const float4 pr = *reinterpret_cast<const float4*>(prow + g4);
                    const float prs[4] = {pr.x, pr.y, pr.z, pr.w};
#pragma unroll
                    for (int gg = 0; gg < 4; ++gg)
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[g4 + gg][e] = fmaf(prs[gg], vf[e], acc[g4 + gg][e]);
                }
            }
        // lane row j receives query head g4 + {0,2,1,3}[j]
        const int gsel = ((j & 1) << 1) | (j >> 1);
#pragma unroll
        for (int g4 = 0; g4 < GT; g4 += 4) {
            float tot[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                tot[e] = reduce4_over_rows(acc[g4][e], acc[g4 + 1][e], acc[g4 + 2][e], acc[g4 + 3][e]);
            float* dst = accs + (wave * GT + g4 + gsel) * kD + 8 * c16;
            reinterpret_cast<float4*>(dst)[0] = make_float4(tot[0], tot[1], tot[2], tot[3]);
            reinterpret_cast<float4*>(dst)[1] = make_float4(tot[4], tot[5], tot[6], tot[7]);
        }
        __syncthreads();
        if (tid < NW * GT) {
            const int g = tid % GT;
            float m = wave_m[0][g];
#pragma unroll
            for (int x = 1; x < NW; ++x) m = fmaxf(m, wave_m[x][g]);
            wave_f[tid] = exp2f(wave_m[tid / GT][g] - m);
            if (tid < GT) {
                float l = 0.f;
#pragma unroll
                for (int x = 0; x < NW; ++x) l += wave_l[x][g] * exp2f(wave_m[x][g] - m);
                put2(mlh, (part * GT + g) * 2, make_float2(m, l));
            }
        }
        __syncthreads();
        if (2 * tid < GT * kD) {
            const int o = 2 * tid;
            float2 v = make_float2(0.f, 0.f);
#pragma unroll
            for (int x = 0; x < NW; ++x) {
                const float2 a = *reinterpret_cast<const float2*>(accs + x * GT * kD + o);
                const float f = wave_f[x * GT + (o >> 7)];
                v.x = fmaf(a.x, f, v.x);
                v.y = fmaf(a.y, f, v.y);
            }
            put2(acch, part * GT * kD + o, v);
        }
        const int n_f4 = min(kRows, n1 - row0) * (GT / 4);           // n1 <= s_rows
        for (int i = tid; i < n_f4; i += NT) {
            float4 v = *reinterpret_cast<const float4*>(prob + 4 * i);
            const float4 f = *reinterpret_cast<const float4*>(wave_f + i / (WR * GT / 4) * GT + 4 * (i % (GT / 4)));
            v.x *= f.x;
            v.y *= f.y;
            v.z *= f.z;
            v.w *= f.w;
            put4(ph, row0 * GT + 4 * i, v);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // what this wave put has arrived
    __syncthreads();
    if (tid == 0) {
        const uint32_t before = __hip_atomic_fetch_add(&counters[h], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        is_last = before == (uint32_t)(np_max - 1);
        if (is_last) __hip_atomic_store(&counters[h], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        victim_slot = -1;
    }
    __syncthreads();
    if (!is_last) return;

    const int posh = pos[h], np = (n1 + kRows - 1) / kRows;
    int b = budget[h];
    b = b < w ? w : b;
    b = b > cap ? cap : b;
    const bool over = n1 > b;
    constexpr int U = GT == 4 ? 8 : 4;
    float4 pr[U][GT / 4];
    float c_in[U];
    int id_in[U];
    auto load_rows = [&](int r0) {                                   // clamped; skipped where no thread has a row
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u > 0 && r0 - tid + u * NT > n) continue;
            const int r = min(r0 + u * NT, n), rc = min(r, cap - 1);
#pragma unroll
            for (int g4 = 0; g4 < GT / 4; ++g4) pr[u][g4] = get4(ph, r * GT + 4 * g4);
            c_in[u] = cumh[rc];
            id_in[u] = idxh[rc];
        }
    };
    load_rows(tid);
    float* coef = accs;                                              // [np][GT]: exp2(m_part - m) / sum
    for (int g = wave; g < GT; g += NW) {                            // a lane per part, once more for every 64 parts
        auto ml = [&](int x) { return get2(mlh, (x * GT + g) * 2); };
        const float2 first = lane < np ? ml(lane) : make_float2(-3.402823466e38f, 0.f);
        float m = first.x;
        for (int x = lane + 64; x < np; x += 64) m = fmaxf(m, ml(x).x);
        m = wave_max(m);
        float l = first.y * exp2f(first.x - m);
        for (int x = lane + 64; x < np; x += 64) {
            const float2 v = ml(x);
            l += v.y * exp2f(v.x - m);
        }
        const float inv = g < G ? 1.0f / wave_sum(l) : 0.f;
        if (lane < np) coef[lane * GT + g] = exp2f(first.x - m) * inv;
        for (int x = lane + 64; x < np; x += 64) coef[x * GT + g] = exp2f(ml(x).x - m) * inv;
    }
    __syncthreads();
    static_assert(GT * kD <= 2 * NT, "two outputs a thread");
    if (2 * tid < G * kD) {
        const int o = 2 * tid;
        float v0 = 0.f, v1 = 0.f;
        for (int x0 = 0; x0 < np; x0 += 8) {
            float2 a[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) a[e] = get2(acch, min(x0 + e, np - 1) * GT * kD + o);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (x0 + e < np) {
                    const float f = coef[(x0 + e) * GT + (o >> 7)];
                    v0 = fmaf(a[e].x, f, v0);
                    v1 = fmaf(a[e].y, f, v1);
                }
            }
        }
        out[(int64_t)h * G * kD + o] = v0;
        out[(int64_t)h * G * kD + o + 1] = v1;
    }
    unsigned long long best = ~0ull;
    int best_r = -1;
    for (int r0 = tid; r0 < n1; r0 += U * NT) {
        if (r0 != tid) load_rows(r0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * NT;
            if (r < n1) {
                const float* cf = coef + (r / kRows) * GT;
                float inc = 0.f;                                     // sum over the query heads of p_gr
#pragma unroll
                for (int g4 = 0; g4 < GT / 4; ++g4) {
                    const float4 cc = *reinterpret_cast<const float4*>(cf + 4 * g4);
                    inc += pr[u][g4].x * cc.x;
                    inc += pr[u][g4].y * cc.y;
                    inc += pr[u][g4].z * cc.z;
                    inc += pr[u][g4].w * cc.w;
                }
                if (r < n) {
                    const float c = c_in[u] + inc;
                    cumh[r] = c;
                    if (id_in[u] <= posh - w) {
                        const unsigned long long key = ((unsigned long long)ascending_key(c) << 32) | (uint32_t)id_in[u];
                        if (key < best) {
                            best = key;
                            best_r = r;
                        }
                    }
                } else {
                    new_cum_s = inc;
                }
            }
        }
    }
    const unsigned long long mine = best;
    best = wave_min_u64(best);
    if (lane == 0) wave_best[wave] = best;
    __syncthreads();
    best = wave_best[0];
#pragma unroll
    for (int x = 1; x < NW; ++x) best = wave_best[x] < best ? wave_best[x] : best;
    if (over && best_r >= 0 && mine == best) victim_slot = best_r;
    __syncthreads();
    place_token(kn, vn, Kh, Vh, idxh, cumh, len + h, evicted != nullptr ? evicted + h : nullptr, tid, n, cap, over,
                victim_slot, (int)(uint32_t)best, posh, new_cum_s);
}

DecodePlan plan_decode(int n_heads, int G, int cap, int wave_rows) {
    DecodePlan p;
    p.GT = G <= 4 ? 4 : (G <= 8 ? 8 : 16);
    // 256-row waves when that still leaves a few thousand waves to spread over the chip
    const int64_t waves256 = (int64_t)n_heads * ((cap + 1 + 255) / 256);
    p.wave_rows = wave_rows > 0 ? wave_rows : (p.GT <= 8 && waves256 >= 2048) ? 256 : 128;
    p.s_rows = (cap + 1 + p.wave_rows - 1) / p.wave_rows * p.wave_rows;
    p.np_max = p.s_rows / p.wave_rows;
    size_t off = 0;
    p.out_off = off;
    off = align_up(off + (size_t)n_heads * G * kD * sizeof(float), 256);
    p.p_off = off;
    off = align_up(off + (size_t)n_heads * p.s_rows * p.GT * sizeof(float), 256);
    p.ml_off = off;
    off = align_up(off + (size_t)n_heads * p.np_max * p.GT * 2 * sizeof(float), 256);
    p.acc_off = off;
    off = align_up(off + (size_t)n_heads * p.np_max * p.GT * kD * sizeof(float), 256);
    p.bytes = off;
    return p;
}

typedef void (*UpdateKernel)(const bf16_bits*, const bf16_bits*, int, const int32_t*, const int32_t*, int, int, bf16_bits*,
                             bf16_bits*, int32_t*, float*, int32_t*, float*, int32_t*, int, int, int, const float*,
                             const float*, const float*);
template <int GT>
static UpdateKernel update_few(bool early) {
    if constexpr (GT == 4) return decode_update_kernel<GT, 512, true>;
    else if constexpr (GT == 8) return early ? decode_update_kernel<GT, 512, true> : decode_update_kernel<GT, 1024, false>;
    else return decode_update_kernel<GT, 1024, false>;
}
// Threads of the update kernel (both kernels of the step, us).  Thousands of heads: 256 (5120 heads of 300 rows, 16 query
// heads: 284, with 384 threads 302); some hundreds: 512 (600 heads of 300 rows, 16 query heads: 38.4, with 1024 threads 42.0);
// fewer: kEarly for up to four query heads (8 heads of 2000 rows: 14.3, with 1024 threads and not early 15.4) and for up to
// eight with many parts to walk (8 heads of up to 4000 rows: 21.3 and 22.9; 1000: 16.5 and 17.4; 700: 16.3 and 16.0),
// else 1024 threads (8 heads of 1000 rows, 16 query heads: 20.0, kEarly 23.2).
constexpr int kUpdateManyHeads = 1280, kUpdateSomeHeads = 512, kUpdateEarlyParts = 16;

template <int GT, int WR>
static hipError_t launch_decode_wave_t(const void* q, const void* k_new, const void* v_new, int n_heads, int G,
                                       const int32_t* pos, const int32_t* budget, int w, int cap, void* Kc,
                                       void* Vc, int32_t* idx, float* cum, int32_t* len, float* out,
                                       int32_t* evicted, const DecodePlan& p, char* ws, const Env& env) {
    float* ws_p = reinterpret_cast<float*>(ws + p.p_off);
    float* ws_ml = reinterpret_cast<float*>(ws + p.ml_off);
    float* ws_acc = reinterpret_cast<float*>(ws + p.acc_off);
    const int64_t waves = (int64_t)n_heads * p.np_max;
    const unsigned grid = (unsigned)((waves + 3) / 4);
    const size_t lds_a = (size_t)4 * WR * GT * sizeof(float);
    env.begin("decode_attend_wave");
    decode_attend_wave_kernel<GT, WR><<<grid, 256, lds_a, env.s>>>(
        static_cast<const bf16_bits*>(q), static_cast<const bf16_bits*>(k_new), static_cast<const bf16_bits*>(v_new),
        n_heads, G, cap, static_cast<const bf16_bits*>(Kc), static_cast<const bf16_bits*>(Vc), len, p.np_max,
        p.s_rows, ws_p, ws_ml, ws_acc);
    env.end();
    env.begin("decode_update");
    const bool some = n_heads >= kUpdateSomeHeads, many = n_heads >= kUpdateManyHeads;
    const bool early = !some && (GT == 4 || (GT == 8 && p.np_max >= kUpdateEarlyParts));
    const int threads = many ? 256 : some || early ? 512 : 1024;
    UpdateKernel update = many ? decode_update_kernel<GT, 256, false> : some ? decode_update_kernel<GT, 512, false> : update_few<GT>(early);
    const size_t lds_u = decode_update_lds_bytes(p) / (early ? 3 : 1);          // early: the weights alone
    update<<<n_heads, threads, lds_u, env.s>>>(
        static_cast<const bf16_bits*>(k_new), static_cast<const bf16_bits*>(v_new), G, pos, budget, w, cap,
        static_cast<bf16_bits*>(Kc), static_cast<bf16_bits*>(Vc), idx, cum, len, out, evicted, WR, p.np_max, p.s_rows, ws_p,
        ws_ml, ws_acc);
    env.end();
    return hipGetLastError();
}

hipError_t launch_decode_wave(const void* q, const void* k_new, const void* v_new, int n_heads, int G,
                              const int32_t* pos, const int32_t* budget, int w, int cap, void* Kc, void* Vc,
                              int32_t* idx, float* cum, int32_t* len, float* out, int32_t* evicted,
                              const DecodePlan& p, char* ws, const Env& env) {
#define UNCOMP_WAVE_CASE(GT, WR)                                                                                  \
    return launch_decode_wave_t<GT, WR>(q, k_new, v_new, n_heads, G, pos, budget, w, cap, Kc, Vc, idx, cum, len, \
                                        out, evicted, p, ws, env)
    if (p.wave_rows == 256) {
        if (p.GT == 4) UNCOMP_WAVE_CASE(4, 256);
        UNCOMP_WAVE_CASE(8, 256);
    }
    if (p.wave_rows == 64) {
        if (p.GT == 4) UNCOMP_WAVE_CASE(4, 64);
        if (p.GT == 8) UNCOMP_WAVE_CASE(8, 64);
        UNCOMP_WAVE_CASE(16, 64);
    }
    if (p.GT == 4) UNCOMP_WAVE_CASE(4, 128);
    if (p.GT == 8) UNCOMP_WAVE_CASE(8, 128);
    UNCOMP_WAVE_CASE(16, 128);
#undef UNCOMP_WAVE_CASE
}

// Waves of one workgroup of the one-kernel step (us, 4 query heads unless noted; even, ragged and mostly empty caches).
// Four, of which a CU holds two or three workgroups: a head's start and end run under the others' streams.
//   1000 heads of 300 rows: 29 with four, 38 with eight; 2048 heads of 2000 rows: 382, two kernels 462.
// Eight, if a CU gets one head anyway (256 heads of up to 4000 rows, ragged: 47, with four 55) or a few long ones (up to
// 4000 rows: 300 heads, with eight budgets among them 108, with four 124; 700 heads 206 and 218).  Where the tables of
// eight do not fit, up to four query heads take two kernels, more of them four waves (300 heads of up to 2000 rows, 8 query
// heads: 54, two kernels 64).
// Two for thousands of short heads, whose time is that of their starts and ends: 5120 heads of 130 rows: 74, with four 78;
// 8 query heads, caches of 300 rows an eighth full: 42 and 60; but 2048 heads of 768 rows: 163 and 152.
static size_t head_lds_bytes(int waves, int G, int cap) {
    return ((size_t)(cap + 16) / 16 * 16 + (size_t)waves * kD) * (G <= 4 ? 4 : 8) * sizeof(float);
}
static int head_waves(int n_heads, int G, int cap) {
    const bool long_heads = n_heads <= 256 || (n_heads < 1024 && cap > 1536);
    if (long_heads && (G <= 4 || head_lds_bytes(8, G, cap) <= kDecodeHeadLdsMax)) return 8;
    return n_heads >= 2048 && cap <= 512 ? 2 : 4;
}

size_t decode_head_lds_bytes(int n_heads, int G, int cap) { return head_lds_bytes(head_waves(n_heads, G, cap), G, cap); }

hipError_t launch_decode_head(const void* q, const void* k_new, const void* v_new, int n_heads, int G, const int32_t* pos,
                              const int32_t* budget, int w, int cap, void* Kc, void* Vc, int32_t* idx, float* cum,
                              int32_t* len, float* out, int32_t* evicted, const Env& env) {
    const int nw = head_waves(n_heads, G, cap);
    const size_t lds = decode_head_lds_bytes(n_heads, G, cap);
    if (lds > kDecodeHeadLdsMax || G > 8) return hipErrorInvalidValue;   // the interface checks before
    auto kern = G <= 4 ? (nw == 8 ? decode_head_kernel<4, 8> : nw == 4 ? decode_head_kernel<4, 4> : decode_head_kernel<4, 2>)
                       : (nw == 8 ? decode_head_kernel<8, 8> : nw == 4 ? decode_head_kernel<8, 4> : decode_head_kernel<8, 2>);
    env.begin("decode_head");
    kern<<<n_heads, 64 * nw, lds, env.s>>>(static_cast<const bf16_bits*>(q), static_cast<const bf16_bits*>(k_new),
                                           static_cast<const bf16_bits*>(v_new), G, pos, budget, w, cap,
                                           static_cast<bf16_bits*>(Kc), static_cast<bf16_bits*>(Vc), idx, cum, len, out,
                                           evicted, (cap + 16) / 16 * 16);
    env.end();
    return hipGetLastError();
}

// 16 rows a wave while that keeps to sixteen parts and half the chip, so that a CU has few rows to fetch; 32 beyond, so that
// there are few parts to merge (us): 8 heads of 1000 rows 9.8 / 11.0, of 2000 rows 11.5 / 11.8, of 3238 rows 14.1 / 13.3; 64
// heads of 500 rows 10.6 / 11.2, of 700 rows 12.4 / 12.2.  64 rows are slower up to 90 thousand rows in all (8 heads of 3238
// rows 15.2) and within 5 % of 32 rows above.
DecodePlan plan_decode_split(int n_heads, int G, int cap) {
    const int wave_rows = cap <= 2048 && (int64_t)n_heads * cap <= 32768 ? 16 : 32;
    DecodePlan p = plan_decode(n_heads, G, cap, kSplitThreads / 64 * wave_rows);
    p.s_rows = (cap + 16) / 16 * 16;                                 // rows that are there: the others are not written
    p.wave_rows = wave_rows;
    p.ml_off = align_up(p.p_off + (size_t)n_heads * p.s_rows * p.GT * sizeof(float), 256);
    p.acc_off = align_up(p.ml_off + (size_t)n_heads * p.np_max * p.GT * 2 * sizeof(float), 256);
    p.bytes = align_up(p.acc_off + (size_t)n_heads * p.np_max * p.GT * kD * sizeof(float), 256);
    return p;
}

hipError_t launch_decode_split(const void* q, const void* k_new, const void* v_new, int n_heads, int G, const int32_t* pos,
                               const int32_t* budget, int w, int cap, void* Kc, void* Vc, int32_t* idx, float* cum,
                               int32_t* len, float* out, int32_t* evicted, const DecodePlan& p, char* ws, uint32_t* counters,
                               const Env& env) {
    if (n_heads > kSplitHeads || p.GT > 8 || p.np_max > kSplitParts) return hipErrorInvalidValue;   // the interface checks before
    auto kern = p.GT == 4 ? (p.wave_rows == 16 ? decode_split_kernel<4, 16> : decode_split_kernel<4, 32>)
                          : (p.wave_rows == 16 ? decode_split_kernel<8, 16> : decode_split_kernel<8, 32>);
    env.begin("decode_split");
    kern<<<dim3((unsigned)p.np_max, (unsigned)n_heads), dim3(kSplitThreads), 0, env.s>>>(
        static_cast<const bf16_bits*>(q), static_cast<const bf16_bits*>(k_new), static_cast<const bf16_bits*>(v_new), G, pos,
        budget, w, cap, static_cast<bf16_bits*>(Kc), static_cast<bf16_bits*>(Vc), idx, cum, len, out, evicted, p.s_rows,
        reinterpret_cast<float*>(ws + p.p_off), reinterpret_cast<float*>(ws + p.ml_off), reinterpret_cast<float*>(ws + p.acc_off),
        counters);
    env.end();
    return hipGetLastError();
}

hipError_t launch_decode_init(const float* score, const int32_t* idx, const int32_t* len, int n_heads,
                              int N, int w, int cap, float* cum, const Env& env) {
    int64_t total = (int64_t)n_heads * cap;
    int blocks = (int)((total + 255) / 256 > 4096 ? 4096 : (total + 255) / 256);
    env.begin("decode_init");
    decode_init_kernel<<<blocks, 256, 0, env.s>>>(score, idx, len, n_heads, N - w, cap, cum);
    env.end();
    return hipGetLastError();
}

// dynamic LDS the one-kernel decode path may ask for: G*(cap+1) <= 36864 floats plus rounding of cap
constexpr size_t kDecodeStepLdsMax = (36864 + 64) * sizeof(float);

// the update kernel's tables: the parts' maxima, sums and weights
size_t decode_update_lds_bytes(const DecodePlan& p) { return (size_t)3 * p.np_max * p.GT * sizeof(float); }

size_t decode_step_lds_bytes(int G, int cap) {
    const size_t S = ((size_t)cap + 1 + 3) / 4 * 4;
    size_t prob = (size_t)G * S;
    size_t part = (size_t)(kDecodeThreads / 64) * G * kD;
    return (prob > part ? prob : part) * sizeof(float);
}

template <typename T, int GT>
static hipError_t launch_decode_step_t(const void* q, const void* k_new, const void* v_new, int n_heads, int G,
                                       const int32_t* pos, const int32_t* budget, int w, int cap, void* Kc,
                                       void* Vc, int32_t* idx, float* cum, int32_t* len, float* out,
                                       int32_t* evicted, const Env& env) {
    const int S = (cap + 1 + 3) / 4 * 4;
    const size_t lds = decode_step_lds_bytes(G, cap);
    auto kern = decode_step_kernel<T, GT>;
    if (lds > kDecodeStepLdsMax) return hipErrorInvalidValue;      // the interface checks G*(cap+1) before
    env.begin("decode_step");
    kern<<<n_heads, kDecodeThreads, lds, env.s>>>(static_cast<const T*>(q), static_cast<const T*>(k_new),
                                                  static_cast<const T*>(v_new), G, pos, budget, w, cap,
                                                  static_cast<T*>(Kc), static_cast<T*>(Vc), idx, cum, len, out,
                                                  evicted, S);
    env.end();
    return hipGetLastError();
}

hipError_t launch_decode_step(const void* q, const void* k_new, const void* v_new, uncomp_dtype dt,
                              int n_heads, int G, const int32_t* pos, const int32_t* budget, int w, int cap,
                              void* Kc, void* Vc, int32_t* idx, float* cum, int32_t* len, float* out,
                              int32_t* evicted, const Env& env) {
#define UNCOMP_DECODE_CASE(T, GT)                                                                          \
    return launch_decode_step_t<T, GT>(q, k_new, v_new, n_heads, G, pos, budget, w, cap, Kc, Vc, idx, cum, \
                                       len, out, evicted, env)
    if (dt == UNCOMP_BF16) {
        if (G <= 4) UNCOMP_DECODE_CASE(bf16_bits, 4);
        if (G <= 8) UNCOMP_DECODE_CASE(bf16_bits, 8);
        UNCOMP_DECODE_CASE(bf16_bits, 16);
    }
    if (G <= 4) UNCOMP_DECODE_CASE(float, 4);
    if (G <= 8) UNCOMP_DECODE_CASE(float, 8);
    UNCOMP_DECODE_CASE(float, 16);
#undef UNCOMP_DECODE_CASE
}

template <typename T, int GT>
static hipError_t allow_decode_step() {
    return allow_dynamic_lds(reinterpret_cast<const void*>(decode_step_kernel<T, GT>), kDecodeStepLdsMax);
}

// the tables may fill the default limit by themselves, and the kernels have a few hundred bytes besides
template <int GT>
static hipError_t allow_decode_update() {
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(decode_update_kernel<GT, 256, false>), kLdsDefaultLimit);
    if (e == hipSuccess) e = allow_dynamic_lds(reinterpret_cast<const void*>(decode_update_kernel<GT, 512, false>), kLdsDefaultLimit);
    return e == hipSuccess ? allow_dynamic_lds(reinterpret_cast<const void*>(update_few<GT>(false)), kLdsDefaultLimit) : e;
}

template <int GT>
static hipError_t allow_decode_head() {
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(decode_head_kernel<GT, 2>), kDecodeHeadLdsMax);
    if (e == hipSuccess) e = allow_dynamic_lds(reinterpret_cast<const void*>(decode_head_kernel<GT, 4>), kDecodeHeadLdsMax);
    return e == hipSuccess ? allow_dynamic_lds(reinterpret_cast<const void*>(decode_head_kernel<GT, 8>), kDecodeHeadLdsMax) : e;
}

hipError_t init_decode_kernels() {
    hipError_t e = allow_decode_step<bf16_bits, 4>();
    if (e == hipSuccess) e = allow_decode_step<bf16_bits, 8>();
    if (e == hipSuccess) e = allow_decode_step<bf16_bits, 16>();
    if (e == hipSuccess) e = allow_decode_step<float, 4>();
    if (e == hipSuccess) e = allow_decode_step<float, 8>();
    if (e == hipSuccess) e = allow_decode_step<float, 16>();
    if (e == hipSuccess) e = allow_decode_update<4>();
    if (e == hipSuccess) e = allow_decode_update<8>();
    if (e == hipSuccess) e = allow_decode_update<16>();
    if (e == hipSuccess) e = allow_decode_head<4>();
    if (e == hipSuccess) e = allow_decode_head<8>();
    return e;
}

}  // namespace uncomp
