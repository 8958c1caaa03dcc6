// Budgets from entropies (Sec. 3.3.3 "Design" and Eq. 11 for the head groups; Sec. 3.3.2
// Eq. 8-10 for the layer stages).  The work is a few hundred comparisons, so that its time is the
// launch: one kernel, whose first workgroup walks the layers while the others rank the heads of every
// (layer, batch) by counting.
#include "common.h"
#include "device_utils.h"

namespace uncomp {

namespace {
constexpr int kBudgetThreads = 1024, kBudgetWaves = kBudgetThreads / 64, kMaxLayers = 4096;
}

__device__ __forceinline__ void head_budgets(const float* __restrict__ entropy, int n_lb, int H, int M, int n_max, int step, int N,
                                             int w, int block, int n_blocks, int32_t* __restrict__ head_budget,
                                             int32_t* __restrict__ head_group) {
    const int total = n_lb * H;
    const int per = H / M;
    for (int e = block * kBudgetThreads + threadIdx.x; e < total; e += n_blocks * kBudgetThreads) {
        const int lb = e / H, h = e - lb * H;
        const float* row = entropy + (int64_t)lb * H;
        const float mine = row[h];
        int rank = 0;                         // heads that come before h: larger entropy, or equal and lower index
        for (int o = 0; o < H; ++o) {
            float v = row[o];
            rank += (v > mine || (v == mine && o < h)) ? 1 : 0;
        }
        const int g = rank / per;
        long long b = (long long)n_max - (long long)g * step;      // g*step may exceed 32 bits
        const long long lo = w < N ? w : N;
        b = b < lo ? lo : b;
        b = b > N ? N : b;
        head_budget[e] = (int32_t)b;
        head_group[e] = g;
    }
}

// One workgroup.  A wave per layer averages exp(entropy) in fp64: the exponentials side by side, their sum in index order
// (one thread for all 64 of a layer of eight prompts took 25 us).  Then the stage boundaries up to each layer are counted.
__device__ __forceinline__ void layer_stages(const float* __restrict__ entropy, int L, int BH, int N, int w, float eps, int delta_n,
                                             bool increase, int32_t* __restrict__ layer_group, int32_t* __restrict__ layer_tokens) {
    __shared__ double mean[kMaxLayers], part[kBudgetWaves][64];
    __shared__ int count[kMaxLayers / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int l = wave; l < L; l += kBudgetWaves) {
        double acc = 0.0;
        for (int i0 = 0; i0 < BH; i0 += 64) {
            if (i0 + lane < BH) part[wave][lane] = exp((double)entropy[(int64_t)l * BH + i0 + lane]);
            __builtin_amdgcn_wave_barrier();
            const int n = min(64, BH - i0);
            for (int i = 0; i < n; ++i) acc += part[wave][i];       // every lane the same sum
            __builtin_amdgcn_wave_barrier();
        }
        if (lane == 0) mean[l] = acc / (double)BH;
    }
    __syncthreads();
    auto boundary = [&](int l) {
        if (l <= 0 || l >= L) return false;
        double d = mean[l - 1] - mean[l];
        if (increase) d = -d;
        return d > (double)eps;
    };
    for (int l0 = 64 * wave; l0 < L; l0 += kBudgetThreads) {
        const unsigned long long m = __ballot(boundary(l0 + lane));
        if (lane == 0) count[l0 / 64] = __builtin_popcountll(m);
    }
    __syncthreads();
    for (int l0 = 64 * wave; l0 < L; l0 += kBudgetThreads) {
        const int l = l0 + lane;
        const unsigned long long m = __ballot(boundary(l));
        int c = __builtin_popcountll(m & (~0ull >> (63 - lane)));   // boundaries of these 64 layers up to this one
        for (int x = 0; x < l0 / 64; ++x) c += count[x];
        if (l < L) {
            layer_group[l] = c;
            const long long t = (long long)N - (long long)c * delta_n;
            layer_tokens[l] = t > w ? (int32_t)t : w;
        }
    }
}

__global__ __launch_bounds__(kBudgetThreads) void budget_kernel(
    const float* __restrict__ entropy, int L, int B, int H, int M, int n_max, int step, int N, int w, float eps, int delta_n,
    int increase, int32_t* __restrict__ head_budget, int32_t* __restrict__ head_group, int32_t* __restrict__ layer_group,
    int32_t* __restrict__ layer_tokens) {
    const int stage_blocks = layer_group != nullptr ? 1 : 0;
    if ((int)blockIdx.x < stage_blocks)
        layer_stages(entropy, L, B * H, N, w, eps, delta_n, increase != 0, layer_group, layer_tokens);
    else
        head_budgets(entropy, L * B, H, M, n_max, step, N, w, (int)blockIdx.x - stage_blocks, (int)gridDim.x - stage_blocks,
                     head_budget, head_group);
}

hipError_t launch_budgets(const float* entropy, int L, int B, int H, int M, int n_max, int step,
                          int N, int w, float eps, int delta_n, unsigned flags,
                          int32_t* head_budget, int32_t* head_group, int32_t* layer_group,
                          int32_t* layer_tokens, const Env& env) {
    if (L > kMaxLayers) return hipErrorInvalidValue;                // the interface checks before
    const int64_t total = (int64_t)L * B * H;
    int64_t blocks = head_budget != nullptr ? (total + kBudgetThreads - 1) / kBudgetThreads : 0;
    if (blocks > 1024) blocks = 1024;
    if (layer_group != nullptr) blocks += 1;
    env.begin("budgets");
    budget_kernel<<<dim3((unsigned)blocks), dim3(kBudgetThreads), 0, env.s>>>(
        entropy, L, B, H, M, n_max, step, N, w, eps, delta_n, (flags & UNCOMP_LAYER_DELTA_INCREASE) ? 1 : 0, head_budget,
        head_group, layer_group, layer_tokens);
    env.end();
    return hipGetLastError();
}

}  // namespace uncomp
