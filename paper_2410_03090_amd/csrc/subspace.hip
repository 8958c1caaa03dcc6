// Truncated matrix entropy of wide token matrices (Sec. 3.1 Eq. 1, Lemma 2; Sec. 3.2 Eq. 5-6 for
// D = 256 ... 8192, e.g. the hidden states H_m of Sec. 3.3.2) without the eigenvalues of the whole
// D x D covariance: only the k largest enter Eq. 5, and those are the Ritz values of a
// 128-dimensional subspace that block power iteration drives onto the dominant eigenvectors.
//
//   x_bar = mean token, C = sum_t (x_t - x_bar)(x_t - x_bar)^T
//   Q_0   = fixed pseudo-random D x 128 block
//   repeat:  Z = X Q  (N x 128),  W = C Q = X^T Z - s (s^T Q)/N  (D x 128),  Q = orth(W)
//   end:     Z = X Q;  the centred covariance of the N projected tokens z_t is Q^T C Q, whose
//            eigenvalues (the ordinary 128-wide entropy path) are the Ritz values; Eq. 5 without
//            renormalisation divides them by trace(C), which one pass over X provides.
//
// An iteration over the tokens reads X twice (HBM-bound: 2 N D e bytes) and costs 4 N D 128 flops.
// Forming C (covariance.hip, bf16 matrices) costs N D^2 once, on the matrix cores, after which an
// iteration reads 4 D^2 bytes: cov_pays() tells which is less time.  orth() is a Cholesky QR with the 128 x 128 Gram of W accumulated in fp64;
// a pivot that vanishes (rank below 128) retires its column.  Convergence of the k-th value goes
// with (lambda_129 / lambda_k)^(2 iterations): fast when the spectrum falls off before the 129th
// eigenvalue, as it does for the matrices the method looks at (that fall-off is the paper's point).
#include "common.h"
#include "device_utils.h"

namespace uncomp {

namespace {

constexpr int kP = 128;                  // width of the iterated block

__device__ __forceinline__ float elem(const bf16_bits* p) { return bf16_to_f32(*p); }
__device__ __forceinline__ float elem(const float* p) { return *p; }

// splitmix-style hash -> value in [-1, 1): the start block must be the same on every run
__device__ __forceinline__ float start_value(uint32_t d, uint32_t j) {
    uint64_t z = ((uint64_t)d << 32 | j) + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (float)((double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0);
}

}  // namespace

// The start block, and as Rinv the multiple of the identity that gives its columns a norm of about one.  A random block is
// well conditioned as it is (singular values within a factor of six even at 256 features), and what the first round
// needs is its span: orthonormalising it too was one Cholesky step in ten, 75 us.
__global__ __launch_bounds__(256) void sub_start_kernel(float* __restrict__ W, int D, float* __restrict__ Rinv) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < D * kP) W[e] = start_value((uint32_t)(e / kP), (uint32_t)(e % kP));
    if (e < kP * kP) Rinv[e] = e / kP == e % kP ? sqrtf(3.f / (float)D) : 0.f;      // D >= 128: one thread per entry
}

// Column sums and sums of squares of X over a chunk of tokens, in fp64: part[chunk][2][D].
// A workgroup covers 512 columns: thread = 8 consecutive columns (read with load8) x one of four row phases,
// eight rows in flight per thread; the four phases are added up in LDS in a fixed order.
template <typename T>
__global__ __launch_bounds__(256) void sub_colstats_kernel(const T* __restrict__ X, int N, int D, int64_t ldx,
                                                           int chunk, double* __restrict__ part) {
    __shared__ double red[3][16][64];
    const int cg = threadIdx.x & 63, ph = threadIdx.x >> 6;
    const int d = (blockIdx.x * 64 + cg) * 8;
    const int c = blockIdx.y;
    const bool live = d < D;
    const int t0 = c * chunk, t1 = min(N, t0 + chunk);
    double s[8], q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] = q[i] = 0.0;
    if (live) {
        for (int t = t0 + ph; t < t1; t += 32) {
            float v[8][8];
#pragma unroll
            for (int u = 0; u < 8; ++u) load8(X + (int64_t)min(t + 4 * u, t1 - 1) * ldx + d, v[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (t + 4 * u < t1) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const double x = (double)v[u][i];
                        s[i] += x;
                        q[i] = fma(x, x, q[i]);
                    }
                }
            }
        }
    }
    if (ph > 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            red[ph - 1][i][cg] = s[i];
            red[ph - 1][8 + i][cg] = q[i];
        }
    }
    __syncthreads();
    if (ph == 0 && live) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            part[((int64_t)c * 2 + 0) * D + d + i] = ((s[i] + red[0][i][cg]) + red[1][i][cg]) + red[2][i][cg];
            part[((int64_t)c * 2 + 1) * D + d + i] = ((q[i] + red[0][8 + i][cg]) + red[1][8 + i][cg]) + red[2][8 + i][cg];
        }
    }
}

// s[d] = sum over chunks; tpart[wg] = this workgroup's share of (sum_d (q_d - s_d^2 / N), sum_d q_d).
__global__ __launch_bounds__(256) void sub_colstats_finish_kernel(const double* __restrict__ part, int n_chunks, int D,
                                                                  int N, double* __restrict__ s,
                                                                  double* __restrict__ tpart) {
    __shared__ double red[2][4];
    const int d = blockIdx.x * 256 + threadIdx.x;
    double tc = 0.0, tu = 0.0;
    if (d < D) {
        double a = 0.0, q = 0.0;
#pragma unroll 8
        for (int c = 0; c < n_chunks; ++c) {
            a += part[((int64_t)c * 2 + 0) * D + d];
            q += part[((int64_t)c * 2 + 1) * D + d];
        }
        s[d] = a;
        tc = q - a * a / (double)N;
        tu = q;
    }
    tc = wave_sum(tc);
    tu = wave_sum(tu);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = tc;
        red[1][threadIdx.x >> 6] = tu;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        tpart[2 * blockIdx.x + 0] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
        tpart[2 * blockIdx.x + 1] = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    }
}
// trace[0] = centred, trace[1] = uncentred trace: the workgroups' shares added in order.
__global__ void sub_trace_kernel(const double* __restrict__ tpart, int n, double* __restrict__ trace) {
    if (threadIdx.x < 2) {
        double t = 0.0;
        for (int i = 0; i < n; ++i) t += tpart[2 * i + threadIdx.x];
        trace[threadIdx.x] = t;
    }
}

// Tall-skinny product with 128 output columns, fp32 accumulation on the plain ALUs.
//   A_KM == false:  out[m][j] = sum_k A[m][k] B[k][j]      (A is M x K, row stride lda)       Z = X Q
//   A_KM == true :  out[m][j] = sum_k A[k][m] B[k][j]      (A is K x M, row stride lda)       W = X^T Z
// blockIdx.x: 64 rows of the output, blockIdx.y: a chunk of k (partial results out[chunk][M][128]).
// B is fp32, K x 128, row stride 128.  A workgroup stages 16 k at a time in LDS; a thread owns
// 4 rows x 8 columns.
template <typename T, bool A_KM>
__global__ __launch_bounds__(256) void sub_gemm_kernel(const T* __restrict__ A, int64_t lda, const float* __restrict__ B,
                                                       int M, int K, int k_chunk, float* __restrict__ out) {
    __shared__ float As[16][64 + 4];
    __shared__ __align__(16) float Bs[16][kP];
    const int m0 = blockIdx.x * 64;
    const int kc = blockIdx.y;
    const int k_begin = kc * k_chunk, k_end = min(K, k_begin + k_chunk);
    const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
    float acc[4][8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
    for (int k0 = k_begin; k0 < k_end; k0 += 16) {
        // stage A: 64 rows x 16 k (four elements per thread)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int idx = tid + 256 * e;
            int m, k;
            if (A_KM) {
                m = idx & 63;
                k = idx >> 6;
            } else {
                k = idx & 15;
                m = idx >> 4;
            }
            float v = 0.f;
            if (m0 + m < M && k0 + k < k_end)
                v = A_KM ? elem(A + (int64_t)(k0 + k) * lda + m0 + m) : elem(A + (int64_t)(m0 + m) * lda + k0 + k);
            As[k][m] = v;
        }
        // stage B: 16 k x 128 (eight floats per thread)
        {
            const int k = tid >> 4, j = (tid & 15) * 8;
            float4 b0 = make_float4(0.f, 0.f, 0.f, 0.f), b1 = b0;
            if (k0 + k < k_end) {
                b0 = *reinterpret_cast<const float4*>(B + (int64_t)(k0 + k) * kP + j);
                b1 = *reinterpret_cast<const float4*>(B + (int64_t)(k0 + k) * kP + j + 4);
            }
            *reinterpret_cast<float4*>(&Bs[k][j]) = b0;
            *reinterpret_cast<float4*>(&Bs[k][j + 4]) = b1;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            float a[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = As[k][4 * ty + i];
            const float4 b0 = *reinterpret_cast<const float4*>(&Bs[k][8 * tx]);
            const float4 b1 = *reinterpret_cast<const float4*>(&Bs[k][8 * tx + 4]);
            const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    float* o = out + (int64_t)kc * M * kP;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + 4 * ty + i;
        if (m < M) {
            *reinterpret_cast<float4*>(o + (int64_t)m * kP + 8 * tx) = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
            *reinterpret_cast<float4*>(o + (int64_t)m * kP + 8 * tx + 4) = make_float4(acc[i][4], acc[i][5], acc[i][6], acc[i][7]);
        }
    }
}

// Q = W Rinv for 32 rows of W per workgroup (fp32 matrix instructions), together with what the next round needs of Q besides:
// its transposed bf16 halves Qt_hi / Qt_lo
// [128][D] (the operand that the MFMA version of Z = X Q streams; skipped when Qt_hi is null) and, when centring
// (s not null), this row block's share of s^T Q in fp64: zpart[block][128].  D is a multiple of 128.
// Bound by latency: Rinv goes to LDS whole, all of it in flight at once.  Rinv is upper triangular: a wave takes columns 16 w and
// on and the mirrored ones of the other end, and of the sum only the terms that are not zero.  6.6 us at D = 4096 (12.5 with the
// products on the fp32 ALUs, three LDS reads to sixteen of them; 14 with Rinv in pieces of sixteen rows).
constexpr int kQRows = 32;
constexpr int kRsLd = kP + 16;           // floats per row of Rinv in LDS: the four rows of an operand start 16 banks apart
constexpr size_t kQLdsBytes = (size_t)(kP * kRsLd + kQRows * (kP + 4)) * sizeof(float);
__global__ __launch_bounds__(256) void sub_q_kernel(const float* __restrict__ W, const float* __restrict__ Rinv, int D,
                                                    const double* __restrict__ s, float* __restrict__ Q,
                                                    uint16_t* __restrict__ Qt_hi, uint16_t* __restrict__ Qt_lo,
                                                    double* __restrict__ zpart) {
    extern __shared__ __align__(16) float qlds[];
    float(*Rs)[kRsLd] = reinterpret_cast<float(*)[kRsLd]>(qlds);
    float(*Ws)[kP + 4] = reinterpret_cast<float(*)[kP + 4]>(qlds + kP * kRsLd);
    float(*Qs)[kP + 1] = reinterpret_cast<float(*)[kP + 1]>(qlds);   // over Rs, once that has been read
    const int d0 = blockIdx.x * kQRows;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, c = lane & 15, kk = lane >> 4;
    {
        float4 wr[4], rr[16];
#pragma unroll
        for (int e = 0; e < 4; ++e) wr[e] = *reinterpret_cast<const float4*>(W + (int64_t)d0 * kP + 4 * (tid + 256 * e));
#pragma unroll
        for (int e = 0; e < 16; ++e) rr[e] = *reinterpret_cast<const float4*>(Rinv + 4 * (tid + 256 * e));
#pragma unroll
        for (int e = 0; e < 4; ++e) *reinterpret_cast<float4*>(&Ws[(tid + 256 * e) >> 5][4 * (tid & 31)]) = wr[e];
#pragma unroll
        for (int e = 0; e < 16; ++e) *reinterpret_cast<float4*>(&Rs[(tid + 256 * e) >> 5][4 * (tid & 31)]) = rr[e];
    }
    __syncthreads();
    const int J[2] = {7 - wv, wv};                                   // blocks of sixteen columns, the longer sum first
    f32x4_t acc[2][2];                                               // [column block][row block]
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[b][0] = acc[b][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int n_k = 16 * (J[b] + 1);
        for (int k0 = 0; k0 < n_k; k0 += 16) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + 4 * u + kk;
                const float r = Rs[k][16 * J[b] + c];
                acc[b][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(Ws[c][k], r, acc[b][0], 0, 0, 0);
                acc[b][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(Ws[16 + c][k], r, acc[b][1], 0, 0, 0);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * i + 4 * kk + v, col = 16 * J[b] + c;
                Q[(int64_t)(d0 + r) * kP + col] = acc[b][i][v];
                Qs[r][col] = acc[b][i][v];
            }
    __syncthreads();
    if (Qt_hi != nullptr) {
        // thread = (column, half of the 32 rows): 16 consecutive d of one column = 32 bytes per bf16 half
        const int col = tid >> 1, r0 = 16 * (tid & 1);
        uint32_t h[8], l[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float v0 = Qs[r0 + 2 * e][col], v1 = Qs[r0 + 2 * e + 1][col];
            const uint32_t h0 = __float_as_uint(v0), h1 = __float_as_uint(v1);
            const uint32_t hi0 = (h0 + 0x7fffu + ((h0 >> 16) & 1u)) >> 16, hi1 = (h1 + 0x7fffu + ((h1 >> 16) & 1u)) >> 16;   // round to nearest even
            const uint32_t g0 = __float_as_uint(v0 - __uint_as_float(hi0 << 16)), g1 = __float_as_uint(v1 - __uint_as_float(hi1 << 16));
            const uint32_t lo0 = (g0 + 0x7fffu + ((g0 >> 16) & 1u)) >> 16, lo1 = (g1 + 0x7fffu + ((g1 >> 16) & 1u)) >> 16;
            h[e] = hi0 | (hi1 << 16);
            l[e] = lo0 | (lo1 << 16);
        }
        uint4* ph = reinterpret_cast<uint4*>(Qt_hi + (int64_t)col * D + d0 + r0);
        uint4* pl = reinterpret_cast<uint4*>(Qt_lo + (int64_t)col * D + d0 + r0);
        ph[0] = make_uint4(h[0], h[1], h[2], h[3]);
        ph[1] = make_uint4(h[4], h[5], h[6], h[7]);
        pl[0] = make_uint4(l[0], l[1], l[2], l[3]);
        pl[1] = make_uint4(l[4], l[5], l[6], l[7]);
    }
    if (s != nullptr && tid < kP) {
        double t = 0.0;
#pragma unroll 8
        for (int r = 0; r < kQRows; ++r) t += s[d0 + r] * (double)Qs[r][tid];
        zpart[(int64_t)blockIdx.x * kP + tid] = t;
    }
}

// zsum[j] = sum_d s[d] Q[d][j] (= column sums of Z = X Q): the row blocks' shares added in a fixed order
// (eight interleaved partial sums side by side, then those in order).
__global__ __launch_bounds__(1024) void sub_zsum_kernel(const double* __restrict__ zpart, int n_parts, double* __restrict__ zsum) {
    __shared__ double part[8][kP];
    const int j = threadIdx.x & (kP - 1), q = threadIdx.x >> 7;
    double t = 0.0;
    for (int b = q; b < n_parts; b += 8) t += zpart[(int64_t)b * kP + j];
    part[q][j] = t;
    __syncthreads();
    if (q == 0) {
#pragma unroll
        for (int x = 1; x < 8; ++x) t += part[x][j];
        zsum[j] = t;
    }
}

// W[d][j] = sum over chunks of part[c][d][j] - s[d] zsum[j] / N   (the mean correction of C Q)
// Eight loads in flight per thread: 16 chunks at D = 4096 in 6.7 us (7.5 as a loop of single ones).
__global__ __launch_bounds__(256) void sub_reduce_kernel(const float* __restrict__ part, int n_chunks, int D,
                                                         const double* __restrict__ s, const double* __restrict__ zsum,
                                                         double inv_n, float* __restrict__ W) {
    const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 2;     // D is a multiple of 128: whole workgroups
    const float* p = part + e;
    double a = 0.0, b = 0.0;
    int c = 0;
    for (; c + 7 < n_chunks; c += 8) {
        float2 v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = *reinterpret_cast<const float2*>(p + (int64_t)(c + x) * D * kP);
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            a += (double)v[x].x;
            b += (double)v[x].y;
        }
    }
    for (; c < n_chunks; ++c) {
        const float2 v = *reinterpret_cast<const float2*>(p + (int64_t)c * D * kP);
        a += (double)v.x;
        b += (double)v.y;
    }
    if (s != nullptr) {
        a -= s[e / kP] * zsum[e % kP] * inv_n;
        b -= s[e / kP] * zsum[e % kP + 1] * inv_n;
    }
    *reinterpret_cast<float2*>(W + e) = make_float2((float)a, (float)b);
}

// Partial Gram of a tall fp32 matrix A (n_rows x 128) in fp64: gpart[slice][128][128] (+ the column sums of
// the slice in spart[slice][128] when asked for) on v_mfma_f64_16x16x4_f64.  Operands: lane l holds row /
// column l%16 at contraction index l/16; result register v of lane l: row 4v + l/16, column l%16.  The rows
// are staged in LDS 64 at a time as fp32 (next tile's loads in flight during the products) and widened on
// the way into the operands (exact).  Only the 36 tiles on and above the diagonal are computed, nine per
// wave (tile rows w and 7 - w); the write-out mirrors them.
constexpr int kGramRows = 64;
constexpr int kGramLd = 144;             // floats per staged row: four consecutive rows start 16 banks apart
constexpr int kGramTiles = 36;           // 16 x 16 tiles on and above the diagonal

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// PACKED (the Gram of the projected tokens, whose partials only feed an fp32 result): the 36 computed tiles go
// out as fp32, tile after tile (fpart[slice][36][16][16], tiles in the order (0,0) (0,1) ... (0,7) (1,1) ...),
// a quarter of the bytes of the mirrored fp64 matrix that the Cholesky step needs.
// MODE 2 (fp32 token matrices of uncomp_head_entropy, 128 features): blockIdx.y is the matrix (mat_stride elements
// apart, rows lda apart), blockIdx.x its token chunk; the chunk's mirrored Gram and column sums go out as fp32 in
// the layout the eigenvalue kernels add up: fpart[(matrix, chunk)][128][128], fsum[(matrix, chunk)][128].
// SLOTS: how many of a wave's nine tiles the workgroup computes, slots SLOTS * blockIdx.z and on.  A short fp32 prompt has
// one chunk per matrix, whose products keep a CU's fp64 matrix cores busy for 100 us: splitting the tiles over nine
// workgroups fills the chip without more partials, at the price of reading the tokens from the caches nine times.
// 8 matrices of 1024 tokens: 110 us with all nine slots, 31 with one.  Every entry is the same sum in the same order.
template <int MODE, int SLOTS = 9>
__global__ __launch_bounds__(256) void sub_gram64_kernel(const float* __restrict__ A_all, int64_t mat_stride, int64_t lda,
                                                         int n_rows, int rows_per_wg, double* __restrict__ gpart,
                                                         float* __restrict__ fpart, double* __restrict__ spart,
                                                         float* __restrict__ fsum) {
    constexpr bool PACKED = MODE == 1;
    __shared__ __align__(16) float rows[kGramRows][kGramLd];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int c = lane & 15, kk = lane >> 4;
    const float* A = A_all + (int64_t)blockIdx.y * mat_stride;
    const int64_t out_idx = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int r_begin = blockIdx.x * rows_per_wg;
    const int r_end = min(n_rows, r_begin + rows_per_wg);
    const int I1 = wv, I2 = 7 - wv, n1 = 8 - wv;             // slot s < n1: tile (I1, I1 + s); else (I2, I2 + s - n1)
    const int slot0 = SLOTS == 9 ? 0 : SLOTS * blockIdx.z;
    f64x4_t acc[SLOTS];
#pragma unroll
    for (int sl = 0; sl < SLOTS; ++sl) acc[sl] = f64x4_t{0.0, 0.0, 0.0, 0.0};
    double csum = 0.0;
    float4 pre[8];
    auto fetch = [&](int r0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int e = tid + 256 * i, rr = e >> 5, q = e & 31;
            pre[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (r0 + rr < r_end) pre[i] = *reinterpret_cast<const float4*>(A + (int64_t)(r0 + rr) * lda + 4 * q);
        }
    };
    if (r_begin < r_end) fetch(r_begin);
    for (int r0 = r_begin; r0 < r_end; r0 += kGramRows) {
        __syncthreads();                                      // the previous tile has been read
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int e = tid + 256 * i;
            *reinterpret_cast<float4*>(&rows[e >> 5][4 * (e & 31)]) = pre[i];
        }
        __syncthreads();
        if (r0 + kGramRows < r_end) fetch(r0 + kGramRows);
        if ((MODE == 2 ? slot0 == 0 : spart != nullptr) && tid < kP) {
#pragma unroll 8
            for (int rr = 0; rr < kGramRows; ++rr) csum += (double)rows[rr][tid];
        }
        for (int k0 = 0; k0 < kGramRows; k0 += 4) {
            const float* row = rows[k0 + kk];
            const double a1 = (double)row[16 * I1 + c], a2 = (double)row[16 * I2 + c];
#pragma unroll
            for (int sl = 0; sl < SLOTS; ++sl) {
                const bool first = slot0 + sl < n1;
                const int J = first ? I1 + slot0 + sl : I2 + slot0 + sl - n1;
                const double bv = (double)row[16 * J + c];
                acc[sl] = __builtin_amdgcn_mfma_f64_16x16x4f64(first ? a1 : a2, bv, acc[sl], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int sl = 0; sl < SLOTS; ++sl) {
        const bool first = slot0 + sl < n1;
        const int I = first ? I1 : I2, J = first ? I1 + slot0 + sl : I2 + slot0 + sl - n1;
        if constexpr (PACKED) {
            float* o = fpart + (out_idx * kGramTiles + (I * 8 - I * (I - 1) / 2 + J - I)) * 256;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[(4 * v + kk) * 16 + c] = (float)acc[sl][v];
        } else if constexpr (MODE == 2) {
            float* o = fpart + out_idx * kP * kP;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * I + 4 * v + kk, col = 16 * J + c;
                o[r * kP + col] = (float)acc[sl][v];
                if (I != J) o[col * kP + r] = (float)acc[sl][v];
            }
        } else {
            double* o = gpart + out_idx * kP * kP;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * I + 4 * v + kk, col = 16 * J + c;
                o[r * kP + col] = acc[sl][v];
                if (I != J) o[col * kP + r] = acc[sl][v];
            }
        }
    }
    if (MODE == 2) {
        if (slot0 == 0 && tid < kP) fsum[out_idx * kP + tid] = (float)csum;
    } else if (spart != nullptr && tid < kP) {
        spart[out_idx * kP + tid] = csum;
    }
}

// Gram partials of fp32 token matrices with 128 features for the 128-wide entropy path (see MODE 2 above):
// exact products, fp64 sums inside a chunk, on the fp64 matrix cores instead of the fp32 ALUs.
hipError_t launch_gram_f32_mfma(const float* X, int n_mat, int N, int64_t mat_stride, int64_t ldx, int n_chunks, int chunk,
                                float* gram_part, float* sum_part, hipStream_t s) {
    // the most workgroups per chunk that still leave the launch under two per CU
    const int64_t n = (int64_t)n_chunks * n_mat;
    const int split = n * 9 <= 512 ? 9 : (n * 3 <= 512 ? 3 : 1);
    auto kern = split == 9 ? sub_gram64_kernel<2, 1> : (split == 3 ? sub_gram64_kernel<2, 3> : sub_gram64_kernel<2>);
    kern<<<dim3((unsigned)n_chunks, (unsigned)n_mat, (unsigned)split), dim3(256), 0, s>>>(X, mat_stride, ldx, N, chunk, nullptr,
                                                                                  gram_part, nullptr, sum_part);
    return hipGetLastError();
}

// gsum = sum of the slices (fixed order); sixteen loads in flight per thread (64 slices: 4.6 us; 7.2 with four).
__global__ __launch_bounds__(256) void sub_gram64_sum_kernel(const double* __restrict__ gpart, int n_slices,
                                                             double* __restrict__ gsum) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    const double* g = gpart + e;
    double a = 0.0;
    int sl = 0;
    for (; sl + 15 < n_slices; sl += 16) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = g[(int64_t)(sl + u) * kP * kP];
#pragma unroll
        for (int u = 0; u < 16; ++u) a += v[u];
    }
    for (; sl < n_slices; ++sl) a += g[(int64_t)sl * kP * kP];
    gsum[e] = a;
}

// The sums for the Gram of the projected tokens, from the packed fp32 tiles, mirrored into the fp32 single-chunk
// layout that the 128-wide eigenvalue kernel reads: gram[128*128], then the column sums sums[128] (last block of
// the grid).  Slices are added in fp64 in a fixed order.
__global__ __launch_bounds__(256) void sub_zgram_finish_kernel(const float* __restrict__ fpart,
                                                               const double* __restrict__ spart, int n_slices,
                                                               float* __restrict__ gram, float* __restrict__ sums) {
    __shared__ double quarter[3][64];
    if (blockIdx.x == kP * kP / 64) {
        if (threadIdx.x < kP) {
            double a = 0.0;
#pragma unroll 8
            for (int sl = 0; sl < n_slices; ++sl) a += spart[(int64_t)sl * kP + threadIdx.x];
            sums[threadIdx.x] = (float)a;
        }
        return;
    }
    // a workgroup adds 64 entries: four quarters of the slices side by side (sixteen loads in flight per thread:
    // the sum is a chain of memory round trips, not of bytes), then the quarters in order
    const int i = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + i;
    const int r = e >> 7, col = e & (kP - 1);
    const int I = min(r, col) >> 4, J = max(r, col) >> 4;          // the tile that holds (r, col) or its mirror image
    const int ri = r <= col ? r : col, ci = r <= col ? col : r;    // inside an off-diagonal tile: (row of I, column of J)
    int at;
    if (I == J) at = (r & 15) * 16 + (col & 15);                    // diagonal tiles are stored whole
    else at = (ri & 15) * 16 + (ci & 15);
    const float* g = fpart + (int64_t)(I * 8 - I * (I - 1) / 2 + J - I) * 256 + at;
    const int64_t stride = (int64_t)kGramTiles * 256;
    const int per = (n_slices + 3) / 4;
    const int s0 = q * per, s1 = min(n_slices, s0 + per);
    double a = 0.0;
    int sl = s0;
    for (; sl + 15 < s1; sl += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = g[(sl + u) * stride];
#pragma unroll
        for (int u = 0; u < 16; ++u) a += (double)v[u];
    }
    for (; sl < s1; ++sl) a += (double)g[sl * stride];
    if (q > 0) quarter[q - 1][i] = a;
    __syncthreads();
    if (q == 0) gram[e] = (float)(((a + quarter[0][i]) + quarter[1][i]) + quarter[2][i]);
}

// 1 / sqrt(x) of a positive fp64 number: the hardware's estimate (2^-24) and one third-order step (the library function
// spends more on denormals and infinities, which a pivot above the tolerance of a finite Gram is not).
__device__ __forceinline__ double inv_sqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// One workgroup: Cholesky G = L L^T (fp64), then Rinv = L^-T as fp32 so that Q = W Rinv has orthonormal columns.  A pivot below
// 1e-12 of the largest diagonal entry retires its column (its row and column of Rinv are zero).
// The elimination runs on G with an identity below it, [G; I] L^-T = [L; L^-T], by columns of 16: whatever the step, 128 rows are
// in play, the rows of G that are left and the rows of I that are no longer zero, so that the inverse costs no phase of its own.
// Row slot r of block column K is the tile (r, K) of G for r >= K and that of I for r < K (tile (K, K) of I is the identity until
// its own step).  Two barriers a step:
//   factor   two waves, a lane per row: 16 pivots in registers.  Every row of 16 lanes also holds the diagonal block, a row a
//            lane, and reads its columns through the DPP broadcast.  The other six waves, which keep the tiles of the columns to
//            come in registers, apply the previous panel to those beyond the next column (v_mfma_f64_16x16x4_f64);
//   update   the next column's tiles get the new panel and go to LDS for the next step.
// Bound by the chain of the 128 pivots: 47 us before (the panel's rows and the diagonal block in one lane's registers, values of
// other rows by v_readlane, three barriers a step, then the inverse by block rows).
constexpr int kCholThreads = 512;
__global__ __launch_bounds__(kCholThreads) void sub_chol_kernel(const double* __restrict__ gsum, float* __restrict__ Rinv) {
    constexpr int B = 16, NB = kP / B, LD = B + 1, kRowWaves = kP / 64, kTileWaves = kCholThreads / 64 - kRowWaves;
    constexpr int kTiles = ((NB - 1) * NB + kTileWaves - 1) / kTileWaves;   // columns 1 .. 7, eight slots each
    __shared__ double raw[kP][LD], pan[2][kP][LD];                   // the column about to be factored; the factored ones
    __shared__ double maxdiag[kRowWaves];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, kk = lane >> 4, w = wv - kRowWaves;
    f64x4_t acc[kTiles];
    if (w >= 0) {
#pragma unroll
        for (int s = 0; s < kTiles; ++s) {
            const int t = w + kTileWaves * s, K = t / NB + 1, r = t % NB;
            acc[s] = f64x4_t{0.0, 0.0, 0.0, 0.0};
            if (K < NB && r >= K) {
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[s][v] = gsum[(B * r + 4 * v + kk) * kP + B * K + c];
            }
        }
    } else {
        const double2* g2 = reinterpret_cast<const double2*>(gsum + tid * kP);
        double2 v[B / 2];
#pragma unroll
        for (int k = 0; k < B / 2; ++k) v[k] = g2[k];
        double m = gsum[tid * (kP + 1)];
#pragma unroll
        for (int k = 0; k < B / 2; ++k) {
            raw[tid][2 * k] = v[k].x;
            raw[tid][2 * k + 1] = v[k].y;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
        if (lane == 0) maxdiag[wv] = m;
    }
    __syncthreads();
    const double tol = fmax(maxdiag[0], maxdiag[1]) * 1e-12;
    // tile (r, K) of a column beyond p minus panel rows r times panel rows K, transposed
    auto apply = [&](f64x4_t& x, int p, int r, int K) {
        double av[4], bv[4];
#pragma unroll
        for (int sx = 0; sx < 4; ++sx) {
            av[sx] = -pan[p & 1][B * r + c][4 * sx + kk];
            bv[sx] = pan[p & 1][B * K + c][4 * sx + kk];
        }
#pragma unroll
        for (int sx = 0; sx < 4; ++sx) x = __builtin_amdgcn_mfma_f64_16x16x4f64(av[sx], bv[sx], x, 0, 0, 0);
    };
    for (int p = 0; p < NB; ++p) {
        if (w < 0) {
            const int row = tid, slot = row >> 4;
            double d[B], a[B];                                       // row c of the diagonal block, this lane's row
#pragma unroll
            for (int k = 0; k < B; ++k) {
                d[k] = raw[B * p + c][k];
                a[k] = raw[row][k];
            }
#pragma unroll
            for (int k = 0; k < B; ++k) a[k] = slot == p ? (k == c ? 1.0 : 0.0) : a[k];
            // pivot j: row j of the diagonal block is in lane j of every row of lanes
            auto rows_from = [&](auto J, auto K0, auto K1, double dj) {      // columns K0 .. K1 - 1 minus their multiple of column J
                each16<K0.value, K1.value>([&](auto k) {
                    if constexpr (k.value > J.value + 1) fnmac_bc<k.value>(d[k.value], dj, dj);
                    if constexpr (k.value > J.value) fnmac_bc<k.value>(a[k.value], dj, a[J.value]);
                });
            };
            double piv = 0.0;
            dpp_ready(d[0], piv);
            fmac_bc<0>(piv, d[0], 1.0);
            double di = piv > tol ? inv_sqrt(piv) : 0.0;
            each16<0>([&](auto J) {
                constexpr int j = J.value;
                double dj = d[j] * di;
                a[j] *= di;
                piv = 0.0;
                dpp_ready(dj, piv);
                using I = std::integral_constant<int, j>;
                // the next pivot's chain, the other columns in its waits
                if constexpr (j + 1 < B) {
                    fnmac_bc<j + 1>(d[j + 1], dj, dj);
                    rows_from(I{}, std::integral_constant<int, j + 1>{}, std::integral_constant<int, (j + 3 < B ? j + 3 : B)>{}, dj);
                    dpp_ready(d[j + 1], piv);
                    fmac_bc<j + 1>(piv, d[j + 1], 1.0);
                    rows_from(I{}, std::integral_constant<int, (j + 3 < B ? j + 3 : B)>{}, std::integral_constant<int, (j + 5 < B ? j + 5 : B)>{}, dj);
                    const double y = __builtin_amdgcn_rsq(piv);
                    rows_from(I{}, std::integral_constant<int, (j + 5 < B ? j + 5 : B)>{}, std::integral_constant<int, (j + 8 < B ? j + 8 : B)>{}, dj);
                    const double e = fma(-piv * y, y, 1.0);
                    rows_from(I{}, std::integral_constant<int, (j + 8 < B ? j + 8 : B)>{}, std::integral_constant<int, (j + 11 < B ? j + 11 : B)>{}, dj);
                    di = piv > tol ? fma(y * e, fma(e, 0.375, 0.5), y) : 0.0;
                    rows_from(I{}, std::integral_constant<int, (j + 11 < B ? j + 11 : B)>{}, std::integral_constant<int, B>{}, dj);
                }
            });
#pragma unroll
            for (int k = 0; k < B; ++k) pan[p & 1][row][k] = a[k];
            float4* out = reinterpret_cast<float4*>(Rinv + row * kP + B * p);
#pragma unroll
            for (int k = 0; k < B; k += 4)
                out[k / 4] = slot <= p ? make_float4((float)a[k], (float)a[k + 1], (float)a[k + 2], (float)a[k + 3])
                                       : make_float4(0.f, 0.f, 0.f, 0.f);
        } else if (p > 0) {
#pragma unroll
            for (int s = 0; s < kTiles; ++s) {
                const int t = w + kTileWaves * s, K = t / NB + 1, r = t % NB;
                if (K < NB && K > p && (r >= K || r < p)) apply(acc[s], p - 1, r, K);
            }
        }
        __syncthreads();
        if (w >= 0 && p + 1 < NB) {
#pragma unroll
            for (int s = 0; s < kTiles; ++s) {
                const int t = w + kTileWaves * s, K = t / NB + 1, r = t % NB;
                if (K == p + 1) {
                    apply(acc[s], p, r, K);
#pragma unroll
                    for (int v = 0; v < 4; ++v) raw[B * r + 4 * v + kk][c] = acc[s][v];
                }
            }
        }
        __syncthreads();
    }
}

MatrixPlan plan_matrix(int N, int D) {
    MatrixPlan p;
    p.stat_chunks = N < 128 * 64 ? (N + 63) / 64 : 128;
    p.stat_chunk = (N + p.stat_chunks - 1) / p.stat_chunks;
    p.stat_chunks = (N + p.stat_chunk - 1) / p.stat_chunk;
    // split of the token sum in W = X^T Z: enough workgroups for the chip, partials kept modest
    const int row_blocks = (D + 63) / 64;
    int kc = (1024 + row_blocks - 1) / row_blocks;
    if (kc > 16) kc = 16;
    const int max_kc = (N + 255) / 256;
    if (kc > max_kc) kc = max_kc;
    if (kc < 1) kc = 1;
    p.w_chunk = ((N + kc - 1) / kc + 15) / 16 * 16;
    p.w_chunks = (N + p.w_chunk - 1) / p.w_chunk;
    // Gram of W: 64-row slices (one staged tile per workgroup); Gram of the projected tokens: one workgroup per CU at most, whole 64-row tiles each
    p.gram_rows = kGramRows;
    p.gram_slices = (D + p.gram_rows - 1) / p.gram_rows;
    p.zgram_rows = ((N + 255) / 256 + kGramRows - 1) / kGramRows * kGramRows;
    p.zgram_slices = (N + p.zgram_rows - 1) / p.zgram_rows;
    // the eigenvalue kernel reads one already summed chunk
    p.ep.n_chunks = 1;
    p.ep.chunk = N;
    p.ep.gram_off = 0;
    p.ep.sum_off = (size_t)kP * kP * sizeof(float);
    p.ep.bytes = p.ep.sum_off + (size_t)kP * sizeof(float);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    p.ep_off = take(p.ep.bytes);
    p.statpart_off = take((size_t)p.stat_chunks * 2 * D * sizeof(double));
    p.s_off = take((size_t)D * sizeof(double));
    p.trace_off = take((size_t)(2 + 2 * ((D + 255) / 256)) * sizeof(double));     // the traces, then per-workgroup shares
    p.zsum_off = take((size_t)(1 + D / kQRows) * kP * sizeof(double));     // the sums, then the row blocks' shares
    p.q_off = take((size_t)D * kP * sizeof(float));
    p.w_off = take((size_t)D * kP * sizeof(float));
    // token chunks of the MFMA version of W = X^T Z (whole rounds of 128 tokens)
    int tn = (512 + D / 128 - 1) / (D / 128);
    if (tn > 16) tn = 16;
    if (tn < 1) tn = 1;
    p.t_chunk = ((N + tn - 1) / tn + 127) / 128 * 128;
    p.t_chunks = (N + p.t_chunk - 1) / p.t_chunk;
    p.wpart_off = take((size_t)(p.w_chunks > p.t_chunks ? p.w_chunks : p.t_chunks) * D * kP * sizeof(float));
    p.z_off = take((size_t)N * kP * sizeof(float));
    const int max_slices = p.gram_slices > p.zgram_slices ? p.gram_slices : p.zgram_slices;
    p.gpart_off = take((size_t)(max_slices + 1) * kP * kP * sizeof(double));     // slices, then their sum
    p.spart_off = take((size_t)p.zgram_slices * kP * sizeof(double));
    p.rinv_off = take((size_t)kP * kP * sizeof(float));
    // bf16 MFMA products: Q^T as two bf16 halves, partial Z of the split over d
    const int row_wgs = (N + 255) / 256;
    int zs = (512 + row_wgs - 1) / row_wgs;
    if (zs > 8) zs = 8;
    if (zs > D / 256) zs = D / 256;
    if (zs < 1) zs = 1;
    p.z_splits = zs;
    p.qt_off = take((size_t)2 * kP * D * sizeof(bf16_bits));
    p.zpart_off = take(zs > 1 ? (size_t)zs * N * kP * sizeof(float) : 0);
    p.zsplit_off = take((((size_t)N + 127) / 128 * 128) * kP * sizeof(bf16_bits));      // Z^T rounded to bf16
    p.bytes = off;
    p.cov = plan_cov(N, D);
    // one workgroup of 128 rows per CU, at least 256 features each (twice the splits: 4 % more time in all at D = 2048 for the
    // partials to add up, 2 % at 1024, 1 % either way at 4096)
    p.c_splits = 256 * 128 / (2 * D);
    if (p.c_splits > D / 256) p.c_splits = D / 256;
    if (p.c_splits < 1) p.c_splits = 1;
    p.cov_off = take(p.cov.cov_bytes);
    const size_t c_part = (size_t)p.c_splits * 2 * D * kP * sizeof(float);      // partials of C Q, over those of C
    p.cov_part_off = take(p.cov.part_bytes > c_part ? p.cov.part_bytes : c_part);
    p.cov_total = off;
    return p;
}

// Whether C pays.  A round over the tokens reads X twice and writes Z in between, a round over C reads C once.  Their difference
// (us): measured 14 at 2048 tokens of 256 features, 15 at 4096 of 1024, 26 at 8192 of 4096, 130 at 32768 of 4096, 435 at 131072 of
// 4096; C itself 20, 29, 188, 564 and 2018.  Eight rounds at 8192 x 4096 are the line: 1170 us in all over X, 1148 over C;
// 131072 x 4096: 5049 and 3589, 131072 x 1024: 2682 and 1103; at 65536 x 8192 X is the better one (5442 and 6514).
bool cov_pays(const MatrixPlan& p, int N, int D, int n_iter) {
    const double gain = 12.0 + N * (3e-4 + 8e-7 * D) - 1e-6 * D * D;
    return p.cov.cost_us < 0.95 * n_iter * gain;
}

template <typename T>
static hipError_t run_matrix_entropy(const T* X, int n_mat, int N, int D, int64_t mat_stride, int64_t ldx,
                                     int k_trunc, unsigned flags, int n_iter, const MatrixPlan& p, char* ws, size_t ws_bytes,
                                     float* entropy_out, float* eig_out, const Env& env) {
    hipStream_t s = env.s;
    const bool center = (flags & UNCOMP_CENTER) != 0;
    double* statpart = reinterpret_cast<double*>(ws + p.statpart_off);
    double* sv = reinterpret_cast<double*>(ws + p.s_off);
    double* trace = reinterpret_cast<double*>(ws + p.trace_off);
    double* zsum = reinterpret_cast<double*>(ws + p.zsum_off);
    float* Q = reinterpret_cast<float*>(ws + p.q_off);
    float* W = reinterpret_cast<float*>(ws + p.w_off);
    float* Wpart = reinterpret_cast<float*>(ws + p.wpart_off);
    float* Z = reinterpret_cast<float*>(ws + p.z_off);
    double* gpart = reinterpret_cast<double*>(ws + p.gpart_off);
    double* gsum = gpart + (size_t)(p.gram_slices > p.zgram_slices ? p.gram_slices : p.zgram_slices) * kP * kP;
    double* spart = reinterpret_cast<double*>(ws + p.spart_off);
    float* Rinv = reinterpret_cast<float*>(ws + p.rinv_off);
    const unsigned dp_blocks = (unsigned)(((int64_t)D * kP + 255) / 256);
    // bf16 inputs with 16-byte aligned rows take the MFMA products, everything else the fp32 ALUs
    // (rows at most 2^22 elements apart: those kernels address 256 rows with 32-bit byte offsets)
    bool mfma = false;
    if constexpr (sizeof(T) == 2)
        mfma = !env.force_alu && (ldx % 8) == 0 && (mat_stride % 8) == 0 && (reinterpret_cast<uintptr_t>(X) & 15u) == 0 &&
               ldx <= ((int64_t)1 << 22);
    const bool use_cov = mfma && p.cov_total <= ws_bytes && cov_pays(p, N, D, n_iter);
    bf16_bits* Cs = reinterpret_cast<bf16_bits*>(ws + p.cov_off);
    float* cov_part = reinterpret_cast<float*>(ws + p.cov_part_off);
    bf16_bits* Qt_hi = reinterpret_cast<bf16_bits*>(ws + p.qt_off);
    bf16_bits* Qt_lo = Qt_hi + (size_t)kP * D;
    auto apply_rinv = [&]() {
        sub_q_kernel<<<dim3((unsigned)(D / kQRows)), dim3(256), kQLdsBytes, s>>>(W, Rinv, D, center ? sv : nullptr, Q,
                                                                       mfma ? Qt_hi : nullptr, Qt_lo, zsum + kP);
    };
    // Q = orth(W): Cholesky QR with the Gram in fp64; the last kernel also leaves the bf16 halves of Q^T and the
    // shares of s^T Q for the round that follows
    auto orth = [&]() {
        // a slice's tiles over as many workgroups as leave the launch under two per CU: D = 4096, 64 slices, 15 us with all
        // of a slice's tiles in one workgroup, 7.0 with a third; the sums are the same
        auto gram = p.gram_slices * 9 <= 512 ? sub_gram64_kernel<0, 1> : (p.gram_slices * 3 <= 512 ? sub_gram64_kernel<0, 3> : sub_gram64_kernel<0>);
        const unsigned split = p.gram_slices * 9 <= 512 ? 9u : (p.gram_slices * 3 <= 512 ? 3u : 1u);
        gram<<<dim3((unsigned)p.gram_slices, 1, split), dim3(256), 0, s>>>(W, 0, kP, D, p.gram_rows, gpart, nullptr, nullptr, nullptr);
        sub_gram64_sum_kernel<<<dim3(kP * kP / 256), dim3(256), 0, s>>>(gpart, p.gram_slices, gsum);
        sub_chol_kernel<<<dim3(1), dim3(kCholThreads), 0, s>>>(gsum, Rinv);
        apply_rinv();
    };
    float* Zpart = reinterpret_cast<float*>(ws + p.zpart_off);
    bf16_bits* Zt = reinterpret_cast<bf16_bits*>(ws + p.zsplit_off);
    hipError_t perr = hipSuccess;
    // Z is always rounded to bf16 on its way into W = X^T Z (2^-9 relative error per element, averaged over the
    // tokens of the sum); Q enters Z = X Q as its high bf16 half in all rounds but the last, and as both halves in
    // the last round and in the final projection.  What a round with rounded factors gets wrong is a small tilt of
    // the iterated subspace, which the next round removes like any other component outside the dominant subspace,
    // and the eigenvalues of the projection move only with the square of the tilt that is left (measured against
    // the fp64 reference: entropy off by 1.6e-6 relative at most; 5e-5 if the last round rounds Q as well; keeping
    // both halves of Z in the last round too changes nothing).
    const int first_precise = n_iter - 1;
    bool zsum_ready = false;                              // the last projection added up the shares of s^T Q as well
    auto project = [&](const T* Xm, bool precise, bool for_round) {       // Z = X Q
        zsum_ready = false;
        if constexpr (sizeof(T) == 2) {
            if (mfma) {
                hipError_t e = launch_xq_mfma(Xm, ldx, N, D, Qt_hi, Qt_lo, p.z_splits, Zpart, Z, s, precise, for_round, Zt,
                                              center ? zsum + kP : nullptr, D / kQRows, zsum, &zsum_ready);
                if (e != hipSuccess) perr = e;
                return;
            }
        }
        sub_gemm_kernel<T, false><<<dim3((unsigned)((N + 63) / 64), 1), dim3(256), 0, s>>>(Xm, ldx, Q, N, D, D, Z);
    };
    for (int m = 0; m < n_mat; ++m) {
        const T* Xm = X + (int64_t)m * mat_stride;
        env.begin("matrix_colstats");
        sub_colstats_kernel<T><<<dim3((unsigned)((D / 8 + 63) / 64), (unsigned)p.stat_chunks), dim3(256), 0, s>>>(
            Xm, N, D, ldx, p.stat_chunk, statpart);
        sub_colstats_finish_kernel<<<dim3((unsigned)((D + 255) / 256)), dim3(256), 0, s>>>(statpart, p.stat_chunks, D, N, sv,
                                                                                          trace + 2);
        sub_trace_kernel<<<dim3(1), dim3(64), 0, s>>>(trace + 2, (D + 255) / 256, trace);
        env.end();
        if constexpr (sizeof(T) == 2) {
            if (use_cov) {
                env.begin("matrix_covariance");
                hipError_t e = launch_cov(Xm, ldx, N, D, center ? sv : nullptr, p.cov, cov_part, Cs, s);
                if (e != hipSuccess) return e;
                env.end();
            }
        }
        env.begin("matrix_subspace");
        sub_start_kernel<<<dim3(dp_blocks), dim3(256), 0, s>>>(W, D, Rinv);
        apply_rinv();
        for (int it = 0; it < n_iter; ++it) {
            const bool precise = it >= first_precise;
            int w_parts = p.w_chunks;
            bool done = false;
            if (use_cov) {
                hipError_t e = launch_cq_mfma(Cs, D, Qt_hi, Qt_lo, p.c_splits, cov_part, precise, s, &w_parts);
                if (e != hipSuccess) return e;
                done = true;
            } else {
                project(Xm, precise, true);
                if (center && !zsum_ready) {
                    sub_zsum_kernel<<<dim3(1), dim3(1024), 0, s>>>(zsum + kP, D / kQRows, zsum);
                }
            }
            if constexpr (sizeof(T) == 2) {
                if (mfma && !done) {
                    hipError_t e = launch_xtz_mfma(Xm, ldx, N, D, Zt, p.t_chunk, p.t_chunks, Wpart, s);
                    if (e != hipSuccess) return e;
                    w_parts = p.t_chunks;
                    done = true;
                }
            }
            if (!done)
                sub_gemm_kernel<T, true><<<dim3((unsigned)((D + 63) / 64), (unsigned)p.w_chunks), dim3(256), 0, s>>>(
                    Xm, ldx, Z, D, N, p.w_chunk, Wpart);
            sub_reduce_kernel<<<dim3((unsigned)(D / 4)), dim3(256), 0, s>>>(use_cov ? cov_part : Wpart, w_parts, D,
                                                                    center && !use_cov ? sv : nullptr, zsum, 1.0 / (double)N, W);
            orth();
            if (it == n_iter - 1) {          // once more: the last Q is orthonormal to fp32 rounding
                hipError_t e = hipMemcpyAsync(W, Q, (size_t)D * kP * sizeof(float), hipMemcpyDeviceToDevice, s);
                if (e != hipSuccess) return e;
                orth();
            }
        }
        project(Xm, true, false);
        env.end();
        if (perr != hipSuccess) return perr;
        // the projected tokens go through the 128-wide entropy path; trace(C) replaces its own trace
        env.begin("matrix_gram");
        float* fpart = reinterpret_cast<float*>(gpart);          // the region of the fp64 slices, free by now
        sub_gram64_kernel<1><<<dim3((unsigned)p.zgram_slices), dim3(256), 0, s>>>(Z, 0, kP, N, p.zgram_rows, nullptr, fpart, spart, nullptr);
        sub_zgram_finish_kernel<<<dim3(kP * kP / 64 + 1), dim3(256), 0, s>>>(
            fpart, spart, p.zgram_slices, reinterpret_cast<float*>(ws + p.ep_off + p.ep.gram_off),
            reinterpret_cast<float*>(ws + p.ep_off + p.ep.sum_off));
        env.end();
        hipError_t e = launch_tridiag_entropy(1, N, k_trunc, flags, p.ep, ws + p.ep_off, entropy_out + m,
                                   eig_out != nullptr ? eig_out + (int64_t)m * kP : nullptr, env,
                                   trace);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

hipError_t launch_matrix_entropy(const void* X, uncomp_dtype dt, int n_mat, int N, int D, int64_t mat_stride,
                                 int64_t ldx, int k_trunc, unsigned flags, int n_iter, const MatrixPlan& p, char* ws,
                                 size_t ws_bytes, float* entropy_out, float* eig_out, const Env& env) {
    if (dt == UNCOMP_BF16)
        return run_matrix_entropy(static_cast<const bf16_bits*>(X), n_mat, N, D, mat_stride, ldx, k_trunc, flags, n_iter,
                                  p, ws, ws_bytes, entropy_out, eig_out, env);
    return run_matrix_entropy(static_cast<const float*>(X), n_mat, N, D, mat_stride, ldx, k_trunc, flags, n_iter, p, ws, ws_bytes,
                              entropy_out, eig_out, env);
}

hipError_t init_subspace_mfma_kernels();

hipError_t init_subspace_kernels() {
    hipError_t e = init_subspace_mfma_kernels();
    if (e != hipSuccess) return e;
    return allow_dynamic_lds(reinterpret_cast<const void*>(sub_q_kernel), kQLdsBytes);
}

}  // namespace uncomp
