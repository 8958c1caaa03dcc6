// Eigen stage of the truncated matrix entropy (Lemma 2: entropy from the eigenvalues of
// the covariance; Sec. 3.2 Eq. 5: only the k largest enter; proof of Lemma 4: unit trace),
// by Householder tridiagonalisation and Sturm-sequence multisection, all in fp64.
//
// One workgroup of 256 threads per matrix:
//   1. add the Gram partials of the matrix in fp64, subtract the mean term s s^T / N
//      (Eq. 1; the common factor 1/(N-1) drops out under the unit-trace scaling) and divide
//      by the trace.  The matrix lives in registers: wave q holds the row blocks q and q + 4
//      (16 rows each), lane l their columns l and l + 64: 64 doubles per lane.
//   2. 126 Householder reflections H = I - beta v v^T bring it to tridiagonal form
//      (A <- A - v w^T - w v^T with p = beta A v, w = p - (beta/2)(v^T p) v).  Once 64 rows are left they move into the
//      registers of one wave, which goes on alone; a 64-wide matrix starts there.
//   3. The eigenvalues of the tridiagonal matrix (d, e) are found by counting sign changes of
//      the characteristic-polynomial recurrence p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}
//      (= number of eigenvalues below x; no division, rescaled every 16 terms): every
//      wanted eigenvalue owns a group of L lanes that cut its bracket into L+1 pieces per
//      round (ballot + count-trailing-zeros picks the piece).  Brackets start at
//      [0, 1 + 2^-10]: the matrix has unit trace and is positive semi-definite up to rounding,
//      and an eigenvalue that rounding pushed below zero is reported as zero, which is what
//      the definition asks for.  Only the k largest are computed unless the caller wants the
//      whole spectrum.
//   4. truncated entropy in fp64.
//
// What bounds step 2 is the serial chain of 126 reflections (latency, with one matrix per CU) and
// the number of vector instructions (with two), so both are kept short:
//   - Row values reach the lanes through the DPP broadcast inside rows of 16 lanes
//     (v_fmac_f64_dpp row_newbcast, the one DPP form the fp64 pipe has): a register pair whose lane
//     l%16 holds row 16b + l%16 serves the 16 rows of a block.  Reading the same values from LDS at
//     uniform addresses was one 128-bit read per FMA pair, which kept the LDS pipe busier than the
//     vector pipe and set the time of the launch.
//   - One barrier per reflection.  Before it every wave leaves its part of A x and the owner of row
//     i + 2 leaves that row; after it every wave forms the reflection's scalars, w, and rows i + 1
//     and i + 2 as the update will leave them (x and y of the next reflection) for itself, with the
//     same operations in the same order, so all waves hold identical bits and none waits for another.
//   - A wave's first row block is skipped once its rows are done.
// Measured: 8 matrices (one per CU) 132 us (133 with all reflections in four waves): 2630 cycles for each of the first 63
// reflections, 1420 for each of the last 63 (one wave, neither barriers nor exchange), 13 us for step 3; 5120 matrices 2.0 ms.  256 matrices of 64 columns 143 -> 51 us
// (before: all 126 reflections of the 128-wide matrix with zeros in half of its rows).
#include "common.h"
#include "device_utils.h"

namespace uncomp {

namespace {

constexpr int kTriThreads = 256, kTriWaves = kTriThreads / 64;
constexpr int kHalf = kD / 2;

struct TriSmem {
    double s[kD];            // column sums of X (for the mean correction)
    double red[kTriWaves];
    double pbuf[2][kTriWaves][kD];   // the waves' parts of A x, double buffered over reflections
    double zrow[2][kD];      // row i + 2
    double d[kD], e2[kD];    // diagonal; e2[i] = e_{i-1}^2, e_{-1} = 0
    double lam[kD];          // eigenvalues, descending
    double tail[kHalf][kHalf];   // the second half of the matrix, on its way into one wave
};

template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_rows(double v) {          // zero in the rows of 16 lanes that ROWS leaves out
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xF, false);
    return __hiloint2double(hi, lo);
}

// value of lane `l` (wave-uniform) in every lane
__device__ __forceinline__ double lane_value(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Sum over the 64 lanes, delivered to every lane with identical bits: rotations inside the rows of 16 lanes (DPP row_ror
// 8, 4, 2, 1), then the last lane of rows 0 and 2 to rows 1 and 3 and of row 1 to rows 2 and 3 (row_bcast 15 and 31), which
// leaves the total in lane 63.  (v_permlane32/16_swap for the last two steps: 8 cycles of the vector pipe each, four of them.)
// The steps depend on each other; `fill` is called between them and may bring in other work.
template <typename F>
__device__ __forceinline__ double wave_allsum(double v, F&& fill) {
    v += dpp_move<0x128>(v);
    fill();
    v += dpp_move<0x124>(v);
    fill();
    v += dpp_move<0x122>(v);
    fill();
    v += dpp_move<0x121>(v);
    fill();
    v += dpp_rows<0x142, 0xa>(v);
    fill();
    v += dpp_rows<0x143, 0xc>(v);
    return lane_value(v, 63);
}
__device__ __forceinline__ double wave_allsum(double v) { return wave_allsum(v, [] {}); }

__device__ __forceinline__ double block_sum(double v, double* red, int tid) {
    v = wave_allsum(v);
    __syncthreads();
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int x = 1; x < kTriWaves; ++x) t += red[x];
    return t;
}

// Number of eigenvalues of the tridiagonal matrix below x: sign changes along
// 1, p_0, p_1, ..., p_{n-1} (a zero takes the sign '+', which gives the same total as the
// textbook rule because the next term then has the opposite sign of the previous one).
// dr / er: d and e^2 of entries 16 j + lane%16, from entry FIRST on.  Signs are shifted into a word, 32 terms at a time.
template <int FIRST>
__device__ __forceinline__ int sturm_count(const double (&dr)[8], const double (&er)[8], double x) {
    double pp = 0.0, p = 1.0;                      // p_{-2}, p_{-1}
    int cnt = 0;
    uint32_t last = 0;
#pragma unroll
    for (int j2 = FIRST / 32; j2 < 4; ++j2) {
        uint32_t signs = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = 2 * j2 + h;
            each16<0>([&](auto U) {
                double t = -x * p;
                fnmac_bc<U.value>(t, er[j], pp);
                fmac_bc<U.value>(t, dr[j], p);
                signs = __builtin_amdgcn_alignbit(signs, (uint32_t)__double2hiint(t), 31);   // signs << 1 | sign of t
                pp = p;
                p = t;
            });
            // Cuts are 2^-32 apart, so |p| shrinks by about 2^-32 a step along a run of equal eigenvalues without coupling
            // (the zeros of a matrix of low rank) and grows by at most 1.25: from [1/2, 1) sixteen steps stay normal.
            const int ex = __builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(pp)));
            p = ldexp(p, -ex);
            pp = ldexp(pp, -ex);
        }
        cnt += __popc(signs ^ (signs >> 1 | last << 31));
        last = signs & 1u;
    }
    return cnt;
}

// The four blocks of 16 entries of a vector held as entry `lane`, each in every row of 16 lanes: the DPP operands of the rows.
// Through LDS: one write and four reads of a single wave, whose latency the caller fills; the same by v_permlane32/16_swap is
// twenty vector instructions, six of them of twelve cycles.
__device__ __forceinline__ void row_forms(double v, double* buf, int lane, double (&rf)[4]) {
    buf[lane] = v;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int b = 0; b < 4; ++b) rf[b] = buf[16 * b + (lane & 15)];
    __builtin_amdgcn_wave_barrier();
}

typedef double f64x16_t __attribute__((ext_vector_type(16)));

// Reflections of a 64 x 64 matrix in the registers of one wave: a[b][u] of lane l is entry (16 b + u, l).  x: the row before
// the first one in play (entries k and on), y: row k.  d[k] and e2[k] come out.  Rows k + 1 and on are in play: those from 16 J
// on in the loop that ends at 16 J + 14.  Bound by the chain from one row to the next (norm, square root and reciprocal beside
// the product, its dot product with the row, w): 1050 cycles a reflection with 16 rows in play, 1650 with 64; one wave alone
// issues a vector instruction every 5.4 cycles.  The update in two halves that fill the waits of the sums, as in the
// reflections of the whole matrix, measured the same.
template <int J>
__device__ __forceinline__ void tail_reflections(f64x16_t (&a)[4], double& x, double& y, int k, double* d, double* e2, double* buf,
                                                 int lane) {
    for (; k < 16 * J + 15; ++k) {
        // x = x1 at entry k and xt behind it; v = x - alpha e_k = v1 at entry k and xt behind it
        const double xt = lane > k ? x : 0.0;
        const double x1 = lane_value(x, k), yk = lane_value(y, k);
        double xr[4];
        row_forms(xt, buf, lane, xr);
        dpp_ready(xr[0], xr[1]);
        dpp_ready(xr[2], xr[3]);
        double p4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int b = J; b < 4; ++b)
            each16<0>([&](auto U) { fmac_bc<U.value>(p4[U.value & 3], xr[b], a[b][U.value]); });
        const double p = (p4[0] + p4[1]) + (p4[2] + p4[3]);             // A xt
        const double s0 = wave_allsum(xt * p);                          // xt^T A xt
        const double pk = lane_value(p, k);                             // (A xt)_k
        const double sigma = fma(x1, x1, wave_allsum(xt * xt));
        double rs = __builtin_amdgcn_rsq(sigma);
        const double t = sigma * rs, er = fma(-t, rs, 1.0);
        rs = fma(rs * er, fma(0.375, er, 0.5), rs);
        const double nrm = sigma * rs, den = fma(fabs(x1), nrm, sigma);
        double beta = __builtin_amdgcn_rcp(den);
        const double eb = fma(-den, beta, 1.0);
        beta = fma(beta, fma(eb, eb, eb), beta);
        const bool some = sigma > 0x1p-400;                             // as in the reflections of the whole matrix
        const double alpha = some ? (x1 >= 0.0 ? -nrm : nrm) : 0.0;
        beta = some ? beta : 0.0;
        const double v1 = x1 - alpha;
        const double vAv = fma(v1, fma(v1, yk, 2.0 * pk), s0);
        const double K = -0.5 * beta * beta * vAv;
        const double v = lane == k ? v1 : xt;
        const double w = fma(K, v, beta * fma(v1, y, p));               // beta A v + K v
        const double wk = lane_value(w, k);
        const double xn = fma(-v1, w, fma(-wk, v, y));                  // row k after the reflection
        double wr[4];
        row_forms(w, buf + kHalf, lane, wr);
        dpp_ready(wr[0], wr[1]);
        dpp_ready(wr[2], wr[3]);
#pragma unroll
        for (int b = J; b < 4; ++b) {
            each16<0>([&](auto U) {
                double e = a[b][U.value];
                fnmac_bc<U.value>(e, xr[b], w);
                fnmac_bc<U.value>(e, wr[b], xt);
                a[b][U.value] = e;
            });
        }
        if (lane == k) {
            d[k] = xn;
            e2[k] = sigma;
        }
        x = xn;
        y = a[J][k + 1 - 16 * J];
    }
}

}  // namespace

// HALF: the matrix has 64 rows and columns (the partial sums hold zeros beyond them), which take the part of the second half
// of a 128-wide one.
template <bool HALF>
__global__ __launch_bounds__(kTriThreads, 2) void tridiag_entropy_kernel(
    const float* __restrict__ gram_part, const float* __restrict__ sum_part, int n_chunks, int N,
    int k_trunc, unsigned flags, float* __restrict__ entropy_out, float* __restrict__ eig_out, int eig_ld,
    const double* __restrict__ trace_total) {
    __shared__ TriSmem sm;
    const int m = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int q = __builtin_amdgcn_readfirstlane(tid >> 6);      // this wave's row blocks: q and q + 4
    const float* Gm = gram_part + (int64_t)m * n_chunks * (kD * kD);
    const float* Sm = sum_part + (int64_t)m * n_chunks * kD;

    // ---- 1. reduce partials, centre, unit trace ------------------------------------------
    if (tid < kD) {
        double acc = 0.0;
        for (int ch = 0; ch < n_chunks; ++ch) acc += (double)Sm[ch * kD + tid];
        sm.s[tid] = acc;
    }
    __syncthreads();
    const bool center = (flags & UNCOMP_CENTER) != 0;
    const double inv_n = 1.0 / (double)N;
    double tr_c = 0.0, tr_u = 0.0;
    if (tid < kD) {
        double acc = 0.0;
        for (int ch = 0; ch < n_chunks; ++ch) acc += (double)Gm[(int64_t)ch * (kD * kD) + tid * (kD + 1)];
        tr_u = acc;
        tr_c = center ? acc - sm.s[tid] * sm.s[tid] * inv_n : acc;
    }
    const double trace = block_sum(tr_c, sm.red, tid);
    const double trace_u = block_sum(tr_u, sm.red, tid);
    // Zero spread: a single token, or a centred trace so far below the second moment that
    // the fp32 partial sums cannot tell it from zero.
    bool degenerate = !(trace > 0.0) || (center && (N < 2 || trace < trace_u * 0x1p-20));
    // A projection of a larger matrix: the verdict comes from the larger matrix' own traces
    // (centred, uncentred; accumulated in fp64), the projection of a constant matrix being noise.
    double whole_raw = 0.0;
    if (trace_total != nullptr) {
        whole_raw = center ? trace_total[0] : trace_total[1];
        degenerate = degenerate || !(whole_raw > 0.0) || (center && whole_raw < trace_total[1] * 0x1p-30);
    }
    if (degenerate) {
        if (tid == 0) entropy_out[m] = 0.f;
        if (eig_out != nullptr && tid < eig_ld) eig_out[(int64_t)m * eig_ld + tid] = 0.f;
        return;
    }
    constexpr int JS0 = HALF ? 1 : 0;                            // first row block and column half in use
    double a[2][2][16];                                          // a[j][s][u] = A[16 (q + 4 j) + u][lane + 64 s]
#pragma unroll
    for (int j = JS0; j < 2; ++j)
#pragma unroll
        for (int s = JS0; s < 2; ++s)
#pragma unroll
            for (int u = 0; u < 16; ++u) a[j][s][u] = 0.0;
    for (int ch = 0; ch < n_chunks; ++ch) {
        const float* g = Gm + (int64_t)ch * (kD * kD) + 16 * q * kD + lane;
        float t[2][2][16];                                       // a chunk's loads are all in flight
#pragma unroll
        for (int j = JS0; j < 2; ++j)
#pragma unroll
            for (int s = JS0; s < 2; ++s)
#pragma unroll
                for (int u = 0; u < 16; ++u) t[j][s][u] = g[(64 * (j - JS0) + u) * kD + 64 * (s - JS0)];
#pragma unroll
        for (int j = JS0; j < 2; ++j)
#pragma unroll
            for (int s = JS0; s < 2; ++s)
#pragma unroll
                for (int u = 0; u < 16; ++u) a[j][s][u] += (double)t[j][s][u];
    }
    {
        const double inv_tr = 1.0 / trace;
        const double sc[2] = {center ? sm.s[lane] * inv_n : 0.0, center ? sm.s[lane + 64] * inv_n : 0.0};
#pragma unroll
        for (int j = JS0; j < 2; ++j)
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double sr = sm.s[16 * q + 64 * (j - JS0) + u];
#pragma unroll
                for (int s = JS0; s < 2; ++s) a[j][s][u] = (a[j][s][u] - sr * sc[s - JS0]) * inv_tr;
            }
    }

    // ---- 2. Householder tridiagonalisation ---------------------------------------------------
    // Every wave carries x = row i (entries at columns <= i zeroed) and y = row i + 1, twice: as entries
    // lane + 64 s and as entries row0 + 64 j, the DPP operands of its row blocks.  Entries at done columns of
    // y, w and A, and done rows of A, hold finite leftovers that only ever meet zeros of x.
    //
    // With v = x - alpha e_{i+1}, A v = A x - alpha y and w = beta A v + K v, the update of what is still in
    // play (rows and columns > i + 1, where v = x) is A -= x (beta A v)^T + (beta A v + 2 K x) x^T: the first
    // half does not wait for K and fills the latency of the sum behind it; the second half and the next A x
    // fill that of the next reflection's norm and square root.  Row i + 3 is put into LDS behind the barrier of
    // reflection i, where the waves wait for their reads, as it stands before that reflection's update, which
    // the readers make up for one reflection later (xo, wo, xro, wro: x and w of the reflection before).
    double x_tail = 0.0, y_tail = 0.0;                           // row 63 and row 64, their second halves
    if constexpr (!HALF) {
        const int row0 = 16 * q + (lane & 15);
        double x[2], y[2], xr[2], yr[2], xo[2] = {0.0, 0.0}, w2r[2] = {0.0, 0.0};
        double wo[2] = {0.0, 0.0}, xro[2] = {0.0, 0.0}, wro[2] = {0.0, 0.0}, x3 = 0.0, w3 = 0.0;
        // Row `row` of the matrix (in the registers of one wave) to LDS: a switch on the wave-uniform register
        // number reaches it without indexing.  (Taking column `row` from one lane of every wave instead needs no
        // branches, but sixteen to thirty-two LDS writes of one lane each take 700 cycles.)
#define UNCOMP_TRI_CASE(K)                                               \
        case K:                                                              \
            to[lane] = a[(K) >> 4][0][(K) & 15];                                 \
            to[lane + 64] = a[(K) >> 4][1][(K) & 15];                            \
            asm volatile("; row %0" ::"n"(K)); /* the cases stay apart: merged, they would index the registers */ \
            break;
#define UNCOMP_TRI_CASE8(K)                                                                          \
        UNCOMP_TRI_CASE(K) UNCOMP_TRI_CASE(K + 1) UNCOMP_TRI_CASE(K + 2) UNCOMP_TRI_CASE(K + 3)          \
        UNCOMP_TRI_CASE(K + 4) UNCOMP_TRI_CASE(K + 5) UNCOMP_TRI_CASE(K + 6) UNCOMP_TRI_CASE(K + 7)
        auto publish = [&](int row, double* to) {
            if (((row >> 4) & 3) != q) return;
            switch ((row >> 6) * 16 + (row & 15)) {
                UNCOMP_TRI_CASE8(0) UNCOMP_TRI_CASE8(8) UNCOMP_TRI_CASE8(16) UNCOMP_TRI_CASE8(24)
                default:
                    break;
            }
        };
#undef UNCOMP_TRI_CASE8
#undef UNCOMP_TRI_CASE
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        publish(0, sm.pbuf[1][0]);
        publish(1, sm.pbuf[1][1]);
        publish(2, sm.zrow[0]);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            x[s] = sm.pbuf[1][0][lane + 64 * s];
            y[s] = sm.pbuf[1][1][lane + 64 * s];
            xr[s] = sm.pbuf[1][0][row0 + 64 * s];
            yr[s] = sm.pbuf[1][1][row0 + 64 * s];
        }
        if (tid == 0) {
            sm.d[0] = x[0];
            sm.e2[0] = 0.0;
        }
        if (lane == 0) x[0] = 0.0;
        if (row0 == 0) xr[0] = 0.0;

        // One reflection.  SPLIT: i = 61, 62, where entries i + 1 .. i + 3 lie in both halves; in the first one before.
        auto reflect = [&](auto SPLIT, int i) {
            auto entry = [&](const double (&v)[2], int r) {         // entry r of a vector held as entries lane + 64 s
                return lane_value(!SPLIT.value || r < 64 ? v[0] : v[1], r & 63);
            };
            double* pb = sm.pbuf[i & 1][0];
            double* zb = sm.zrow[i & 1];
            const bool top = 16 * q + 15 > i;            // this wave's first row block still in play
            double p[2][2] = {{0.0, 0.0}, {0.0, 0.0}};
            // pending second half of the previous update and the product A x on one row block, four FMAs a call
            dpp_ready(w2r[0], w2r[1]);
            dpp_ready(xr[0], xr[1]);
            auto chunk = [&](auto J, auto C) {
                constexpr int kPer = 8;                             // chunks of the update, then as many of the product
                constexpr int c = C.value % kPer, s = c / 4, u0 = 4 * (c % 4);
                if constexpr (C.value < kPer)
                    each16<u0, u0 + 4>([&](auto U) { fnmac_bc<U.value>(a[J.value][s][U.value], w2r[J.value], xo[s]); });
                else                                                // two chains of the product side by side
                    each16<2 * c, 2 * c + 2>([&](auto U) {
                        fmac_bc<U.value>(p[J.value][0], xr[J.value], a[J.value][0][U.value]);
                        fmac_bc<U.value>(p[J.value][1], xr[J.value], a[J.value][1][U.value]);
                    });
            };
            // sigma = |x|^2, alpha = -sign(x_{i+1}) |x|, beta = 1 / (sigma + |x_{i+1}| |x|); e_i^2 = sigma.  The
            // hardware estimates (2^-24) are brought to full precision by one third-order step each.
            const double x1 = entry(x, i + 1), x2 = entry(x, i + 2);
            const double y1 = entry(y, i + 1);
            double sigma = fma(x[0], x[0], x[1] * x[1]);
#define UNCOMP_CHUNK(c) chunk(I1{}, std::integral_constant<int, (c)>{})
            int n_fill = 0;
            auto fill = [&] {
                if (n_fill == 0) UNCOMP_CHUNK(0);
                if (n_fill == 1) UNCOMP_CHUNK(1);
                if (n_fill == 2) UNCOMP_CHUNK(2);
                if (n_fill == 3) UNCOMP_CHUNK(3);
                if (n_fill == 4) UNCOMP_CHUNK(4);
                ++n_fill;
            };
            sigma = wave_allsum(sigma, fill);
            UNCOMP_CHUNK(5);
            double rs = __builtin_amdgcn_rsq(sigma);
            UNCOMP_CHUNK(6);
            const double t = sigma * rs;
            UNCOMP_CHUNK(7);
            const double er = fma(-t, rs, 1.0);
            UNCOMP_CHUNK(8);
            rs = fma(rs * er, fma(0.375, er, 0.5), rs);
            UNCOMP_CHUNK(9);
            const double nrm = sigma * rs;
            UNCOMP_CHUNK(10);
            const double den = fma(fabs(x1), nrm, sigma);
            UNCOMP_CHUNK(11);
            double beta = __builtin_amdgcn_rcp(den);
            UNCOMP_CHUNK(12);
            const double eb = fma(-den, beta, 1.0);
            UNCOMP_CHUNK(13);
            beta = fma(beta, fma(eb, eb, eb), beta);
            UNCOMP_CHUNK(14);
            UNCOMP_CHUNK(15);
#undef UNCOMP_CHUNK
            // Nothing to reflect: beta = 0 leaves the matrix as it is.  The trace is one, so entries below 2^-200 are nothing,
            // and beta^2 ~ sigma^-2 stays finite: a matrix with zero rows left residues of 1e-160, infinities and then NaN.
            const bool some = sigma > 0x1p-400;
            const double alpha = some ? (x1 >= 0.0 ? -nrm : nrm) : 0.0;
            beta = some ? beta : 0.0;
            if (top) each16<0>([&](auto C) { chunk(I0{}, C); });
            pb[q * kD + lane] = p[0][0] + p[1][0];
            pb[q * kD + lane + 64] = p[0][1] + p[1][1];
            if (tid == 0) sm.e2[i + 1] = sigma;
            __syncthreads();

            double wb[2], wbr[2], z[2], zr[2], pc[2][4], pr[2][4], sum = 0.0;           // wb = beta A v
            double p_own[2];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    pc[s][t] = pb[t * kD + lane + 64 * s];
                    pr[s][t] = pb[t * kD + row0 + 64 * s];
                }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                z[s] = zb[lane + 64 * s];
                zr[s] = zb[row0 + 64 * s];
            }
            __builtin_amdgcn_sched_barrier(0);                      // the reads are on their way
            publish(i + 3, sm.zrow[(i + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                p_own[s] = (pc[s][0] + pc[s][1]) + (pc[s][2] + pc[s][3]);
                const double p_row = (pr[s][0] + pr[s][1]) + (pr[s][2] + pr[s][3]);
                sum = fma(x[s], p_own[s], sum);
                wb[s] = beta * fma(-alpha, y[s], p_own[s]);
                wbr[s] = beta * fma(-alpha, yr[s], p_row);
            }
            const double p1 = entry(p_own, i + 1);
            int n_fill2 = 0;
            auto first = [&](auto J, auto S, auto U0) {             // A -= x (beta A v)^T, four rows of one column half
                each16<U0.value, U0.value + 4>([&](auto U) { fnmac_bc<U.value>(a[J.value][S.value][U.value], xr[J.value], wb[S.value]); });
            };
            auto fill2 = [&] {
                if (n_fill2 == 0) first(I1{}, I1{}, std::integral_constant<int, 0>{});
                if (n_fill2 == 1) first(I1{}, I1{}, std::integral_constant<int, 4>{});
                if (n_fill2 == 2) first(I1{}, I1{}, std::integral_constant<int, 8>{});
                if (n_fill2 == 3) first(I1{}, I1{}, std::integral_constant<int, 12>{});
                if (n_fill2 == 4) first(I1{}, I0{}, std::integral_constant<int, 0>{});
                ++n_fill2;
            };
            sum = wave_allsum(sum, fill2);
            // v^T A v = x^T A x - 2 alpha (A x)_{i+1} + alpha^2 A_{i+1,i+1}
            const double vAv = fma(alpha, fma(alpha, y1, -2.0 * p1), sum);
            first(I1{}, I0{}, std::integral_constant<int, 4>{});
            const double K = -0.5 * beta * beta * vAv;
            const double v1 = x1 - alpha, w1 = fma(K, v1, beta * fma(-alpha, y1, p1));
            first(I1{}, I0{}, std::integral_constant<int, 8>{});
            double w[2], wr[2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                w[s] = fma(K, x[s], wb[s]);
                wr[s] = fma(K, xr[s], wbr[s]);
                w2r[s] = fma(K, xr[s], wr[s]);
            }
            first(I1{}, I0{}, std::integral_constant<int, 12>{});
            if (top) {
                each16<0>([&](auto U) { fnmac_bc<U.value>(a[0][0][U.value], xr[0], wb[0]); });
                each16<0>([&](auto U) { fnmac_bc<U.value>(a[0][1][U.value], xr[0], wb[1]); });
            }
            // row i + 2 as the previous update left it, then rows i + 1 and i + 2 as this one leaves them
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                z[s] = fma(-x3, wo[s], fma(-w3, xo[s], z[s]));
                zr[s] = fma(-x3, wro[s], fma(-w3, xro[s], zr[s]));
            }
            const double w2 = entry(w, i + 2);
            if (tid == 0) sm.d[i + 1] = fma(-2.0 * v1, w1, y1);
            x3 = entry(x, i + 3);
            w3 = entry(w, i + 3);
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const double xn = fma(-v1, w[s], fma(-w1, x[s], y[s])), xnr = fma(-v1, wr[s], fma(-w1, xr[s], yr[s]));
                y[s] = fma(-x2, w[s], fma(-w2, x[s], z[s]));
                yr[s] = fma(-x2, wr[s], fma(-w2, xr[s], zr[s]));
                xo[s] = x[s];
                wo[s] = w[s];
                xro[s] = xr[s];
                wro[s] = wr[s];
                x[s] = lane + 64 * s > i + 1 ? xn : 0.0;
                xr[s] = row0 + 64 * s > i + 1 ? xnr : 0.0;
            }
        };
        for (int i = 0; i < 61; ++i) reflect(std::false_type{}, i);
        for (int i = 61; i < 63; ++i) reflect(std::true_type{}, i);
        // the second half of what is pending on rows and columns 64 and on, which are all that is in play now
        dpp_ready(w2r[0], w2r[1]);
        each16<0>([&](auto U) { fnmac_bc<U.value>(a[1][1][U.value], w2r[1], xo[1]); });
        x_tail = x[1];
        y_tail = y[1];
    }
    // The last 64 rows and columns: one wave keeps them in registers and needs neither LDS nor barriers.
#pragma unroll
    for (int u = 0; u < 16; ++u) sm.tail[16 * q + u][lane] = a[1][1][u];
    if (HALF && tid < kHalf) sm.d[tid] = 0.0;
    __syncthreads();
    if (q == 0) {
        f64x16_t t[4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int u = 0; u < 16; ++u) t[b][u] = sm.tail[16 * b + u][lane];
        double* d = sm.d + kHalf;
        double* e2 = sm.e2 + kHalf;
        if constexpr (HALF) {                                    // the first row is there, nothing was reflected yet
            x_tail = t[0][0];
            y_tail = t[0][1];
            if (lane == 0) {
                d[0] = x_tail;
                e2[0] = 0.0;
            }
        }
        tail_reflections<0>(t, x_tail, y_tail, HALF ? 1 : 0, d, e2, sm.lam, lane);
        tail_reflections<1>(t, x_tail, y_tail, 15, d, e2, sm.lam, lane);
        tail_reflections<2>(t, x_tail, y_tail, 31, d, e2, sm.lam, lane);
        tail_reflections<3>(t, x_tail, y_tail, 47, d, e2, sm.lam, lane);
        if (lane == kHalf - 1) {                                 // x: row 62, y: row 63
            d[kHalf - 1] = y_tail;
            e2[kHalf - 1] = x_tail * x_tail;
        }
    }
    __syncthreads();
    if (tid < kD) sm.lam[tid] = 0.0;
    __syncthreads();

    // ---- 3. eigenvalues by multisection on the Sturm count ------------------------------------
    const int k = k_trunc < kD ? k_trunc : kD;
    constexpr int kN = HALF ? kHalf : kD;                        // rows that are there: the eigenvalues beyond them stay zero
    const int n_need = eig_out != nullptr || k > kN ? kN : k;
    // lanes per eigenvalue: as many as the workgroup can give every wanted eigenvalue
    const int L = kTriThreads / 8 >= n_need ? 8 : (kTriThreads / 4 >= n_need ? 4 : 2);
    const int rounds = L == 8 ? 10 : (L == 4 ? 14 : 20);         // (L+1)^rounds >= 2^31
    {
        double dr[8], er[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            dr[j] = sm.d[16 * j + (lane & 15)];
            er[j] = sm.e2[16 * j + (lane & 15)];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) dpp_ready(dr[j], er[j]);
        const int n = tid / L, s = tid % L;                      // eigenvalue n (0 = largest), piece s
        const int j = kN - 1 - n;                                // its index in ascending order
        const double inv = 1.0 / (double)(L + 1);
        double lo = 0.0, hi = 1.0 + 0x1p-10;
        for (int it = 0; it < rounds; ++it) {
            const double step = (hi - lo) * inv;
            const int cnt = sturm_count<kD - kN>(dr, er, lo + step * (double)(s + 1));
            const unsigned long long mask = __ballot(cnt > j);
            const unsigned bits = (unsigned)(mask >> (lane - s)) & ((1u << L) - 1u);
            const int piece = bits ? __builtin_ctz(bits) : L;    // first cut with more than j eigenvalues below it
            const double nlo = lo + step * (double)piece;
            hi = piece == L ? hi : lo + step * (double)(piece + 1);
            lo = nlo;
        }
        // a bracket that still starts at zero (3e-10 of the trace) is a zero eigenvalue: a matrix of low rank has up to 128,
        // and their middles would add 1e-7 to the entropy
        if (s == 0 && n < n_need) sm.lam[n] = lo > 0.0 ? 0.5 * (lo + hi) : 0.0;
    }
    __syncthreads();

    // ---- 4. entropy --------------------------------------------------------------------------
    const double mine = tid < kD ? sm.lam[tid] : 0.0;
    const double total = block_sum(tid < kD ? sm.d[tid] : 0.0, sm.red, tid);   // the trace: sum of all eigenvalues
    const double topk = block_sum(tid < k ? mine : 0.0, sm.red, tid);
    // total = 1 up to rounding (the matrix was scaled to unit trace).  When the matrix is a projection
    // of a larger one, the eigenvalues' share of the larger trace is what Eq. 5 and eig_out mean.
    const double whole = trace_total != nullptr ? total * (whole_raw / trace) : total;
    const double denom = (flags & UNCOMP_TRUNC_RENORM) ? topk : whole;
    double term = 0.0;
    if (tid < k && mine > 0.0 && denom > 0.0) {
        const double sgm = mine / denom;
        term = -sgm * log(sgm);
    }
    const double H = block_sum(term, sm.red, tid);
    if (tid == 0) entropy_out[m] = (float)H;
    if (eig_out != nullptr && tid < eig_ld)        // eig_ld values per matrix: all 128, or the leading 64 of a 64-wide input
        eig_out[(int64_t)m * eig_ld + tid] = whole > 0.0 ? (float)(mine / whole) : 0.f;
}

hipError_t launch_tridiag_entropy(int n_mat, int N, int k_trunc, unsigned flags, const EntropyPlan& p,
                                  char* ws, float* entropy_out, float* eig_out, const Env& env,
                                  const double* trace_total, int eig_ld) {
    const float* gram = reinterpret_cast<const float*>(ws + p.gram_off);
    const float* sums = reinterpret_cast<const float*>(ws + p.sum_off);
    env.begin("tridiag_entropy");
    auto kern = eig_ld == kHalf ? tridiag_entropy_kernel<true> : tridiag_entropy_kernel<false>;
    kern<<<dim3(n_mat), dim3(kTriThreads), 0, env.s>>>(gram, sums, p.n_chunks, N, k_trunc, flags, entropy_out, eig_out, eig_ld,
                                                       trace_total);
    env.end();
    return hipGetLastError();
}

}  // namespace uncomp
