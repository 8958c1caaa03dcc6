// Covariance C = X^T X - s s^T / N of a wide bf16 token matrix X [N][D] (Sec. 3.1 Eq. 1), for the wide-matrix entropy of
// matrices with many tokens for their width: the block iteration of subspace.hip then multiplies C instead of X and X^T.
// C only steers the iterated subspace (the Ritz values come from the tokens), so its errors enter them squared: products are
// exact, sums fp32 inside a chunk and fp64 across chunks, entries kept to 17 bits.
//
// cov_tile_kernel: one 256 x 256 tile on or below the diagonal over one chunk of tokens per workgroup.  Four waves hold 128 x 128
// each (sixteen 32 x 32 accumulators in the accumulation registers).  The contraction runs over tokens, the slow index of X, so
// the operands (eight tokens of one feature per lane) come out of LDS through the transposing read: lane i of sixteen fetches
// four features of token i / 4 and receives four tokens of feature i.  Token rows of 512 bytes are stored with their 32-byte
// pieces exchanged by a pattern of the token, so that the eight token rows a read touches lie in different banks.  Two tiles of
// 32 tokens in LDS, two more on their way in registers, one barrier per tile.
// The tiles of one token chunk are neighbours on one XCD, whose L2 then fetches that chunk's rows alone (whole launch, with
// neighbours on eight: 131072 tokens of 1024 features 244 -> 212 us, of 2048 622 -> 575, 41047 of 3584 593 -> 567; of 4096 the same).
// Bound by the matrix cores under the power limit: 131072 tokens of 4096 features in 2.1 ms, 1.05 PFLOP/s over the tiles on and
// below the diagonal; 16 passes over the tokens instead took 3.75 ms.  Steps on the way: products, reads and stores in the
// compiler's order 3.0 ms; staged pieces of a struct type, which it keeps in scratch memory, 7.0 ms.
#include "common.h"
#include "device_utils.h"

namespace uncomp {

namespace {

constexpr int kTile = 256, kStep = 32;                       // features of a tile side, tokens of an LDS tile
constexpr int kRowBytes = kTile * 2, kPanelBytes = kStep * kRowBytes;

typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));

// which 32-byte pieces of token t's row change places
__device__ __forceinline__ int swizzle(int t) { return (t & 3) | ((t >> 3) & 1) << 2; }

__device__ __forceinline__ s16x4_t read_transposed(const unsigned char* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)p);
}

// round-to-nearest-even bf16 of a finite float
__device__ __forceinline__ uint32_t bf16_rne(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// tile number t of the lower triangle, row by row: (I, J), I >= J
__host__ __device__ inline void tile_of(int t, int* I, int* J) {
    int i = 0;
    while ((i + 1) * (i + 2) / 2 <= t) ++i;
    *I = i;
    *J = t - i * (i + 1) / 2;
}

}  // namespace

// part[chunk][tile][256][256]; features beyond D repeat the last eight, and nobody reads what comes of them
__global__ __launch_bounds__(256, 1) void cov_tile_kernel(const bf16_bits* __restrict__ X, int64_t ldx, int N, int D, int chunk,
                                                          int n_tiles, float* __restrict__ part) {
    __shared__ __align__(16) unsigned char lds[2][2][kPanelBytes];        // [buffer][panel: rows of the tile, columns]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, wr = wv >> 1, wc = wv & 1;
    // workgroup numbers go round the eight XCDs: neighbours in (chunk, tile) order on one of them
    const int n_wg = gridDim.x, xcd = blockIdx.x & 7;
    const int wg = xcd * (n_wg >> 3) + min(xcd, n_wg & 7) + (blockIdx.x >> 3);
    const int c = wg / n_tiles, tile = wg % n_tiles;
    int I, J;
    tile_of(tile, &I, &J);
    const int t_begin = c * chunk, t_end = min(N, t_begin + chunk);
    const int n_steps = (t_end - t_begin) / kStep, left = (t_end - t_begin) % kStep;      // whole tiles, tokens behind them

    // staging: piece tid % 32 (eight features) of tokens tid / 32 + 8 i of either panel; addresses are a base that is uniform over
    // the workgroup and 32-bit offsets (the launcher checks that 32 rows of X span less than 2 GiB)
    const int piece = tid & 31, tok0 = tid >> 5;
    const char* panel0 = reinterpret_cast<const char*>(X + (int64_t)t_begin * ldx);
    const uint32_t row_step = (uint32_t)(8 * ldx * 2);
    const uint32_t off0 = (uint32_t)(tok0 * ldx * 2) + 2u * min(kTile * I + 8 * piece, D - 8);
    const uint32_t off1 = (uint32_t)(tok0 * ldx * 2) + 2u * min(kTile * J + 8 * piece, D - 8);
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    struct Pieces {
        u32x4_t v[2][4];                                                    // [panel][i]
    };
    Pieces ra, rb;                                                        // two tiles on their way
    // One panel of a whole tile.  Past the last whole tile that one is read again, without a branch: a choice between loads puts
    // the pieces into scratch memory.
    auto fetch = [&](u32x4_t (&r)[4], uint32_t off, int step) {
        const char* b = panel0 + (int64_t)min(step, n_steps - 1) * kStep * ldx * 2;
        each16<0, 4>([&](auto i) { r[i.value] = *reinterpret_cast<const u32x4_t*>(b + (off + i.value * row_step)); });
    };
    int put[4];                                                           // where this thread's pieces go in a panel
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = tok0 + 8 * i;
        put[i] = t * kRowBytes + ((((piece >> 1) ^ swizzle(t)) << 1 | (piece & 1)) << 4);
    }
    // operands: lanes of group g (of sixteen) hold features 16 (g & 1) + lane % 16 of a block of 32, tokens 8 (g >> 1) and on
    const int g = lane >> 4, i16 = lane & 15;
    const int hx = (i16 >> 2) | (g >> 1) << 2, base = (8 * (g >> 1) + (i16 >> 2)) * kRowBytes + (i16 & 3) * 8;
    int at[2][4];                                                         // [panel][block of 32 features]
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        at[0][b] = base + (((2 * (4 * wr + b) + (g & 1)) ^ hx) << 5);
        at[1][b] = base + (((2 * (4 * wc + b) + (g & 1)) ^ hx) << 5);
    }
    f32x16_t acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    struct Operands {
        s16x4_t v[2][4][2];                                               // [panel][block][tokens 0-3, 4-7 of the lane's eight]
    };
    // Sixteen products, with `beside(n)` issued before the n-th: one wave per SIMD has nothing else to fill the matrix cores'
    // time with, and its order is kept.
    auto products = [&](const Operands& o, auto&& beside) {
        each16<0>([&](auto n) {                                           // indexes are constants from the start: registers
            constexpr int a = n.value / 4, b = n.value % 4;
            beside(n);
            const s16x8_t x = __builtin_shufflevector(o.v[0][a][0], o.v[0][a][1], 0, 1, 2, 3, 4, 5, 6, 7);
            const s16x8_t y = __builtin_shufflevector(o.v[1][b][0], o.v[1][b][1], 0, 1, 2, 3, 4, 5, 6, 7);
            // accumulation registers, named in the statement: the compiler would keep them in vector ones
            asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc[a][b]) : "v"(x), "v"(y));
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // The compiler does not look into the statements: where products end, they have left the matrix cores before anything else
    // reads or moves what they wrote.
    auto settle = [&]() {
        asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15"
                     : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[0][2]), "+a"(acc[0][3]),
                     "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[1][2]), "+a"(acc[1][3]),
                     "+a"(acc[2][0]), "+a"(acc[2][1]), "+a"(acc[2][2]), "+a"(acc[2][3]),
                     "+a"(acc[3][0]), "+a"(acc[3][1]), "+a"(acc[3][2]), "+a"(acc[3][3]));
    };
    auto read = [&](Operands& o, auto BUF, auto KS, auto N_) {            // the n-th of sixteen reads
        constexpr int n = N_.value, p = n & 1, b = n >> 2, h = (n >> 1) & 1;
        o.v[p][b][h] = read_transposed(&lds[BUF.value][p][at[p][b]] + (16 * KS.value + 4 * h) * kRowBytes);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    Operands oa, ob;                                                      // second and first half of a tile
    each16<0>([&](auto n) { oa.v[n.value & 1][n.value >> 2][(n.value >> 1) & 1] = s16x4_t{0, 0, 0, 0}; });
    // tile `step` is in buf; oa holds the second half of the one before.  next: tile step + 1, on its way to the other buffer
    auto tile_step = [&](int step, auto BUF, Pieces& next) {
        constexpr int buf = decltype(BUF)::value;
        products(oa, [&](auto n) { read(ob, BUF, I0{}, n); });
        products(ob, [&](auto n) {
            read(oa, BUF, I1{}, n);
            if constexpr (n.value < 8)
                *reinterpret_cast<u32x4_t*>(&lds[buf ^ 1][n.value >> 2][put[n.value & 3]]) = next.v[n.value >> 2][n.value & 3];
            if constexpr (n.value == 8) fetch(next.v[0], off0, step + 3);
            if constexpr (n.value == 12) fetch(next.v[1], off1, step + 3);
        });
        __syncthreads();
    };
    if (n_steps > 0) {
        fetch(ra.v[0], off0, 0);
        fetch(ra.v[1], off1, 0);
        fetch(rb.v[0], off0, 1);
        fetch(rb.v[1], off1, 1);
        each16<0, 8>([&](auto n) { *reinterpret_cast<u32x4_t*>(&lds[0][n.value >> 2][put[n.value & 3]]) = ra.v[n.value >> 2][n.value & 3]; });
        fetch(ra.v[0], off0, 2);
        fetch(ra.v[1], off1, 2);
        __syncthreads();
        int step = 0;
        for (; step + 1 < n_steps; step += 2) {
            tile_step(step, I0{}, rb);
            tile_step(step + 1, I1{}, ra);
        }
        if (step < n_steps) tile_step(step, I0{}, rb);
        products(oa, [](auto) {});
        settle();
    }
    if (left > 0) {                                                       // zeros behind the last token
        const char* b = panel0 + (int64_t)n_steps * kStep * ldx * 2;
        for (int i = 0; i < 4; ++i) {
            const bool has = tok0 + 8 * i < left;
            const uint32_t row = has ? i * row_step : 0u, keep = has ? 0xffffffffu : 0u, o = has ? 0u : (uint32_t)(tok0 * ldx * 2);
            const uint4 x = *reinterpret_cast<const uint4*>(b + (off0 - o + row)), y = *reinterpret_cast<const uint4*>(b + (off1 - o + row));
            const int t = tok0 + 8 * i, at_lds = t * kRowBytes + ((((piece >> 1) ^ swizzle(t)) << 1 | (piece & 1)) << 4);
            *reinterpret_cast<uint4*>(&lds[0][0][at_lds]) = make_uint4(x.x & keep, x.y & keep, x.z & keep, x.w & keep);
            *reinterpret_cast<uint4*>(&lds[0][1][at_lds]) = make_uint4(y.x & keep, y.y & keep, y.z & keep, y.w & keep);
        }
        __syncthreads();
        each16<0>([&](auto n) {
            read(ob, I0{}, I0{}, n);
            read(oa, I0{}, I1{}, n);
        });
        products(ob, [](auto) {});
        products(oa, [](auto) {});
        settle();
    }
    float* out = part + ((int64_t)c * n_tiles + tile) * kTile * kTile;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                out[(128 * wr + 32 * a + (v >> 2) * 8 + 4 * (lane >> 5) + (v & 3)) * kTile + 128 * wc + 32 * b + (lane & 31)] = acc[a][b][v];
        }
}

// Cs[r][c], r < D: C as bf16; r >= D: what that leaves, as bf16 (|error| <= 2^-17 of the entry).  Partials added in fp64, mean term
// subtracted there (s: column sums, nullptr for none).  A workgroup takes a 64 x 64 block on or below the diagonal and mirrors it
// (whole lines of either half both ways, four entries per thread for the memory's latency).
constexpr int kFin = 64;
__global__ __launch_bounds__(1024) void cov_finish_kernel(const float* __restrict__ part, int n_chunks, int n_tiles, int D,
                                                         const double* __restrict__ s, double inv_n, bf16_bits* __restrict__ Cs) {
    __shared__ bf16_bits blk[2][kFin][kFin + 2];
    int bi, bj;
    tile_of(blockIdx.x, &bi, &bj);
    const int cl = threadIdx.x & 63, rl0 = threadIdx.x >> 6, r0 = kFin * bi, c0 = kFin * bj;
    const int I = r0 / kTile, J = c0 / kTile, tile = I * (I + 1) / 2 + J;
    const float* p = part + (int64_t)tile * kTile * kTile + ((r0 & (kTile - 1)) + rl0) * kTile + (c0 & (kTile - 1)) + cl;
    const int64_t stride = (int64_t)n_tiles * kTile * kTile;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int x = 0; x < n_chunks; ++x)
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] += (double)p[x * stride + 16 * i * kTile];
#pragma unroll
    for (int i = 0; i < 4; ++i) {                                         // D is a multiple of the block
        const int rl = rl0 + 16 * i, r = r0 + rl, c = c0 + cl;
        if (s != nullptr) a[i] -= s[r] * s[c] * inv_n;
        const float f = (float)a[i];
        const uint32_t hi = bf16_rne(f), lo = bf16_rne(f - __uint_as_float(hi << 16));
        Cs[(int64_t)r * D + c] = (bf16_bits)hi;
        Cs[(int64_t)(D + r) * D + c] = (bf16_bits)lo;
        blk[0][rl][cl] = (bf16_bits)hi;
        blk[1][rl][cl] = (bf16_bits)lo;
    }
    if (bi == bj) return;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int rl = rl0 + 16 * i, r = c0 + rl, c = r0 + cl;
        Cs[(int64_t)r * D + c] = blk[0][cl][rl];
        Cs[(int64_t)(D + r) * D + c] = blk[1][cl][rl];
    }
}

// Chunks of tokens: whole rounds of one workgroup per CU against the partials to write and to add up.
CovPlan plan_cov(int N, int D) {
    CovPlan p;
    constexpr int kCus = 256;
    const int nb = (D + kTile - 1) / kTile;
    p.n_tiles = nb * (nb + 1) / 2;
    double best = 0.0;
    p.n_chunks = 1;
    for (int n = 1; n <= 64; ++n) {
        const int chunk = ((N + n - 1) / n + kStep - 1) / kStep * kStep;
        if (n > 1 && chunk < 512) break;
        const int real = (N + chunk - 1) / chunk;
        const int64_t rounds = ((int64_t)p.n_tiles * real + kCus - 1) / kCus;
        // us: a tile of 32 tokens at 0.65 of the matrix cores' rate at 2 GHz, 12 to start and to write; 8 bytes an entry at 4 TB/s
        const double cost = (double)rounds * (chunk / 32.0 * 0.8 + 12.0) + (double)p.n_tiles * real * kTile * kTile * 8.0 / 4e6;
        if (best == 0.0 || cost < best) {
            best = cost;
            p.n_chunks = real;
            p.chunk = chunk;
            p.cost_us = cost;
        }
    }
    p.part_bytes = (size_t)p.n_chunks * p.n_tiles * kTile * kTile * sizeof(float);
    p.cov_bytes = (size_t)2 * D * D * sizeof(bf16_bits);
    return p;
}

hipError_t launch_cov(const uint16_t* X, int64_t ldx, int N, int D, const double* s, const CovPlan& p, float* part, uint16_t* Cs,
                      hipStream_t st) {
    cov_tile_kernel<<<dim3((unsigned)(p.n_tiles * p.n_chunks)), dim3(256), 0, st>>>(X, ldx, N, D, p.chunk, p.n_tiles, part);
    const int nb = D / kFin;
    cov_finish_kernel<<<dim3((unsigned)(nb * (nb + 1) / 2)), dim3(1024), 0, st>>>(part, p.n_chunks, p.n_tiles, D, s, 1.0 / (double)N, Cs);
    return hipGetLastError();
}

}  // namespace uncomp
