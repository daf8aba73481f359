// Calibration eigenvectors: all rotations at once.
//
// Near the end, and long before it, a sweep's worth of rotations can be made by one orthogonal transformation of all rows,
// built from matrix products alone (no chain of dependent rounds).  With the angles of all pairs in a skew matrix E, the rows of
// X G are nearly orthogonal for any orthogonal X = I + E + O(E^2), and the angles that are left are quadratic in the former ones.
//
//   small angles   X = exp(E), cut behind E^2 or E^4, in fp64 (see sals_calib_eigenvectors for where the cut is below rounding)
//   any angles     X = the orthogonal polar factor of I + E, which turns an invariant plane of E by the arc tangent of its
//                  angle, so that large angles are damped.  A pair's entry is ab / sqrt(d^2 + 4 ab^2), d the difference of the
//                  squared norms: half the sine of twice the angle that makes the two rows orthogonal, and the angle itself
//                  where it is small.  Rows are sorted by norm, so that the pairs with large angles lie near the diagonal; those
//                  inside and next to a 32-row block are rotated one by one first (three Jacobi steps).
//
// The polar factor is found by Newton-Schulz steps in pairs of bf16, the last one in fp32 (X <- a X - b (X X^T) X, scaled by the
// bounds of its singular values: J. Chen, E. Chow, "A stable scaling of Newton-Schulz for improving the sign function computation of
// a Hermitian matrix", 2014), and only *found* there: what is left, delta = X X^T - I (at most 1e-5: 6.7e-6 where the last step begins
// with the smallest singular values it may, and the rounding of fp32; measured 5e-7 to 4e-6; where rows go in floats, below, it is the
// product of many coarser factors, brought there by steps in fp32, see FloatDefect), is formed in fp64 and taken out to third order,
// G <- (I - delta / 2 + 3/8 delta^2) X G, with fp64 products.  The next term, 5/16 delta^3, is below 4e-16, so what a
// transformation does to G is orthogonal to the rounding of those products (G^T G changed by 2e-15 to 3e-15 of its norm, D = 256 to 1024),
// and which transformation is made decides nothing but how fast the rows converge.  (D = 1024, r = 640: eigenvalues off by 1.2e-14 of
// themselves against a 64-bit eigensolver, by 2.4e-14 with sweeps alone.)  With X (X X^T) in the place of (X X^T) X, which is the same
// for a normal X only, rounding adds up from step to step: delta 2e-5 to 4e-5, G^T G changed by 1.1e-14 at D = 256.
#pragma once
#include "common.hpp"
#include "k_calib.hpp"
#include "k_gemm.hpp"
#include "polar_plan.hpp"

namespace sals {

// ---- 64 x 64 tiles of products of [D, D] matrices --------------------------------------------------------------------
// Tile (blockIdx.y, blockIdx.x) of A B^T (NN: of A B), summed in ACC; rows of A are D apart, those of B ldb.  A step is 128 bytes of a row:
// 32 floats or 16 doubles of the contraction.  Both operands go from memory straight into LDS, three steps ahead in four stages;
// eight waves, each half of a step's contraction for a quarter of the tile.  16-byte piece p of row r lies at piece p ^ ((r >> 1) & 7): no bank conflicts.
// Bound by the matrix cores from D = 2048 on (131 TFLOP/s in fp32, 66 in fp64); at D = 1024, one tile per compute unit, 22 and 38 us
// a product, where operands straight from memory took 33 and 47 (rows a power of two apart, and four waves asking for each).
// finish(part, row, col, e, value): called by the first four waves, element e = 0 .. 15 of lane's sixteen.
constexpr int kProdThreads = 512, kProdStages = 4;
template <typename TA, typename TB, bool NN> constexpr size_t prod_lds()
{
    return (size_t)kProdStages * (8192 + (NN ? 128 / sizeof(TA) * 64 * sizeof(TB) : 8192));
}
template <typename TA, typename TB, bool NN, typename ACC, typename Finish>
__device__ __forceinline__ void calib_product(const TA* A, const TB* B, int D, int ldb, Finish finish)
{
    static_assert(NN || sizeof(TA) == sizeof(TB), "operand layout");
    constexpr int KS = 128 / (int)sizeof(TA), EPV = 16 / (int)sizeof(TA), RB = 64 * (int)sizeof(TB);
    constexpr int B_BYTES = NN ? KS * RB : 8192, STAGE = 8192 + B_BYTES, ST = kProdStages;
    constexpr int NB = B_BYTES / 8192, NL = 1 + NB;   // loads of a wave per step
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kg = lane >> 4;
    const int part = wave & 3, ks = wave >> 2;
    const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    const uint32_t lds0 = lds_offset(lds);
    auto swz128 = [](int row, int pc) { return row * 128 + ((pc ^ ((row >> 1) & 7)) << 4); };
    const int prow = wave * 8 + (lane >> 3);
    const uint32_t piece = (uint32_t)(((lane & 7) ^ ((prow >> 1) & 7)) << 4);
    const uint32_t off_a = (uint32_t)prow * (uint32_t)D * sizeof(TA) + piece;
    // NN: B as it lies, row k of a step in RB bytes; of floats, 16-byte piece p of row k lies at piece p ^ 4 (k / 4 % 4), so that the four
    // groups of lanes that read four rows apart do not meet
    constexpr int LPR = RB / 16, RPL = 8 * (64 / LPR);   // lanes a row, rows a load of all waves
    const int krow = wave * (64 / LPR) + lane / LPR;
    const uint32_t off_b = NN ? (uint32_t)krow * (uint32_t)ldb * sizeof(TB) + (uint32_t)(((lane % LPR) ^ (sizeof(TB) == 4 ? (krow >> 2 & 3) << 2 : 0)) << 4)
                              : (uint32_t)prow * (uint32_t)ldb * sizeof(TB) + piece;
    const unsigned char* a = reinterpret_cast<const unsigned char*>(A + (size_t)r0 * D);
    const unsigned char* b = reinterpret_cast<const unsigned char*>(NN ? B + c0 : B + (size_t)c0 * ldb);
    const int n = D / KS;   // (at least 8)
    auto load = [&](int s) {
        const size_t t = (size_t)min(s, n - 1);   // (past the end: a step that nothing reads any more)
        const uint32_t st = lds0 + (uint32_t)(s % ST) * STAGE + wave * 1024;
        load_lds16(a + t * 128, off_a, st);
        if (NN) {
#pragma unroll
            for (int i = 0; i < NB; ++i) load_lds16(b + (t * KS + RPL * i) * ldb * sizeof(TB), off_b, st + 8192 * (1 + i));
        } else {
            load_lds16(b + t * 128, off_b, st + 8192);
        }
    };
#pragma unroll
    for (int s = 0; s < ST - 1; ++s) load(s);
    typename mma_tile<ACC>::acc acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[u][v][e] = 0;
    const int rr = (part >> 1) * 32 + l16, cc = (part & 1) * 32 + l16;
    typedef TA VA __attribute__((ext_vector_type(EPV)));
    for (int s = 0; s < n; ++s) {
        vm_wait<(ST - 2) * NL>();   // step s has landed, everywhere; every wave is done with step s - 1
        wg_barrier();
        load(s + ST - 1);
        const unsigned char* st = lds + (s % ST) * STAGE;
        VA x[2];
        ACC y[2][EPV];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            x[u] = *reinterpret_cast<const VA*>(st + swz128(rr + 16 * u, ks * 4 + kg));
            if (NN) {
#pragma unroll
                for (int e = 0; e < EPV; ++e)
                    y[u][e] = (ACC)*reinterpret_cast<const TB*>(st + 8192 + ((ks * 4 + kg) * EPV + e) * RB +
                                                                ((cc + 16 * u) * (int)sizeof(TB) ^ (sizeof(TB) == 4 ? kg << 6 : 0)));
            } else {
                const VA t = *reinterpret_cast<const VA*>(st + 8192 + swz128(cc + 16 * u, ks * 4 + kg));
#pragma unroll
                for (int e = 0; e < EPV; ++e) y[u][e] = (ACC)t[e];
            }
        }
#pragma unroll
        for (int e = 0; e < EPV; ++e)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v) acc[u][v] = mma_step((ACC)x[u][e], y[v][e], acc[u][v]);
    }
    vm_wait<0>();
    wg_barrier();
    // the two halves of the contraction
    ACC* red = reinterpret_cast<ACC*>(lds) + part * 1024;
    if (ks) {
#pragma unroll
        for (int i = 0; i < 16; ++i) red[i * 64 + lane] = acc[i >> 3][(i >> 2) & 1][i & 3];
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int u = i >> 3, v = (i >> 2) & 1, e = i & 3;
            finish(r0 + (part >> 1) * 32 + u * 16 + mma_tile<ACC>::row(kg, e), c0 + (part & 1) * 32 + v * 16 + l16, acc[u][v][e] + red[i * 64 + lane]);
        }
    }
}

// The symmetric A A^T, each pair of elements once: below the diagonal in halves of tiles, 64 rows x 32 columns, on the diagonal whole
// tiles less their upper 16 x 16 blocks, 10 blocks instead of 8.  (D / 64)^2 workgroups, so one for every compute unit at D = 1024 as
// with whole tiles, each with half of the work.  A step is 256 bytes of a row; the eight waves are two groups of blocks x four parts of a
// step's contraction.  Piece p of row r lies at piece p ^ (r & 15): no bank conflicts.
// Bound by the matrix cores.  Against whole tiles of the full product, with what is done to the result, D = 1024: fp64 products and
// the rows' shares 42.5 -> 28.6 us, defect 39.9 -> 27.5, angles 46 -> 30, fp32 21.8 -> 15.4; a call 5.15 -> 4.78 ms (with the launch of
// the angles below), D = 2048 24.4 -> 21.6 ms.  (Products of pairs are bound by what a compute unit draws and stay whole.)
// finish(rb, cb, v, both): 16 x 16 block (rb, cb) of the tile, element e of a lane at row 16 rb + mma_tile::row(lane / 16, e), column 16 cb +
// lane % 16; both: the mirrored elements are this workgroup's too (not so for blocks on the diagonal, which come whole).
constexpr size_t kSymLds = (size_t)kProdStages * 24576;
struct SymTile { int row, col, half; __device__ __forceinline__ bool diag() const { return row == col; } };   // in tiles of 64
__device__ __forceinline__ SymTile sym_tile(int block, int D)
{
    const int nb = (unsigned)D / 64, w = xcd_item(block, nb * nb);
    if (w < nb) return SymTile{w, w, 0};
    const int t = (w - nb) >> 1;
    int r = (int)((1.f + sqrtf(1.f + 8.f * (float)t)) * 0.5f);   // t = r (r - 1) / 2 + column
    while (r * (r - 1) / 2 > t) --r;
    while (r * (r + 1) / 2 <= t) ++r;
    return SymTile{r, t - r * (r - 1) / 2, (w - nb) & 1};
}
template <typename TA, typename ACC, typename Finish>
__device__ __forceinline__ void calib_product_sym(const TA* A, int D, int pitch, const SymTile& tile, Finish finish)
{
    constexpr int KS = 256 / (int)sizeof(TA), EPV = 16 / (int)sizeof(TA), STAGE = 24576, ST = kProdStages;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];   // per stage: 64 rows | 32 rows
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kg = lane >> 4;
    const int part = wave & 1, ks = wave >> 1;
    const uint32_t lds0 = lds_offset(lds);
    const size_t row_bytes = (size_t)pitch * sizeof(TA);
    auto at = [](int row, int pc) { return row * 256 + ((pc ^ (row & 15)) << 4); };
    const int prow = wave * 4 + kg;
    const uint32_t off = (uint32_t)prow * (uint32_t)row_bytes + (uint32_t)((l16 ^ (prow & 15)) << 4);
    const unsigned char* a = reinterpret_cast<const unsigned char*>(A) + (size_t)tile.row * 64 * row_bytes;
    const unsigned char* b = reinterpret_cast<const unsigned char*>(A) + ((size_t)tile.col * 64 + tile.half * 32) * row_bytes;
    const int n = D / KS;   // (at least 4)
    auto load = [&](int s) {
        const size_t k = (size_t)min(s, n - 1) * 256;   // (past the end: a step that nothing reads any more)
        const uint32_t st = lds0 + (uint32_t)(s % ST) * STAGE + wave * 1024;
        load_lds16(a + k, off, st);
        load_lds16(a + 32 * row_bytes + k, off, st + 8192);
        load_lds16(b + k, off, st + 16384);   // (on the diagonal nothing reads it)
    };
#pragma unroll
    for (int s = 0; s < ST - 1; ++s) load(s);
    typename mma_tile<ACC>::acc acc[5];
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][e] = 0;
    typedef TA VA __attribute__((ext_vector_type(EPV)));
    auto run = [&](auto diag) {
        constexpr bool DG = decltype(diag)::value;
        for (int s = 0; s < n; ++s) {
            vm_wait<(ST - 2) * 3>();   // step s has landed, everywhere; every wave is done with step s - 1
            wg_barrier();
            load(s + ST - 1);
            const unsigned char* st = lds + (s % ST) * STAGE;
            auto rows = [&](int block) { return *reinterpret_cast<const VA*>(st + at(block * 16 + l16, ks * 4 + kg)); };
            const VA x0 = rows(2 * part), x1 = rows(2 * part + 1);
            if (DG) {   // blocks 2 part .. against themselves, block 2 + part against the first two
                const VA x2 = rows(2 + part), y0 = rows(0), y1 = rows(1);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    acc[0] = mma_step((ACC)x0[e], (ACC)x0[e], acc[0]);
                    acc[1] = mma_step((ACC)x1[e], (ACC)x0[e], acc[1]);
                    acc[2] = mma_step((ACC)x1[e], (ACC)x1[e], acc[2]);
                    acc[3] = mma_step((ACC)x2[e], (ACC)y0[e], acc[3]);
                    acc[4] = mma_step((ACC)x2[e], (ACC)y1[e], acc[4]);
                }
            } else {
                const VA y0 = rows(4), y1 = rows(5);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    acc[0] = mma_step((ACC)x0[e], (ACC)y0[e], acc[0]);
                    acc[1] = mma_step((ACC)x1[e], (ACC)y0[e], acc[1]);
                    acc[2] = mma_step((ACC)x0[e], (ACC)y1[e], acc[2]);
                    acc[3] = mma_step((ACC)x1[e], (ACC)y1[e], acc[3]);
                }
            }
        }
    };
    const bool dg = tile.diag();   // uniform
    if (dg) run(std::true_type{}); else run(std::false_type{});
    vm_wait<0>();
    wg_barrier();
    // the four parts of the contraction: part b % 4 finishes block b
    ACC* red = reinterpret_cast<ACC*>(lds) + part * (5 * 4 * 256);
#pragma unroll
    for (int i = 0; i < 5; ++i)
        if ((i & 3) != ks) {
#pragma unroll
            for (int e = 0; e < 4; ++e) red[((i * 4 + ks) * 4 + e) * 64 + lane] = acc[i][e];
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        if ((i & 3) == ks && (i < 4 || dg)) {   // uniform
            typename mma_tile<ACC>::acc v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ACC sum = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) sum += k == (i & 3) ? acc[i][e] : red[((i * 4 + k) * 4 + e) * 64 + lane];
                v[e] = sum;
            }
            if (!dg) finish(2 * part + (i & 1), i >> 1, v, true);
            else if (i < 3) finish(2 * part + (i + 1) / 2, 2 * part + i / 2, v, i == 1);
            else finish(2 + part, i - 3, v, true);
        }
    }
}

// Behind the loop of a product of 32 x 32 parts by two halves of the waves: the first half adds up both, finish(u, v, sum).
template <typename Finish>
__device__ __forceinline__ void sum_halves(const f32x4 (&acc)[2][2], int ks, int part, unsigned char* lds, Finish finish)
{
    const int lane = threadIdx.x & 63;
    vm_wait<0>();
    wg_barrier();
    float* red = reinterpret_cast<float*>(lds) + part * 1024;
    if (ks) {
#pragma unroll
        for (int i = 0; i < 16; ++i) red[i * 64 + lane] = acc[i >> 3][(i >> 2) & 1][i & 3];
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int u = i >> 1, v = i & 1;
            f32x4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = acc[u][v][e] + red[(i * 4 + e) * 64 + lane];
            finish(u, v, x);
        }
    }
}

// Matrices of floats as pairs of bf16, x = hi + lo to 2^-17: one 32-bit word an element, hi in the upper half.
__device__ __forceinline__ uint32_t pack_pair(float x)
{
    const bf16_t hi = f32_to_bf16(x);
    return (uint32_t)hi << 16 | f32_to_bf16(x - bf16_to_f32(hi));
}
__device__ __forceinline__ float pair_value(uint32_t w) { return bf16hi(w) + bf16lo(w); }

// The same for A B^T (NN: A B) of such matrices: hi hi + hi lo + lo hi on the bf16 matrix cores, summed in fp32.  A step is 64 elements of a
// row, 32 for either half of the waves.  Bound by what a compute unit draws, 13 us a product at D = 1024, where fp32 instructions take 22.
// finish(i, j, v): rows i .. i + 3 of column j, by the first four waves.
constexpr size_t kPairLds = (size_t)kProdStages * 32768;
template <bool NN, typename Finish>
__device__ __forceinline__ void calib_product_pairs(const uint32_t* A, const uint32_t* B, int D, Finish finish)
{
    constexpr int STAGE = 32768, ST = kProdStages;   // [A: two 32-element pieces of 64 rows | B]
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kg = lane >> 4;
    const int part = wave & 3, ks = wave >> 2;
    const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    const uint32_t lds0 = lds_offset(lds);
    auto swz128 = [](int row, int pc) { return row * 128 + ((pc ^ ((row >> 1) & 7)) << 4); };
    const int prow = wave * 8 + (lane >> 3);
    const uint32_t off = (uint32_t)prow * (uint32_t)D * 4 + (uint32_t)(((lane & 7) ^ ((prow >> 1) & 7)) << 4);
    const unsigned char* a = reinterpret_cast<const unsigned char*>(A + (size_t)r0 * D);
    // NN: B as it lies, row k of a step in 256 bytes, 16-byte piece p of row k at piece p ^ 4 (k / 8 % 4)
    const int krow = wave * 4 + kg;
    const uint32_t off_b = NN ? (uint32_t)krow * (uint32_t)D * 4 + (uint32_t)((l16 ^ ((krow >> 3 & 3) << 2)) << 4) : off;
    const unsigned char* b = reinterpret_cast<const unsigned char*>(NN ? B + c0 : B + (size_t)c0 * D);
    const int n = D / 64;   // (at least 4)
    auto load = [&](int s) {
        const size_t at = (size_t)min(s, n - 1) * 256;   // (past the end: a step that nothing reads any more)
        const uint32_t st = lds0 + (uint32_t)(s % ST) * STAGE + wave * 1024;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            load_lds16(a + at + 128 * i, off, st + 8192 * i);
            load_lds16(NN ? b + (at / 4 + 32 * i) * D * 4 : b + at + 128 * i, off_b, st + 16384 + 8192 * i);
        }
    };
#pragma unroll
    for (int s = 0; s < ST - 1; ++s) load(s);
    f32x4 acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int rr = (part >> 1) * 32 + l16, cc = (part & 1) * 32 + l16;
    struct Pair { u32x4 hi, lo; };
    auto split = [](const u32x4& x, const u32x4& y) {
        auto upper = [](uint32_t w0, uint32_t w1) { return __builtin_amdgcn_perm(w1, w0, 0x07060302u); };
        auto lower = [](uint32_t w0, uint32_t w1) { return __builtin_amdgcn_perm(w1, w0, 0x05040100u); };
        return Pair{u32x4{upper(x.x, x.y), upper(x.z, x.w), upper(y.x, y.y), upper(y.z, y.w)},
                    u32x4{lower(x.x, x.y), lower(x.z, x.w), lower(y.x, y.y), lower(y.z, y.w)}};
    };
    auto fragment = [&](const unsigned char* st, int row) {   // eight elements of a row, from 8 kg on
        return split(*reinterpret_cast<const u32x4*>(st + swz128(row, 2 * kg)), *reinterpret_cast<const u32x4*>(st + swz128(row, 2 * kg + 1)));
    };
    auto column = [&](const unsigned char* st, int col) {   // eight elements of a column, from row 8 kg on
        const unsigned char* at = st + kg * 2048 + ((col * 4) ^ (kg << 6));
        uint32_t w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = *reinterpret_cast<const uint32_t*>(at + e * 256);
        return split(u32x4{w[0], w[1], w[2], w[3]}, u32x4{w[4], w[5], w[6], w[7]});
    };
    auto mma = [](const u32x4& x, const u32x4& y, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
    };
    for (int s = 0; s < n; ++s) {
        vm_wait<(ST - 2) * 4>();   // step s has landed, everywhere; every wave is done with step s - 1
        wg_barrier();
        load(s + ST - 1);
        const unsigned char* st = lds + (s % ST) * STAGE + ks * 8192;
        Pair x[2], y[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) { x[u] = fragment(st, rr + 16 * u); y[u] = NN ? column(st + 16384, cc + 16 * u) : fragment(st + 16384, cc + 16 * u); }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                acc[u][v] = mma(x[u].lo, y[v].hi, acc[u][v]);
                acc[u][v] = mma(x[u].hi, y[v].lo, acc[u][v]);
                acc[u][v] = mma(x[u].hi, y[v].hi, acc[u][v]);
            }
    }
    sum_halves(acc, ks, part, lds, [&](int u, int v, const f32x4& x) {
        finish(r0 + (part >> 1) * 32 + u * 16 + 4 * kg, c0 + (part & 1) * 32 + v * 16 + l16, x);
    });
}

// The same for A B^T of plain bf16 matrices, summed in fp32.  A step is 128 elements of a row, 64 for either half of the waves.
constexpr size_t kPlainLds = (size_t)kProdStages * 32768;
// meanwhile(): while the first steps are on their way.
template <typename Meanwhile, typename Finish>
__device__ __forceinline__ void calib_product_plain(const bf16_t* A, const bf16_t* B, int D, Meanwhile meanwhile, Finish finish)
{
    constexpr int STAGE = 32768, ST = kProdStages;   // [A: two 64-element pieces of 64 rows | B]
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, kg = lane >> 4;
    const int part = wave & 3, ks = wave >> 2;
    const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    const uint32_t lds0 = lds_offset(lds);
    auto swz128 = [](int row, int pc) { return row * 128 + ((pc ^ ((row >> 1) & 7)) << 4); };
    const int prow = wave * 8 + (lane >> 3);
    const uint32_t off = (uint32_t)prow * (uint32_t)D * 2 + (uint32_t)(((lane & 7) ^ ((prow >> 1) & 7)) << 4);
    const unsigned char* a = reinterpret_cast<const unsigned char*>(A + (size_t)r0 * D);
    const unsigned char* b = reinterpret_cast<const unsigned char*>(B + (size_t)c0 * D);
    const int n = D / 128;   // (at least 2)
    auto load = [&](int s) {
        const size_t at = (size_t)min(s, n - 1) * 256;   // (past the end: a step that nothing reads any more)
        const uint32_t st = lds0 + (uint32_t)(s % ST) * STAGE + wave * 1024;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            load_lds16(a + at + 128 * i, off, st + 8192 * i);
            load_lds16(b + at + 128 * i, off, st + 16384 + 8192 * i);
        }
    };
#pragma unroll
    for (int s = 0; s < ST - 1; ++s) load(s);
    meanwhile();
    f32x4 acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int rr = (part >> 1) * 32 + l16, cc = (part & 1) * 32 + l16;
    for (int s = 0; s < n; ++s) {
        vm_wait<(ST - 2) * 4>();   // step s has landed, everywhere; every wave is done with step s - 1
        wg_barrier();
        load(s + ST - 1);
        const unsigned char* st = lds + (s % ST) * STAGE + ks * 8192;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            bf16x8 x[2], y[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                x[u] = *reinterpret_cast<const bf16x8*>(st + swz128(rr + 16 * u, 4 * k + kg));
                y[u] = *reinterpret_cast<const bf16x8*>(st + 16384 + swz128(cc + 16 * u, 4 * k + kg));
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v) acc[u][v] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u], y[v], acc[u][v], 0, 0, 0);
        }
    }
    sum_halves(acc, ks, part, lds, [&](int u, int v, const f32x4& x) {
        finish(r0 + (part >> 1) * 32 + u * 16 + 4 * kg, c0 + (part & 1) * 32 + v * 16 + l16, x);
    });
}

// Y = G + f A B (ADD), or f A B.  Y may be G, not B.
template <typename TA, bool ADD>
__global__ __launch_bounds__(kProdThreads) void calib_apply_kernel(const TA* A, const double* B, const double* G, double f, double* Y, int D)
{
    calib_product<TA, double, true, double>(A, B, D, D, [&](int r, int c, double v) {
        const size_t at = (size_t)r * D + c;
        Y[at] = ADD ? fma(f, v, G[at]) : f * v;
    });
}

// exp(E) - I for a small skew E, so that one product with G takes all its terms: X = E - P / 2 with P = E E^T = -E^2 summed in fp64 and,
// LONG, the terms of third and fourth order, (P / 24 - E / 6) P, by a product in fp32 behind it: with |E|_F at most 5.7e-3 (the limit is
// one of the pairs) they are 3e-8, and fp32 leaves 2e-15 of them, in the Frobenius norm.  At D = 1024 28 + 22 + 44 us for four terms,
// and 28 + 44 for two, where a product with G took 44 for each term.
template <bool LONG>
__global__ __launch_bounds__(kProdThreads) void calib_series_kernel(const double* __restrict__ E, int D, double* __restrict__ X, float* __restrict__ P,
                                                                    float* __restrict__ L)
{
    const SymTile tile = sym_tile(blockIdx.x, D);
    const int lane = threadIdx.x & 63;
    calib_product_sym<double, double>(E, D, D, tile, [&](int rb, int cb, const f64x4& v, bool both) {
        const int j = tile.col * 64 + tile.half * 32 + cb * 16 + (lane & 15);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = tile.row * 64 + rb * 16 + mma_tile<double>::row(lane >> 4, e);
            const size_t at = (size_t)i * D + j, mirrored = (size_t)j * D + i;
            const double p = v[e], x = E[at];
            X[at] = fma(-0.5, p, x);
            if (both) X[mirrored] = fma(-0.5, p, -x);
            if (LONG) {
                P[at] = (float)p;
                L[at] = (float)(p * (1.0 / 24.0) - x * (1.0 / 6.0));
                if (both) { P[mirrored] = (float)p; L[mirrored] = (float)(p * (1.0 / 24.0) + x * (1.0 / 6.0)); }
            }
        }
    });
}
// X += L P, P symmetric
__global__ __launch_bounds__(kProdThreads) void calib_series_rest_kernel(const float* __restrict__ L, const float* __restrict__ P, int D,
                                                                         double* __restrict__ X)
{
    calib_product<float, float, false, float>(L, P, D, D, [&](int i, int j, float v) { X[(size_t)i * D + j] += (double)v; });
}

// ---- Angles -----------------------------------------------------------------------------------------------------------
// Both forms start from G G^T; `norm`: the rows' norms.
//
// The last angles: E = -t (fp64), t = ab / d, over the pairs that are not orthogonal to working precision and of which one row has a
// squared norm >= lead; where both have, their cosine counts as well as t (beside a far larger row, t is small long before the smaller
// row's direction is right).  found: per tile {largest |t| (at most 1/2), sum of t^2}.
__global__ __launch_bounds__(kProdThreads) void calib_angles_kernel(const double* __restrict__ G, int D, const double* __restrict__ norm,
                                                                    const double* __restrict__ lead_at, double* __restrict__ E,
                                                                    f64x2* __restrict__ found)
{
    const double lead = *lead_at;
    __shared__ f64x2 s_found[8];
    double most = 0.0, sum = 0.0;
    const SymTile tile = sym_tile(blockIdx.x, D);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    calib_product_sym<double, double>(G, D, D, tile, [&](int rb, int cb, const f64x4& v, bool both) {
        const int j = tile.col * 64 + tile.half * 32 + cb * 16 + (lane & 15);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = tile.row * 64 + rb * 16 + mma_tile<double>::row(lane >> 4, e);
            const double ab = v[e], ni = norm[i], nj = norm[j], aa = ni * ni, bb = nj * nj, d = bb - aa;
            const bool counts = i != j && fmax(aa, bb) >= lead && jac_open(aa, bb, ab);
            const double th = counts ? ab / d : 0.0;
            if (counts && (both || i < j)) {
                most = fmax(most, fabs(ab) / fmax(fabs(d), 2.0 * fabs(ab)));
                if (fmin(aa, bb) >= lead) most = fmax(most, fabs(ab) / (ni * nj));
                sum += th * th;
            }
            E[(size_t)i * D + j] = -th;
            if (both) E[(size_t)j * D + i] = th;
        }
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { most = fmax(most, __shfl_xor(most, o, kWave)); sum += __shfl_xor(sum, o, kWave); }
    if (lane == 0) s_found[wave] = f64x2{most, sum};
    __syncthreads();
    if (threadIdx.x == 0) {
        f64x2 t = s_found[0];
#pragma unroll
        for (int w = 1; w < 8; ++w) t = f64x2{fmax(t.x, s_found[w].x), t.y + s_found[w].y};
        found[blockIdx.x] = t;
    }
}

// Any angles, of rows sorted by norm, for the pairs that are not orthogonal to 1e-12 and of which one row has a squared norm of at
// least a thousandth of the r-th largest one (smaller ones hardly move a leading row).  A pair of nearly equal norms is turned far by
// a small ab, and in vain while the norms still move: row i's squared norm is off by about the sum of ab^2 / h over its pairs, h =
// sqrt(d^2 + 4 ab^2).  So the entry is ab / sqrt(h^2 + (off_i + off_j)^2), which is as good once the rows are nearly orthogonal and
// saves a transformation of ten (weights 0, 0.1, 0.3, 1 and 3 of its square: 5.93, 5.17, 5.15, 5.21 and 5.54 ms at D = 1024, r = 640;
// 6.0, 5.0, 5.3, 6.8 and 7.4 with eigenvalues within 1e-3 of each other).  First the products (fp32) and the workgroups'
// shares of `off`, [share][row]: a row of tile I has D / 64 + I of them, two from a tile before its own, one from its own and from later ones ...
//
// Products and norms are scaled by the power of two that takes the largest norm below one: any covariance that fp64 holds has products
// that floats hold (angles do not depend on the scale).
constexpr double kAllDamp = 0.1, kAllOpen = 1e-24, kAllTail = 1e-3;
constexpr double kFloatOpen = 1e-13;   // of rows in floats, whose products are off by 1e-7 of the norms
// ... and their weight, larger as they go the longer way, from larger angles (0.1, 0.15, 0.2, 0.25, 0.3, 0.4 and 0.5, calls with 48 matrices
// of D = 256 to 1024 and four spectra: 1, 0.998, 0.982, 0.979, 0.979, 0.975 and 0.967 of the time; the 24 of a spectrum 1 / c alone 1, 0.999,
// 0.998, 0.999, 1.01, 1.03 and 1.02)
constexpr double kFloatDamp = 0.25;
__device__ __forceinline__ double all_scale(const double* __restrict__ norm) { return ldexp(1.0, -__builtin_amdgcn_frexp_exp(norm[0])); }
struct AllPair { bool counts; double d, h2; };
__device__ __forceinline__ AllPair all_pair(double ni, double nj, double ab, double least, double open)
{
    const double aa = ni * ni, bb = nj * nj, d = bb - aa;
    return AllPair{fmax(aa, bb) >= least && ab * ab > open * (aa * bb), d, fma(4.0 * ab, ab, d * d)};
}
template <typename T>
__global__ __launch_bounds__(kProdThreads) void calib_gram_kernel(const T* __restrict__ G, int D, int pitch, const double* __restrict__ norm, int r,
                                                                  float* __restrict__ W, float* __restrict__ off)
{
    __shared__ float s_off[2][4][64];   // of the tile's rows by 16-column block, of its columns by 16-row block (the diagonal: all the former)
    const double unit = all_scale(norm), n_r = norm[r - 1] * unit, lead = 0.999 * n_r * n_r, least = kAllTail * lead;
    const SymTile tile = sym_tile(blockIdx.x, D);
    const int lane = threadIdx.x & 63, l16 = lane & 15, kg = lane >> 4;
    const int i0 = tile.row * 64, j0 = tile.col * 64 + tile.half * 32;
    calib_product_sym<T, T>(G, D, pitch, tile, [&](int rb, int cb, const typename mma_tile<T>::acc& v, bool both) {
        const int j = j0 + cb * 16 + l16;
        float col = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int at = rb * 16 + mma_tile<T>::row(kg, e), i = i0 + at;
            const double ab = v[e] * unit * unit;
            W[(size_t)i * D + j] = (float)ab;
            if (both) W[(size_t)j * D + i] = (float)ab;
            const AllPair p = all_pair(norm[i] * unit, norm[j] * unit, ab, least, sizeof(T) == 8 ? kAllOpen : kFloatOpen);
            const float share = i != j && p.counts ? (float)(ab * ab * rsqrt_f64(p.h2)) : 0.f;
            col += share;
            const float t = row16_sum(share);
            if (l16 == 0) s_off[0][cb][at] = t;
        }
        if (both) {
            col += __shfl_xor(col, 16, kWave);
            col += __shfl_xor(col, 32, kWave);
            if (kg == 0) s_off[tile.diag() ? 0 : 1][rb][cb * 16 + l16] = col;
        }
    });
    __syncthreads();
    const int t = threadIdx.x;
    if (tile.diag()) {
        if (t < 64) off[(size_t)(2 * tile.row) * D + i0 + t] = (s_off[0][0][t] + s_off[0][1][t]) + (s_off[0][2][t] + s_off[0][3][t]);
    } else if (t < 64) {
        off[(size_t)(2 * tile.col + tile.half) * D + i0 + t] = s_off[0][0][t] + s_off[0][1][t];
    } else if (t < 96) {
        const int c = t - 64;
        off[(size_t)(tile.col + tile.row) * D + j0 + c] = (s_off[1][0][c] + s_off[1][1][c]) + (s_off[1][2][c] + s_off[1][3][c]);
    }
}
// ... then E (pairs of bf16, or plain bf16), kAngleRows rows x 256 columns a workgroup, and per workgroup the sum of squares of ab / h over
// the pairs with a leading row; COUNT: also how many these are, behind all sums.  (8.9 us at D = 1024; 26.5 with 256 columns after the
// other in a workgroup.)
constexpr int kAngleRows = 8;
template <typename TE, bool COUNT = false>
__global__ __launch_bounds__(256) void calib_all_angles_kernel(const float* __restrict__ W, int D, const double* __restrict__ norm, int r,
                                                               const float* __restrict__ off, double open, double damp, TE* __restrict__ E,
                                                               double* __restrict__ found)
{
    static_assert(kAngleRows == 8 && kCalThreads == 256, "32 lanes a row; D is a multiple of the columns");
    __shared__ double s_sum[4];
    __shared__ int s_open[4];
    __shared__ float s_off[kAngleRows];
    int n_open = 0;   // of this wave
    const double unit = all_scale(norm), n_r = norm[r - 1] * unit, lead = 0.999 * n_r * n_r, least = kAllTail * lead;
    const int tid = threadIdx.x, i0 = blockIdx.x * kAngleRows, j = blockIdx.y * 256 + tid, nb = D / 64;
    float w[kAngleRows];
#pragma unroll
    for (int u = 0; u < kAngleRows; ++u) w[u] = W[(size_t)(i0 + u) * D + j];
    float off_j = 0.f, mine = 0.f;
    for (int t = tid & 31; t < nb + i0 / 64; t += 32) mine += off[(size_t)t * D + i0 + (tid >> 5)];
    const int n_j = nb + wave_uniform(j / 64);
#pragma unroll 8
    for (int t = 0; t < n_j; ++t) off_j += off[(size_t)t * D + j];
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) mine += __shfl_xor(mine, o, kWave);
    if ((tid & 31) == 0) s_off[tid >> 5] = mine;
    __syncthreads();
    const double nj = norm[j] * unit;
    double sum = 0.0;
#pragma unroll
    for (int u = 0; u < kAngleRows; ++u) {
        const int i = i0 + u;
        const double ab = w[u], ni = norm[i] * unit, o = (double)s_off[u] + off_j;
        const AllPair p = all_pair(ni, nj, ab, least, open);
        const bool counts = p.counts && i != j;
        const double s = counts ? ab * rsqrt_f64(fma(damp * o, o, p.h2)) : 0.0;
        const float e = (float)(p.d < 0.0 || (p.d == 0.0 && i > j) ? s : -s);
        E[(size_t)i * D + j] = sizeof(TE) == 2 ? (TE)f32_to_bf16(e) : (TE)pack_pair(e);
        const bool leads = counts && i < j && fmax(ni, nj) * fmax(ni, nj) >= lead;
        if (leads) sum += ab * ab / p.h2;
        if (COUNT) n_open += __popcll(__ballot(leads));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, kWave);
    if ((tid & 63) == 0) { s_sum[tid >> 6] = sum; if (COUNT) s_open[tid >> 6] = n_open; }
    __syncthreads();
    if (tid != 0) return;
    double* const mine_found = found + blockIdx.y * gridDim.x + blockIdx.x;
    *mine_found = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
    if (COUNT) mine_found[gridDim.x * gridDim.y] = (s_open[0] + s_open[1]) + (s_open[2] + s_open[3]);
}

// ---- Polar factor -----------------------------------------------------------------------------------------------------
// The first four waves' sums of squares, added up for the tile
__device__ __forceinline__ void tile_square(double sum, double* s_sum, double* square)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, kWave);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0 && wave < 4) s_sum[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) square[blockIdx.y * gridDim.x + blockIdx.x] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}
// O = d I + s S + t T + f A B^T (S, T: N > 0, N > 1; N == 1: A B) from pairs of bf16, left as such pairs or (LAST) in fp32.  SQUARE: also
// the sum of squares of every tile of O.
template <int N, bool SQUARE, bool LAST>
__global__ __launch_bounds__(kProdThreads) void calib_polar_kernel(const uint32_t* A, const uint32_t* B, int D, float f, float d, float s,
                                                                   const uint32_t* S, float t, const uint32_t* T, uint32_t* O, double* square)
{
    __shared__ double s_sum[4];
    double sum = 0.0;
    calib_product_pairs<N == 1>(A, B, D, [&](int i0, int j, const f32x4& v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + e;
            const size_t at = (size_t)i * D + j;
            float o = f * v[e];
            if (N > 0) o = fmaf(s, pair_value(S[at]), o);
            if (N > 1) { o = fmaf(t, pair_value(T[at]), o); o += i == j ? d : 0.f; }
            O[at] = LAST ? __float_as_uint(o) : pack_pair(o);
            if (SQUARE) sum += (double)o * (double)o;
        }
    });
    if (!SQUARE) return;
    tile_square(sum, s_sum, square);
}
constexpr int kPolarFound = 4;   // a thread's tiles, of at most (kFloatMaxD / 64)^2
static_assert((kFloatMaxD / 64) * (kFloatMaxD / 64) <= kPolarFound * kProdThreads, "every tile's sum is read");
// The steps of a polar factor that only steers, in plain bf16: O = d I + f A B^T (N == 0, symmetric), f A B^T + s S (N == 1), or
// d I + s E + t A + f A E^T (N == 2, B = S = E, which is skew).  What is symmetric or skew is read and written by rows for columns, four
// elements a lane; of what is neither, S and OT are the transposes.  Left as plain bf16 or in fp32.
//
// Bound by what a compute unit draws, of which a pair's half is half: 7 us a product at D = 1024 where pairs take 12 to 15, a call when
// this was made 3300 -> 3110 us (D = 2048 18.5 -> 15.4 ms) with all steps but the last one so, and 2824 -> 2667 (13.4 -> 12.4) with that
// one too.  Rounding X to 2^-9 turns the
// rows by 2^-9 of the angles that are taken out, while these are still large, and moves its singular values by 2e-3 (noise of 2^-9 / sqrt(3 D) an
// element), which the last step, the one that leaves fp32, takes to the square of that.  The steps multiply with X X^T - I, whose rounding is a
// small part of what is still to be made good; the diagonal of X X^T alone would be off by 4e-3.  (FloatDefect has what is left.)  Not once V
// is polished: the last angles are told in pairs.
enum PolarOut { kOutPlain, kOutFloat };
//
// FIND: the scalars of the first step (N == 2) from the sums of squares of A's tiles, as polar_plan has them, so that the step need not wait for the
// host to learn them: that costs 12 us of an idle device each time.
template <int N, bool SQUARE, PolarOut OUT, bool FIND>
__global__ __launch_bounds__(kProdThreads) void calib_polar_plain_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, int D, float f,
                                                                         float d, float s, const bf16_t* __restrict__ S, float t,
                                                                         void* __restrict__ O, bf16_t* __restrict__ OT, double* __restrict__ square)
{
    struct alignas(8) Four { bf16_t x[4]; };
    static_assert(!FIND || (N == 2 && !SQUARE), "the first step");
    __shared__ double s_sum[kProdThreads / kWave];
    double sum = 0.0, found[kPolarFound];
    const int n_tiles = gridDim.x * gridDim.y;
    if (FIND) {   // (requested ahead of the operands)
#pragma unroll
        for (int u = 0; u < kPolarFound; ++u) found[u] = square[min((int)threadIdx.x + u * kProdThreads, n_tiles - 1)];
    }
    auto scalars = [&]() {
        if (!FIND) return;
        double a2 = 0.0;
#pragma unroll
        for (int u = 0; u < kPolarFound; ++u) a2 += (int)threadIdx.x + u * kProdThreads < n_tiles ? found[u] : 0.0;
        a2 = wave_sum_f64(a2);
        if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = a2;
        __syncthreads();
        a2 = 0.0;
#pragma unroll
        for (int w = 0; w < kProdThreads / kWave; ++w) a2 += s_sum[w];
        const double bound = sqrt(sqrt(a2)), tau = bound > kAllCap ? kAllCap / bound : 1.0, tb = tau * bound, top = sqrt(1.0 + tb * tb);
        const double low = 1.0 / top, a = low < kFloatPolar ? sqrt(3.0 / (1.0 + low + low * low)) : 1.0;
        const double w = 0.5 * a * a * a / (top * top * top), c1 = 1.5 * a / top - w;
        f = (float)(w * tau * tau * tau); d = (float)c1; s = (float)(c1 * tau); t = (float)(-w * tau * tau);
    };
    calib_product_plain(A, B, D, scalars, [&](int i0, int j, const f32x4& v) {
        const size_t tr = (size_t)j * D + i0;
        Four add{}, sym{}, out;
        if (N > 0) add = *reinterpret_cast<const Four*>(S + tr);
        if (N > 1) sym = *reinterpret_cast<const Four*>(A + tr);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + e;
            const size_t at = (size_t)i * D + j;
            float o = f * v[e];
            if (N == 0) o += i == j ? d : 0.f;
            if (N == 1) o = fmaf(s, bf16_to_f32(add.x[e]), o);
            if (N == 2) { o = fmaf(-s, bf16_to_f32(add.x[e]), o); o = fmaf(t, bf16_to_f32(sym.x[e]), o); o += i == j ? d : 0.f; }
            if (SQUARE) sum += (double)o * (double)o;
            out.x[e] = f32_to_bf16(o);
            if (OUT == kOutFloat) static_cast<float*>(O)[at] = o;
            else if (N > 0) static_cast<bf16_t*>(O)[at] = out.x[e];
        }
        if (OUT == kOutPlain) *reinterpret_cast<Four*>((N > 0 ? OT : static_cast<bf16_t*>(O)) + tr) = out;
    });
    if (!SQUARE) return;
    tile_square(sum, s_sum, square);
}
// The last step in fp32: O = X X^T ...
__global__ __launch_bounds__(kProdThreads) void calib_polar_square_kernel(const float* X, int D, int pitch, float* O)
{
    const SymTile tile = sym_tile(blockIdx.x, D);
    const int lane = threadIdx.x & 63;
    calib_product_sym<float, float>(X, D, pitch, tile, [&](int rb, int cb, const f32x4& v, bool both) {
        const int j = tile.col * 64 + tile.half * 32 + cb * 16 + (lane & 15);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = tile.row * 64 + rb * 16 + mma_tile<float>::row(lane >> 4, e);
            O[(size_t)i * D + j] = v[e];
            if (both) O[(size_t)j * D + i] = v[e];
        }
    });
}
// ... and O = f A B + s B
__global__ __launch_bounds__(kProdThreads) void calib_polar_last_kernel(const float* A, const float* B, int D, float f, float s, float* O)
{
    calib_product<float, float, true, float>(A, B, D, D, [&](int i, int j, float v) {
        const size_t at = (size_t)i * D + j;
        O[at] = fmaf(s, B[at], f * v);
    });
}
// delta = X X^T - I, summed in fp64, and its rounding to pairs of bf16
__global__ __launch_bounds__(kProdThreads) void calib_defect_kernel(const float* X, int D, double* delta, uint32_t* rounded)
{
    const SymTile tile = sym_tile(blockIdx.x, D);
    const int lane = threadIdx.x & 63;
    calib_product_sym<float, double>(X, D, D, tile, [&](int rb, int cb, const f64x4& v, bool both) {
        const int j = tile.col * 64 + tile.half * 32 + cb * 16 + (lane & 15);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = tile.row * 64 + rb * 16 + mma_tile<double>::row(lane >> 4, e);
            const double o = i == j ? v[e] - 1.0 : v[e];
            const uint32_t pair = pack_pair((float)o);
            delta[(size_t)i * D + j] = o;
            rounded[(size_t)i * D + j] = pair;
            if (both) { delta[(size_t)j * D + i] = o; rounded[(size_t)j * D + i] = pair; }
        }
    });
}
// delta <- -delta / 2 + 3/8 delta^2 (the square, 1e-12, from the rounded one)
__global__ __launch_bounds__(kProdThreads) void calib_correction_kernel(const uint32_t* rounded, int D, double* delta)
{
    calib_product_pairs<false>(rounded, rounded, D, [&](int i0, int j, const f32x4& v) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const size_t at = (size_t)(i0 + e) * D + j;
            delta[at] = fma(0.375, (double)v[e], -0.5 * delta[at]);
        }
    });
}

// ---- Rows in floats -----------------------------------------------------------------------------------------------------
// From the factor to nearly orthogonal rows it is as far in floats as in doubles, and most of what is computed on the way only steers.
// So the rows are taken there in floats, [G | V], D rows of 2 D floats: G = V times the factor (scaled so that its largest norm is about
// one) and V the orthogonal matrix that all transformations so far amount to.  A transformation is that of above: steps inside and next to
// blocks (calib_jacobi_*<float>), a polar factor, and one product, of [G | V].  Its polar factor is sloppier (plain bf16 up to where V is
// polished, pairs of bf16 behind that; see kFloatPolar): V is made orthogonal behind one of the last transformations and at the end, by one
// Newton-Schulz step each in fp32 (or more, see FloatDefect), and at last to rounding, in fp64, as it is applied to the factor's doubles:
// what it cost in bits is some angles of the size of fp32 rounding over the relative distance of two eigenvalues, which the fp64 steps that
// follow take out.  Fewer fp64 products round the result: eigenvalues off by 1e-15 of the largest one where they were by 3e-15, D = 1024,
// r = 640.
// At D = 1024 a transformation takes 0.18 ms (fp64: 0.38), of which the product takes 41 us (105 of the 131 TFLOP/s of the fp32 matrix cores), the
// polar factor six to eight products of 7 to 9, the steps in blocks 33 + 16 and 5 for each Gram matrix, the Gram matrix of all rows and the
// angles 26, norms and order 11; and no sweep (0.85 ms) comes before them.
__global__ __launch_bounds__(kCalThreads) void calib_float_rows_kernel(const double* __restrict__ G, int D, double scale, float* __restrict__ GV)
{
    const int i = blockIdx.x;
    for (int d = threadIdx.x; d < D; d += kCalThreads) {
        GV[(size_t)i * 2 * D + d] = (float)(G[(size_t)i * D + d] * scale);
        GV[(size_t)i * 2 * D + D + d] = d == i ? 1.f : 0.f;
    }
}
// norms of the rows of G, one wave a row
__global__ __launch_bounds__(256) void calib_float_norm_kernel(const float* __restrict__ GV, int D, double* __restrict__ norm)
{
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    double sum = 0.0;
    for (int d = lane_id() * 4; d < D; d += 256) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(GV + (size_t)i * 2 * D + d);
#pragma unroll
        for (int e = 0; e < 4; ++e) sum = fma((double)x[e], (double)x[e], sum);
    }
    sum = wave_sum_f64(sum);
    if (lane_id() == 0) norm[i] = sqrt(sum);
}
// Y = f A B + s B; columns of B and Y as the grid has them, rows ldb and ldy apart
__global__ __launch_bounds__(kProdThreads) void calib_float_apply_kernel(const float* A, const float* B, int D, int ldb, float f, float s, float* Y, int ldy)
{
    calib_product<float, float, true, float>(A, B, D, ldb, [&](int i, int j, float v) {
        Y[(size_t)i * ldy + j] = s != 0.f ? fmaf(s, B[(size_t)i * ldb + j], f * v) : f * v;
    });
}

// Row i of G goes to row rank of S, rank = number of rows with a larger norm (equal ones by row index), with its norm.
__global__ __launch_bounds__(kCalThreads) void calib_sort_kernel(const double* __restrict__ G, const double* __restrict__ norm, int D,
                                                                 double* __restrict__ S, double* __restrict__ sorted)
{
    __shared__ int cnt[kCalThreads / kWave];
    const int i = blockIdx.x, tid = threadIdx.x;
    const int rank = calib_rank(norm, D, i, cnt);
    if (tid == 0) sorted[rank] = norm[i];
    for (int d = tid * 2; d < D; d += kCalThreads * 2)
        *reinterpret_cast<f64x2*>(S + (size_t)rank * D + d) = *reinterpret_cast<const f64x2*>(G + (size_t)i * D + d);
}

}  // namespace sals
