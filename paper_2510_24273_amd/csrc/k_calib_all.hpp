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
// The polar factor is found by Newton-Schulz steps in fp32 (X <- a X - b X X^T X, scaled by the bounds of its singular values:
// J. Chen, E. Chow, "A stable scaling of Newton-Schulz for improving the sign function computation of a Hermitian matrix",
// 2014), and only *found* there: what is left, delta = X X^T - I (1e-6), is formed in fp64 and taken out to third order,
// G <- (I - delta / 2 + 3/8 delta^2) X G, with fp64 products.  What a transformation does to G is orthogonal to 1e-16 like a
// rotation made in fp64, and which transformation is made decides nothing but how fast the rows converge.  (D = 1024, r = 640:
// eigenvalues off by 1.5e-14 of themselves against a 64-bit eigensolver, by 2.0e-14 with sweeps alone.)
#pragma once
#include "common.hpp"
#include "k_calib.hpp"
#include "k_gemm.hpp"

namespace sals {

// ---- 64 x 64 tiles of products of [D, D] matrices --------------------------------------------------------------------
__device__ __forceinline__ f64x4 mma_step(double a, double b, f64x4 c) { return mma_f64(a, b, c); }
__device__ __forceinline__ f32x4 mma_step(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
template <typename ACC> struct mma_tile;   // result element e of a 16 x 16 tile: row, column lane % 16
template <> struct mma_tile<double> { typedef f64x4 acc; static __device__ __forceinline__ int row(int kg, int e) { return kg + 4 * e; } };
template <> struct mma_tile<float> { typedef f32x4 acc; static __device__ __forceinline__ int row(int kg, int e) { return 4 * kg + e; } };

// Tile (blockIdx.y, blockIdx.x) of A B^T (NN: of A B, B in doubles), summed in ACC.  A step is 128 bytes of a row: 32 floats or 16 doubles
// of the contraction.  Both operands go from memory straight into LDS, three steps ahead in four stages; eight waves, each half
// of a step's contraction for a quarter of the tile.  16-byte piece p of row r lies at piece p ^ ((r >> 1) & 7): no bank conflicts.
// Bound by the matrix cores from D = 2048 on (131 TFLOP/s in fp32, 66 in fp64); at D = 1024, one tile per compute unit, 22 and 38 us
// a product, where operands straight from memory took 33 and 47 (rows a power of two apart, and four waves asking for each).
// finish(part, row, col, e, value): called by the first four waves, element e = 0 .. 15 of lane's sixteen.
constexpr int kProdThreads = 512, kProdStages = 4;
template <typename TA, typename TB, bool NN> constexpr size_t prod_lds()
{
    return (size_t)kProdStages * (8192 + (NN ? 128 / sizeof(TA) * 64 * sizeof(TB) : 8192));
}
template <typename TA, typename TB, bool NN, typename ACC, typename Finish>
__device__ __forceinline__ void calib_product(const TA* A, const TB* B, int D, Finish finish)
{
    static_assert(NN ? sizeof(TB) == 8 : sizeof(TA) == sizeof(TB), "operand layout");
    constexpr int KS = 128 / (int)sizeof(TA), EPV = 16 / (int)sizeof(TA), B_BYTES = NN ? KS * 512 : 8192, STAGE = 8192 + B_BYTES, ST = kProdStages;
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
    const uint32_t off_b = NN ? (uint32_t)(wave * 2 + (lane >> 5)) * (uint32_t)D * 8 + ((lane & 31) << 4) : off_a;
    const unsigned char* a = reinterpret_cast<const unsigned char*>(A + (size_t)r0 * D);
    const unsigned char* b = reinterpret_cast<const unsigned char*>(NN ? B + c0 : B + (size_t)c0 * D);
    const int n = D / KS;   // (at least 8)
    auto load = [&](int s) {
        const size_t t = (size_t)min(s, n - 1);   // (past the end: a step that nothing reads any more)
        const uint32_t st = lds0 + (uint32_t)(s % ST) * STAGE + wave * 1024;
        load_lds16(a + t * 128, off_a, st);
        if (NN) {
#pragma unroll
            for (int i = 0; i < NB; ++i) load_lds16(b + (t * KS + 16 * i) * D * 8, off_b, st + 8192 * (1 + i));
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
                    y[u][e] = (ACC)*reinterpret_cast<const TB*>(st + 8192 + ((ks * 4 + kg) * EPV + e) * 512 + (cc + 16 * u) * 8);
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

// Y = G + f A B (ADD), or f A B.  Y may be G, not B.
template <typename TA, bool ADD>
__global__ __launch_bounds__(kProdThreads) void calib_apply_kernel(const TA* A, const double* B, const double* G, double f, double* Y, int D)
{
    calib_product<TA, double, true, double>(A, B, D, [&](int r, int c, double v) {
        const size_t at = (size_t)r * D + c;
        Y[at] = ADD ? fma(f, v, G[at]) : f * v;
    });
}

// ---- Angles -----------------------------------------------------------------------------------------------------------
// From G G^T, rows' norms in `norm`.
// ALL: E as above (fp32) for the pairs that are not orthogonal to 1e-12 and of which one row has a squared norm of at least a
// thousandth of the r-th largest one (smaller ones hardly move a leading row); found: per tile {sum of its squares over the pairs with
// a leading row, largest of them}.  The rows are sorted.
// Otherwise: E = -t (fp64), t = ab / d, over the pairs that are not orthogonal to working precision and of which one row has a squared
// norm >= lead; where both have, their cosine counts as well as t (beside a far larger row, t is small long before the smaller
// row's direction is right); found: per tile {largest |t| (at most 1/2), sum of t^2}.
constexpr double kAllOpen = 1e-24, kAllTail = 1e-3;
template <bool ALL>
__global__ __launch_bounds__(kProdThreads) void calib_angles_kernel(const double* __restrict__ G, int D, const double* __restrict__ norm,
                                                                    int r, double lead, void* __restrict__ E_out, f64x2* __restrict__ found)
{
    __shared__ f64x2 s_found[4];
    if (ALL) { const double nr = norm[r - 1]; lead = 0.999 * nr * nr; }
    double most = 0.0, sum = 0.0;
    calib_product<double, double, false, double>(G, G, D, [&](int i, int j, double ab) {
        const double ni = norm[i], nj = norm[j], aa = ni * ni, bb = nj * nj, d = bb - aa, hi = fmax(aa, bb);
        const size_t at = (size_t)i * D + j;
        if (ALL) {
            const bool counts = i != j && hi >= kAllTail * lead && ab * ab > kAllOpen * (aa * bb);
            const double s = counts ? ab * rsqrt_f64(fma(4.0 * ab, ab, d * d)) : 0.0;
            const double e = d < 0.0 || (d == 0.0 && i > j) ? s : -s;
            static_cast<float*>(E_out)[at] = (float)e;
            if (i < j && hi >= lead) { most = fmax(most, fabs(e)); sum += e * e; }
        } else {
            const bool counts = i != j && hi >= lead && jac_open(aa, bb, ab);
            const double th = counts ? ab / d : 0.0;
            if (counts && i < j) {
                most = fmax(most, fabs(ab) / fmax(fabs(d), 2.0 * fabs(ab)));
                if (fmin(aa, bb) >= lead) most = fmax(most, fabs(ab) / (ni * nj));
                sum += th * th;
            }
            static_cast<double*>(E_out)[at] = -th;
        }
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { most = fmax(most, __shfl_xor(most, o, kWave)); sum += __shfl_xor(sum, o, kWave); }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0 && wave < 4) s_found[wave] = f64x2{most, sum};
    __syncthreads();
    if (threadIdx.x == 0)
        found[blockIdx.y * gridDim.x + blockIdx.x] = f64x2{fmax(fmax(s_found[0].x, s_found[1].x), fmax(s_found[2].x, s_found[3].x)),
                                                           (s_found[0].y + s_found[1].y) + (s_found[2].y + s_found[3].y)};
}

// ---- Polar factor -----------------------------------------------------------------------------------------------------
// O = d I + s S + t T + f A B^T in fp32 (S, T: N > 0, N > 1).  SQUARE: also the sum of squares of every tile of O.
template <int N, bool SQUARE>
__global__ __launch_bounds__(kProdThreads) void calib_polar_kernel(const float* A, const float* B, int D, float f, float d, float s,
                                                                   const float* S, float t, const float* T, float* O, double* square)
{
    __shared__ double s_sum[4];
    double sum = 0.0;
    calib_product<float, float, false, float>(A, B, D, [&](int i, int j, float v) {
        const size_t at = (size_t)i * D + j;
        float o = f * v;
        if (N > 0) o = fmaf(s, S[at], o);
        if (N > 1) { o = fmaf(t, T[at], o); o += i == j ? d : 0.f; }
        O[at] = o;
        if (SQUARE) sum += (double)o * (double)o;
    });
    if (!SQUARE) return;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, kWave);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0 && wave < 4) s_sum[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) square[blockIdx.y * gridDim.x + blockIdx.x] = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}
// delta = X X^T - I, summed in fp64, and its rounding to fp32
__global__ __launch_bounds__(kProdThreads) void calib_defect_kernel(const float* X, int D, double* delta, float* delta32)
{
    calib_product<float, float, false, double>(X, X, D, [&](int i, int j, double v) {
        const double o = i == j ? v - 1.0 : v;
        delta[(size_t)i * D + j] = o;
        delta32[(size_t)i * D + j] = (float)o;
    });
}
// delta <- -delta / 2 + 3/8 delta^2 (the square, 1e-12, from the fp32 rounding)
__global__ __launch_bounds__(kProdThreads) void calib_correction_kernel(const float* delta32, int D, double* delta)
{
    calib_product<float, float, false, float>(delta32, delta32, D, [&](int i, int j, float v) {
        const size_t at = (size_t)i * D + j;
        delta[at] = fma(0.375, (double)v, -0.5 * delta[at]);
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
