// Offline calibration (Sec. 4.2): covariance of the calibration keys, C = K^T K, and its leading eigenvectors.
//
//   covariance   The contraction runs over the tokens, the axis along which the keys are NOT contiguous.  bf16: token rows
//                go to LDS as they lie and the matrix operands come out of transposing LDS reads (calib_cov_kernel).
//                fp32: the keys of a chunk are transposed once (calib_transpose_kernel, a plain LDS tile transpose) and
//                the product is then the row-by-row form the matrix-core GEMM of the prompt compression computes,
//                C += K^T (K^T)^T.  Either way fp32 tile sums over at most 4096 tokens are added to the fp64 matrix.
//   eigenvectors One-sided Jacobi on the rows of G = R, the Cholesky factor of C + shift I = R^T R: a plane rotation of rows
//                p, q makes them orthogonal.  With J the product of all rotations, G = J R keeps G^T G = C + shift I; once
//                all rows are orthogonal, the normalised rows are eigenvectors of C and the squared row norms less the shift
//                the eigenvalues, so no rotation matrix is kept.  (Starting from the rows of C itself, as a first form did,
//                works on C^2: 15 to 32 sweeps instead of about 10, since the off-diagonal part has twice the dynamic range
//                to lose.)
//                A sweep rotates every pair of rows once: a first step inside 32-row blocks, then D / 32 - 1 steps of
//                disjoint pairs of such blocks (round-robin).  A step is two launches: one forms the pairs' 64 x 64 Gram
//                matrices, a second one rotates them to orthogonality in LDS and applies the accumulated rotations to the
//                rows with the fp64 matrix instructions.  Where that is faster, orthogonal transformations of all rows at
//                once take the place of most sweeps (k_calib_all.hpp).
//                Rows, Gram matrices and everything that is applied to the rows: fp64 throughout.
#pragma once
#include "common.hpp"
#include "k_gemm.hpp"

namespace sals {

constexpr int kCalTile = 64;        // transpose tile (elements)
constexpr int kCalThreads = 256;    // workgroup of the row kernels (D is a multiple of it)
constexpr int kCalMaxD = 8192;

// XT[d, t] = X[t, d] for t < n, zero for n <= t < n_pad; X [n, D], XT [D, n_pad]
__global__ __launch_bounds__(256) void calib_transpose_kernel(const float* __restrict__ X, float* __restrict__ XT, long long n, int D,
                                                              long long n_pad)
{
    __shared__ float tile[kCalTile][kCalTile + 2];
    const long long t0 = (long long)blockIdx.x * kCalTile;
    const int d0 = blockIdx.y * kCalTile;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;  // 64 x 4
#pragma unroll
    for (int i = 0; i < kCalTile; i += 4) {
        const long long t = t0 + ty + i;
        const int d = d0 + tx;
        tile[ty + i][tx] = t < n && d < D ? X[(size_t)t * D + d] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kCalTile; i += 4) {
        const int d = d0 + ty + i;
        const long long t = t0 + tx;
        if (d < D && t < n_pad) XT[(size_t)d * n_pad + t] = tile[tx][ty + i];
    }
}

// Covariance of bf16 keys, C += X^T X, as tiles of 256 x 256 of the upper triangle: P[slice][tile] = the fp32 tile sums over
// one slice of the tokens (at most 4096 of them).  grid (tiles * slices), 512 threads, one workgroup per compute unit.
// Matrix-bound: 1.04 PFLOP/s sustained at D = 4096, 32768 tokens (560 us for 1088 items of 0.54 GFLOP, 545 to 575 from run
// to run), what the chip's power leaves of its rate on such operands (cutting the last, partly filled round into quarter items
// changed nothing).  The additions of the whole rounds' tiles run on the compute units that the last round leaves idle
// (cov_first_tiles): 588 to 610 us a call against 644 to 665 with all of them behind; 260 against 286 at 12000 tokens, 212
// against 225 at 8192.  A transposing copy of the keys, 256 x 128 tiles staged through registers and an addition per 4096 tokens
// took 1400 us.
//
// The contraction runs over the tokens, the axis along which the keys are not contiguous: token rows go to LDS as they
// lie in memory (32 tokens x 256 columns for either side, 16 bytes per lane without passing through registers, four
// stages) and the MFMA operands are read with the transposing LDS read.  64-byte pieces of a row are stored at their
// index XOR a number made of token bits that differ among the eight rows one read touches: no bank conflicts.
// Eight waves of 128 x 64: while the MFMAs of one half step (16 tokens) run, the fragments of the next are read; one
// barrier per 32 tokens, which also publishes the step after, and the loads of the step three ahead are issued behind it.
constexpr int kCovTile = 256, kCovStep = 32, kCovStages = 4;
constexpr int kCovSide = kCovStep * kCovTile * 2;              // bytes of one operand's stage
constexpr size_t kCovLds = (size_t)kCovStages * 2 * kCovSide;  // 128 KB
__device__ u32x4 g_cov_zero;                                   // stands in for tokens past the end

__device__ __forceinline__ void cov_tile(int id, int nt, int* row, int* col)  // tiles of the upper triangle, row by row
{
    int r = 0;
    while (id >= nt - r) { id -= nt - r; ++r; }
    *row = r; *col = r + id;
}

// C[i, j] += sum over the slices of P[slice][tile][i, j] in slice order, in fp64, for i <= j, and the same value to C[j, i]:
// one 32 x 32 block of a tile by 256 threads (x), with 32 * 33 doubles of LDS.  Every thread of the workgroup has to come here (barrier).
__device__ __forceinline__ void cov_add(double* __restrict__ C, const float* __restrict__ P, int D, int nt, int slices, int tile,
                                        int block, int x, double* __restrict__ t)
{
    int tr, tc;
    cov_tile(tile, nt, &tr, &tc);
    const int bi = block >> 3, bj = block & 7;
    const int i0 = tr * kCovTile + bi * 32, j0 = tc * kCovTile + bj * 32;
    const bool live = i0 < D && j0 < D && j0 >= i0;
    const int tx = x & 7, ty = x >> 3;  // four columns of one row per thread
    if (live) {
        const float* src = P + (size_t)tile * (kCovTile * kCovTile) + (bi * 32 + ty) * kCovTile + bj * 32 + tx * 4;
        const size_t stride = (size_t)(nt * (nt + 1) / 2) * (kCovTile * kCovTile);
        double* dst = C + (size_t)(i0 + ty) * D + j0 + tx * 4;
        double s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = 0.0;
        for (int z0 = 0; z0 < slices; z0 += 8) {  // eight slices requested together, from clamped slice numbers
            f32x4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = ld16_f32_stream(src + (size_t)min(z0 + u, slices - 1) * stride);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (z0 + u < slices) { s[0] += (double)v[u].x; s[1] += (double)v[u].y; s[2] += (double)v[u].z; s[3] += (double)v[u].w; }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double c = dst[e] + s[e];
            t[ty * 33 + tx * 4 + e] = c;
            if (i0 < j0 || ty <= tx * 4 + e) dst[e] = c;
        }
    }
    __syncthreads();
    if (live) {
        double* mir = C + (size_t)(j0 + ty) * D + i0 + tx * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i0 < j0 || ty > tx * 4 + e) mir[e] = t[(tx * 4 + e) * 33 + ty];
    }
}

// tiles tile0 .. tile0 + n_tiles; workgroups behind theirs add up tiles 0, 1, ... of an earlier launch (32 workgroups each)
__global__ __launch_bounds__(512, 2) void calib_cov_kernel(const bf16_t* __restrict__ X, long long n_tok, int D, int nt,
                                                           int slice_tok, int slices, float* __restrict__ P, int tile0, int n_tiles,
                                                           double* __restrict__ C)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];  // [stage][A | B]
    if ((int)blockIdx.x >= n_tiles * slices) {
        const int id = (int)blockIdx.x - n_tiles * slices, part = (int)threadIdx.x >> 8;
        cov_add(C, P, D, nt, slices, id >> 5, (id & 31) * 2 + part, threadIdx.x & 255, reinterpret_cast<double*>(lds) + part * (32 * 33));
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int wm = wave >> 2, wn = wave & 3;
    // consecutive ids go to different XCDs: each XCD takes a run of the list (slice slowest), so the tiles that share token
    // rows meet in its L2
    int tile, slice;
    {
        const int total = n_tiles * slices;
        const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds, qn = total / kXcds, rem = total % kXcds;
        const int w = (xcd < rem ? xcd * (qn + 1) : rem * (qn + 1) + (xcd - rem) * qn) + slot;
        slice = w / n_tiles; tile = tile0 + w - slice * n_tiles;
    }
    int tr, tc;
    cov_tile(tile, nt, &tr, &tc);
    const long long t_begin = (long long)slice * slice_tok;
    const int n_live = (int)min((long long)slice_tok, n_tok - t_begin);   // tokens of this slice (the host gives it some)
    const int n_steps = (n_live + kCovStep - 1) / kCovStep;

    // This wave's share of a stage: two pieces of 1 KB (two token rows) of either operand.  Lane -> token lane / 32 of the
    // pair, position lane % 32 of 16 bytes.
    const uint32_t lds0 = lds_offset(lds);
    const unsigned char* src[2][2];
    int tok_in_step[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int t = (wave * 2 + u) * 2 + hi;                       // token within the step
        const int f = (t & 3) | ((t >> 3) & 1) << 2;
        const int piece = (((l32 >> 2) ^ f) << 2) | (l32 & 3);       // 16-byte piece of the tile row that lies at position l32
        tok_in_step[u] = t;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int col = min((s ? tc : tr) * kCovTile + piece * 8, D - 8);  // (columns past D: computed, never used)
            src[u][s] = reinterpret_cast<const unsigned char*>(X + (size_t)t_begin * D + col);
        }
    }
    const size_t row_bytes = (size_t)D * 2;
    auto load_step = [&](int step) {
        const int sc = min(step, n_steps - 1);                       // (past the end: a step that nothing reads any more)
        const uint32_t st = lds0 + (uint32_t)(step & (kCovStages - 1)) * (2 * kCovSide);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int t = sc * kCovStep + tok_in_step[u];
            const bool in = t < n_live;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const void* p = in ? static_cast<const void*>(src[u][s] + (size_t)t * row_bytes) : static_cast<const void*>(&g_cov_zero);
                load_lds16(p, st + s * kCovSide + (wave * 2 + u) * 1024);
            }
        }
    };

    // fragment addresses: 32 columns (one 64-byte slot of a row) x 16 tokens; lane -> column l32, tokens 8 hi .. 8 hi + 7
    const int tt = (lane & 15) >> 2, cc = lane & 3, half = (lane >> 4) & 1;
    const int f = tt | hi << 2;
    uint32_t a_at[4], b_at[2];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) a_at[mb] = (hi * 8 + tt) * 512 + (((wm * 4 + mb) ^ f) << 6) + half * 32 + cc * 8;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) b_at[nb] = kCovSide + (hi * 8 + tt) * 512 + (((wn * 2 + nb) ^ f) << 6) + half * 32 + cc * 8;
    struct Frags { u32x4 a[4], b[2]; };
    auto frag = [&](uint32_t at) {
        const s16x4 x = lds_read_tr(lds + at), y = lds_read_tr(lds + at + 4 * 512);
        const uint2 lo = __builtin_bit_cast(uint2, x), up = __builtin_bit_cast(uint2, y);
        return u32x4{lo.x, lo.y, up.x, up.y};
    };
    auto read_frags = [&](Frags& F, int stage, int ks) {
        const uint32_t o = stage * (2 * kCovSide) + ks * (16 * 512);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) F.b[nb] = frag(b_at[nb] + o);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) F.a[mb] = frag(a_at[mb] + o);
    };
    f32x16 acc[4][2];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;
    auto mma_frags = [&](const Frags& F) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) mma_op<bf16_t>::run(F.a[mb], F.b[nb], acc[mb][nb]);
    };

    load_step(0); load_step(1); load_step(2);
    vm_wait<8>();
    wg_barrier();
    Frags F0, F1;
    read_frags(F0, 0, 0);
    for (int s0 = 0; s0 < n_steps; s0 += kCovStages) {
#pragma unroll
        for (int u = 0; u < kCovStages; ++u) {
            if (s0 + u < n_steps) {  // uniform
                // steps up to s + 1 have landed, everywhere; every wave is done with step s - 1
                vm_wait<4>();
                wg_barrier();
                load_step(s0 + u + 3);
                read_frags(F1, u, 1);
                mma_frags(F0);
                read_frags(F0, (u + 1) & (kCovStages - 1), 0);
                mma_frags(F1);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // LDS reads
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
            }
        }
    }
    vm_wait<0>();  // (no load may land in LDS that another workgroup has been given)

    float* out = P + ((size_t)slice * (nt * (nt + 1) / 2) + tile) * (kCovTile * kCovTile);
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = wm * 128 + mb * 32 + (v >> 2) * 8 + hi * 4 + (v & 3);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                __builtin_nontemporal_store(acc[mb][nb][v], out + r * kCovTile + wn * 64 + nb * 32 + l32);
        }
}

// The additions alone, of the tiles from tile0 on: grid (64, tiles).  A stream: 486 MB in 101 us at D = 4096 and eight slices
// if all are left to it.
__global__ __launch_bounds__(256) void calib_cov_reduce_kernel(double* __restrict__ C, const float* __restrict__ P, int D, int nt,
                                                               int slices, int tile0)
{
    __shared__ double t[32 * 33];
    cov_add(C, P, D, nt, slices, tile0 + blockIdx.y, blockIdx.x, threadIdx.x, t);
}

// C[i, j] += sum over the slices of P[slice][i, j], for the elements the covariance kernel computed: those of the
// tiles (tile_rows x tile_cols) that reach the upper triangle.  Slices are added in slice order, in fp64.
__global__ __launch_bounds__(256) void calib_reduce_kernel(double* __restrict__ C, const float* __restrict__ P, int D,
                                                           int slices, int tile_rows, int tile_cols)
{
    const size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;  // four consecutive columns
    if (e >= (size_t)D * D) return;
    const int i = (int)(e / D), j = (int)(e % D);
    if (j / tile_cols < (i / tile_rows) * (tile_rows / tile_cols)) return;  // tile not computed (mirrored later)
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    for (int z = 0; z < slices; ++z) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(P + (size_t)z * D * D + e);
        s0 += (double)v.x; s1 += (double)v.y; s2 += (double)v.z; s3 += (double)v.w;
    }
    C[e] += s0; C[e + 1] += s1; C[e + 2] += s2; C[e + 3] += s3;
}

// C[i, j] = C[j, i] for i > j: the covariance kernel fills the tiles that reach the upper triangle only
__global__ __launch_bounds__(256) void calib_mirror_kernel(double* __restrict__ C, int D)
{
    __shared__ double tile[32][33];
    const int bi = blockIdx.y, bj = blockIdx.x;   // tile of rows bi*32.., columns bj*32..
    if (bj > bi) return;                           // (strictly upper tiles are sources only)
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
#pragma unroll
    for (int k = 0; k < 32; k += 8) tile[ty + k][tx] = C[(size_t)(bj * 32 + ty + k) * D + bi * 32 + tx];  // the upper twin, [col][row]
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 32; k += 8) {
        const int i = bi * 32 + ty + k, j = bj * 32 + tx;
        if (i > j) C[(size_t)i * D + j] = tile[tx][ty + k];
    }
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// pair k of step s in the round-robin schedule over n (even) rows: n - 1 steps, every pair once
__device__ __forceinline__ void calib_pair(int n, int s, int k, int* p, int* q)
{
    if (k == 0) { *p = n - 1; *q = s; return; }
    const int m = n - 1;
    *p = (s + k) % m;
    *q = (s - k + m) % m;
}

// ---- Cholesky factor ---------------------------------------------------------------------------------------------
// G holds a copy of C and becomes R (upper triangular, C + shift I = R^T R), in panels of kCalPanel rows.
//
// The shift (1e-14 of C's scale at first) keeps the pivots of eigenvalues that are zero to working precision positive, and
// leaves the eigenvectors as they are.  Dropping rows of small pivots instead is not safe without a search for the largest
// pivot: the row's other entries may be as large as the square root of the pivot times a later diagonal entry (a channel of
// little variance ahead of the one it follows: eigenvectors at 1e-8 of the largest eigenvalue came out wrong by 8e-4).  A
// factorisation whose pivots are all positive is backward stable whatever its pivots are, since the columns of R have the
// norms sqrt(C_jj + shift); one that meets another pivot (C is indefinite by more than the shift, as the covariance of fewer
// tokens than channels is by its fp32 sums) sets `fail` and the host starts again with 64 times the shift.
constexpr int kCalPanel = 64;
constexpr double kCalShift = 1e-14;

typedef double f64x4 __attribute__((ext_vector_type(4)));
// v_mfma_f64_16x16x4: lane holds A[l % 16][l / 16] and B[l / 16][l % 16]; result element i is row l / 16 + 4 i, column l % 16
__device__ __forceinline__ f64x4 mma_f64(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f64x4 mma_step(double a, double b, f64x4 c) { return mma_f64(a, b, c); }
__device__ __forceinline__ f32x4 mma_step(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
template <typename ACC> struct mma_tile;   // result element e of a 16 x 16 tile: row, column lane % 16
template <> struct mma_tile<double> { typedef f64x4 acc; static __device__ __forceinline__ int row(int kg, int e) { return kg + 4 * e; } };
template <> struct mma_tile<float> { typedef f32x4 acc; static __device__ __forceinline__ int row(int kg, int e) { return 4 * kg + e; } };

// x of lane K of the row of 16 lanes
template <int K> __device__ __forceinline__ double row16_value(double x)
{
    const int2 u = __builtin_bit_cast(int2, x);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, u.x, 0x150 + K, 0xf, 0xf, true),
                                                __builtin_amdgcn_update_dpp(0, u.y, 0x150 + K, 0xf, 0xf, true)));
}
template <typename F, int... K> __device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, K...>)
{
    (f(std::integral_constant<int, K>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F&& f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// 1 / sqrt(x) for normal x: the hardware's estimate and one third-order step (full precision)
__device__ __forceinline__ double rsqrt_f64(double x)
{
    const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Panel at row k0: every workgroup factors the 64 x 64 diagonal block by itself (repeating it beats another launch) and carries
// 64 columns of the panel along, all in LDS, 16 rows at a time: one wave factors the 16 x 16 diagonal block in registers (a column per
// lane, the pivot row passed along the lanes), two waves carry the columns behind it through the triangular solve (a column per
// thread), and the matrix cores take the 16 rows out of those below; of these the first wave takes the next diagonal block alone and
// factors it while the other waves do the rest.  Bound by the 64 dependent pivots.  15.4 us at D = 1024; 18.8 with the pivot row
// passed through scalar registers (two reads per element, and what did not fit of them spilled), 20.1 with the factoring behind all tiles as
// well; one pivot at a time over the whole block (a barrier and a division each) and a solve of 64 unrolled steps per column took 62.
// The factored block goes to `diag` (other workgroups still read the original).  grid max(1, (D - k0 - 64) / 64).
constexpr int kCholLd = 2 * kCalPanel + 2;   // row pitch: the diagonal block's columns, then the workgroup's 64 columns
// The shift is `f` times 1e-14 of `scale` (see calib_scale_kernel).
__global__ __launch_bounds__(256) void calib_chol_panel_kernel(double* __restrict__ G, int D, int k0, const double* __restrict__ scale, double f,
                                                               double* __restrict__ diag, int* __restrict__ fail)
{
    __shared__ double M[kCalPanel * kCholLd];
    __shared__ double invd[kCalPanel];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, kg = lane >> 4;
    const int c0 = k0 + kCalPanel + blockIdx.x * 64;
    const bool panel = c0 < D;   // uniform
    double* rows = G + (size_t)(k0 + wave) * D + lane;   // row u 4 + wave of the panel, column `lane` of a block
    const size_t four = (size_t)4 * D;
    {   // (all loads requested together)
        const int* const sc = reinterpret_cast<const int*>(scale);
        const int2 s2 = make_int2(ld_uniform_i32(sc), ld_uniform_i32(sc + 1));
        const double *block = rows + k0, *column = rows + (panel ? c0 : k0);   // (without a panel: again, and not used)
        double v[2][16];
#pragma unroll
        for (int u = 0; u < 16; ++u) { v[0][u] = *block; v[1][u] = *column; block += four; column += four; }
        const double shift = kCalShift * __builtin_bit_cast(double, s2) * f;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int i = u * 4 + wave;
            M[i * kCholLd + lane] = v[0][u] + (i == lane ? shift : 0.0);
            M[i * kCholLd + kCalPanel + lane] = v[1][u];
        }
    }
    bool good = true;
    auto factor_block = [&](int b) {   // by one wave
        double a[16], mine = 0.0;   // column l16 of the block (in every row of 16 lanes), 1 / pivot l16
#pragma unroll
        for (int r = 0; r < 16; ++r) a[r] = M[(b + r) * kCholLd + b + l16];
        static_for<16>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const double pv = row16_value<k>(a[k]);
            good = good && pv > 0.0;
            const double inv = pv > 0.0 ? rsqrt_f64(pv) : 0.0;
            a[k] *= inv;                                  // row k of the factor
            mine = l16 == k ? inv : mine;
            static_for<15 - k>([&](auto rc) {
                constexpr int r = k + 1 + decltype(rc)::value;
                a[r] = fma(-row16_value<r>(a[k]), a[k], a[r]);
            });
        });
        if (kg == 0) {
            invd[b + l16] = mine;
#pragma unroll
            for (int r = 0; r < 16; ++r) M[(b + r) * kCholLd + b + l16] = l16 >= r ? a[r] : 0.0;
        }
    };
    // tile (i, j) less what the 16 rows at b contribute to it, by one wave
    auto take_out = [&](int b, int i, int j) {
        f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double* r = M + (b + 4 * s + kg) * kCholLd + l16;
            acc = mma_f64(r[i], r[j], acc);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) M[(i + kg + 4 * e) * kCholLd + j + l16] -= acc[e];
    };
    __syncthreads();
#pragma unroll 1
    for (int b = 0; b < kCalPanel; b += 16) {
        // The first wave brings the diagonal block up to date and factors it, the others bring the other tiles (row block i, column block
        // j >= i) up to date meanwhile
        if (wave == 0) {
            if (b > 0) take_out(b - 16, b, b);
            asm volatile("" ::: "memory");   // (a wave's LDS instructions are carried out in order)
            __builtin_amdgcn_wave_barrier();
            factor_block(b);
        } else if (b > 0) {
            int t = 0;
#pragma unroll 1
            for (int i = b; i < kCalPanel; i += 16)
#pragma unroll 1
                for (int j = i == b ? i + 16 : i; j < (panel ? 2 : 1) * kCalPanel; j += 16)
                    if (t++ % 3 + 1 == wave) take_out(b - 16, i, j);   // uniform
        }
        __syncthreads();
        if (wave < 2 && tid >= b + 16) {   // column tid: forward substitution R_bb^T x = a
            double x[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = M[(b + r) * kCholLd + tid];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                x[k] *= invd[b + k];
#pragma unroll
                for (int m = k + 1; m < 16; ++m) x[m] -= M[(b + k) * kCholLd + b + m] * x[k];
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) M[(b + r) * kCholLd + tid] = x[r];
        }
        __syncthreads();
    }
    if (!good && lane == 0 && wave == 0 && blockIdx.x == 0) *fail = 1;
    if (blockIdx.x == 0) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int i = u * 4 + wave;
            diag[(size_t)(k0 + i) * kCalPanel + lane] = lane >= i ? M[i * kCholLd + lane] : 0.0;
        }
    }
    if (panel) {
#pragma unroll
        for (int u = 0; u < 16; ++u) { rows[c0] = M[(u * 4 + wave) * kCholLd + kCalPanel + lane]; rows += four; }
    }
}

// Trailing update behind the panel at k0: A[i, j] -= sum_k R[k, i] R[k, j] over the panel's 64 rows, 64 x 64 tiles that
// reach the upper triangle.  grid (tiles, tiles)
// Everything is requested together: a tile takes one memory round trip and 0.9 us of matrix instructions (5.7 us a launch; 10.5
// with the old values fetched behind the products, on half the waves).
__global__ __launch_bounds__(512) void calib_chol_update_kernel(double* __restrict__ G, int D, int k0)
{
    if (blockIdx.x < blockIdx.y) return;
    const int base = k0 + kCalPanel, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, kg = lane >> 4;
    const int i0 = base + blockIdx.y * 64 + (wave >> 1) * 16, c0 = base + blockIdx.x * 64 + (wave & 1) * 32;
    double x[kCalPanel / 4][3];
#pragma unroll
    for (int s = 0; s < kCalPanel / 4; ++s) {
        const double* r = G + (size_t)(k0 + 4 * s + kg) * D + l16;
        x[s][0] = r[i0]; x[s][1] = r[c0]; x[s][2] = r[c0 + 16];
    }
    f64x4 acc[2];
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[v][e] = G[(size_t)(i0 + kg + 4 * e) * D + c0 + v * 16 + l16];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < kCalPanel / 4; ++s)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[v] = mma_f64(-x[s][0], x[s][1 + v], acc[v]);
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) G[(size_t)(i0 + kg + 4 * e) * D + c0 + v * 16 + l16] = acc[v][e];
}

// the factored diagonal blocks into place, zeros below the diagonal
__global__ __launch_bounds__(256) void calib_chol_finish_kernel(double* __restrict__ G, int D, const double* __restrict__ diag)
{
    const int i = blockIdx.x, k0 = i / kCalPanel * kCalPanel;
    for (int j = threadIdx.x; j < k0 + kCalPanel; j += 256)
        G[(size_t)i * D + j] = j < k0 ? 0.0 : diag[(size_t)i * kCalPanel + j - k0];
}

// ---- Jacobi steps ------------------------------------------------------------------------------------------------------
// A sweep rotates every pair of rows once.  Its first step (calib_jacobi_inside) takes the pairs inside 32-row blocks, the
// others (calib_jacobi_rotate) disjoint pairs (P, Q) of such blocks, every row of P with every row of Q.  What a step costs
// beside its rotations (two launches, the matrix read twice and written once across the dies' caches, the sums of the partial
// Gram matrices) is the same for any block height: with 16-row blocks, 63 steps a sweep at D = 1024, it took 13 of the 18.7 us
// of a step, and at D = 4096 the step was bound by the stream of the matrix.
constexpr int kJacB = 16;                   // rows of a small block: 16 pairs of rows are rotated side by side
constexpr int kJacBig = 2 * kJacB;          // rows of a block of the schedule
constexpr int kJacTile = kJacB * kJacB;
constexpr int kJacRec = 3 * kJacTile;       // Gram matrix of a 32-row block: small blocks (0,0), (0,1), (1,1)
// Gram matrix of a pair (P, Q) of blocks, small blocks P0 P1 Q0 Q1 = 0 1 2 3: tiles (0,0) (0,1) (1,1) (0,2) (1,2), (2,2) (2,3)
// (3,3) (0,3) (1,3)
constexpr int kJacTiles = 10, kJacBigRec = kJacTiles * kJacTile;
constexpr int kTile00 = 0, kTile01 = 1, kTile11 = 2, kTile02 = 3, kTile12 = 4, kTile22 = 5, kTile23 = 6, kTile33 = 7, kTile03 = 8;
// tile of small blocks u <= v, and the blocks of a tile
__device__ __forceinline__ int jac_tile_of(int u, int v) { return (int)(0x7000650094208310ull >> (4 * (4 * u + v))) & 15; }
__device__ __forceinline__ int jac_tile_row(int t) { return (int)(0x1032210100ull >> (4 * t)) & 3; }
__device__ __forceinline__ int jac_tile_col(int t) { return (int)(0x3333222110ull >> (4 * t)) & 3; }

// first row of small block `sub` (0 .. 3: P0 P1 Q0 Q1) of the blocks p, q
__device__ __forceinline__ int jac_row(int p, int q, int sub) { return (sub < 2 ? p : q) * kJacBig + (sub & 1) * kJacB; }

// The waves' partial sums of NT 16 x 16 tiles, added in wave order and left by the first wave.
template <typename T, int NT>
__device__ __forceinline__ void jac_gram_store(const typename mma_tile<T>::acc (&acc)[NT], T (&red)[3][NT * kJacTile], T* __restrict__ out)
{
    const int lane = lane_id(), wave = threadIdx.x >> 6, l16 = lane & 15, kg = lane >> 4;
    if (wave > 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave - 1][t * kJacTile + mma_tile<T>::row(kg, e) * 16 + l16] = acc[t][e];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int at = t * kJacTile + mma_tile<T>::row(kg, e) * 16 + l16;
                out[at] = acc[t][e] + red[0][at] + red[1][at] + red[2][at];
            }
    }
}

// Partial Gram matrices of the 32-row blocks over one slice of the columns: part[slice][block][3][16][16].
// grid (blocks, slices); four waves, each taking every fourth group of 16 columns (a lane reads four consecutive columns
// of its row, which serve as four contraction steps of the fp64 MFMA for either operand).
__global__ __launch_bounds__(256) void calib_jacobi_inside_gram_kernel(const double* __restrict__ G, int pitch, int slice_cols, double* __restrict__ part)
{
    typedef double T;
    typedef typename mma_tile<T>::acc V4;
    __shared__ T red[3][kJacRec];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kg = lane >> 4;
    const T* gp = G + (size_t)(blockIdx.x * kJacBig + l16) * pitch + blockIdx.y * slice_cols + kg * 4;
    const T* gq = gp + (size_t)kJacB * pitch;
    V4 acc[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) acc[t] = V4{0, 0, 0, 0};
    for (int c = wave * 16; c < slice_cols; c += 64) {
        const V4 a = *reinterpret_cast<const V4*>(gp + c), b = *reinterpret_cast<const V4*>(gq + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc[0] = mma_step(a[e], a[e], acc[0]);
            acc[1] = mma_step(a[e], b[e], acc[1]);
            acc[2] = mma_step(b[e], b[e], acc[2]);
        }
    }
    jac_gram_store<T, 3>(acc, red, part + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kJacRec);
}

// Pairs of blocks of a step: those of a sweep, or neighbours
constexpr int kJacNearEven = -1, kJacNearOdd = -2;   // blocks 2 k, 2 k + 1; 2 k + 1, 2 k + 2 (the last one with the first)
__device__ __forceinline__ void jac_pair(int n, int step, int k, int* p, int* q)
{
    if (step >= 0) { calib_pair(n, step, k, p, q); return; }
    *p = 2 * k + (step == kJacNearOdd ? 1 : 0);
    *q = *p + 1 < n ? *p + 1 : 0;
}

// The same for the step's pairs of blocks: part[slice][pair][10][16][16], five tiles per workgroup (grid (pairs, slices, 2)).
// The pair index runs fastest in both launches of a step, so a pair's sums are written and read on one die.
template <typename T>
__global__ __launch_bounds__(256) void calib_jacobi_gram_kernel(const T* __restrict__ G, int D, int pitch, int step, int slice_cols,
                                                                T* __restrict__ part)
{
    typedef typename mma_tile<T>::acc V4;
    constexpr int NT = kJacTiles / 2;
    __shared__ T red[3][NT * kJacTile];
    int p, q;
    jac_pair(D / kJacBig, step, blockIdx.x, &p, &q);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, kg = lane >> 4;
    const bool half = blockIdx.z != 0;  // uniform
    const T* g[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = G + (size_t)(jac_row(p, q, u) + l16) * pitch + blockIdx.y * slice_cols + kg * 4;
    V4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = V4{0, 0, 0, 0};
    for (int c = wave * 16; c < slice_cols; c += 128) {  // two groups requested together, the second from a clamped column
        V4 x[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k) x[u][k] = *reinterpret_cast<const V4*>(g[k] + min(c + 64 * u, slice_cols - 16));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (c + 64 * u >= slice_cols) break;  // uniform
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const T p0 = x[u][0][e], p1 = x[u][1][e], q0 = x[u][2][e], q1 = x[u][3][e];
                // tiles (0,0) (0,1) (1,1) (0,2) (1,2), or (2,2) (2,3) (3,3) (0,3) (1,3)
                const T a = half ? q0 : p0, b = half ? q1 : p1, last = half ? q1 : q0;
                acc[0] = mma_step(a, a, acc[0]);
                acc[1] = mma_step(a, b, acc[1]);
                acc[2] = mma_step(b, b, acc[2]);
                acc[3] = mma_step(p0, last, acc[3]);
                acc[4] = mma_step(p1, last, acc[4]);
            }
        }
    }
    jac_gram_store<T, NT>(acc, red, part + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kJacBigRec + (half ? NT * kJacTile : 0));
}

// cosine and sine of the rotation (g_p, g_q) -> (c g_p - s g_q, s g_p + c g_q) that makes two rows with squared norms aa,
// bb and inner product ab orthogonal, by the smaller angle: with h = sqrt((bb-aa)^2 + 4 ab^2) the double angle has
// cosine |bb-aa| / h and sine 2 |ab| / h, so two reciprocal square roots do.  Rows orthogonal to working precision are left
// alone.  (No row is too small to count: beside a large one, a row of squared norm w left as it is moves the large one's
// eigenvector by up to w over its eigenvalue.)
__device__ __forceinline__ bool jac_open(double aa, double bb, double ab) { return ab * ab > 1e-30 * (aa * bb); }
__device__ __forceinline__ void jac_rotation(double aa, double bb, double ab, double* c, double* s, double* tan)
{
    const bool ok = jac_open(aa, bb, ab);
    // (the smallest normal number keeps two zero rows finite)
    const double d = bb - aa, hi = rsqrt_f64(fma(4.0 * ab, ab, fma(d, d, 2.2250738585072014e-308)));
    const double c2 = fma(0.5 * fabs(d), hi, 0.5), ci = rsqrt_f64(c2);
    uint2 ab_d = __builtin_bit_cast(uint2, ab);     // ab with its sign turned by d's
    ab_d.y ^= __builtin_bit_cast(uint2, d).y & 0x80000000u;
    *c = ok ? c2 * ci : 1.0;
    *s = ok ? __builtin_bit_cast(double, ab_d) * hi * ci : 0.0;
    *tan = *s * ci;
}
__device__ __forceinline__ bool jac_open(float aa, float bb, float ab) { return ab * ab > 1e-14f * (aa * bb); }
// (rows of norms whose fourth powers floats do not hold are left alone)
__device__ __forceinline__ void jac_rotation(float aa, float bb, float ab, float* c, float* s, float* tan)
{
    const float d = bb - aa, h2 = fmaf(4.f * ab, ab, d * d), hi = __builtin_amdgcn_rsqf(fmaxf(h2, 1e-30f));
    const bool ok = jac_open(aa, bb, ab) && h2 > 1e-30f;
    const float c2 = fmaf(0.5f * fabsf(d), hi, 0.5f), ci = __builtin_amdgcn_rsqf(c2);
    *c = ok ? c2 * ci : 1.f;
    *s = ok ? __uint_as_float(__float_as_uint(ab) ^ (__float_as_uint(d) & 0x80000000u)) * hi * ci : 0.f;
    *tan = *s * ci;
}
// What is applied to the rows turns by these: c so that c^2 + s^2 = 1 to rounding.  (As computed it is above 1 by 5e-17 on average
// where the angles are small, ten sweeps of which added 1.8e-13 to every eigenvalue at D = 1024.)
template <typename T> __device__ __forceinline__ T jac_unit(T c, T s) { return fma((T)0.5 * c, fma(-s, s, fma(-c, c, (T)1)), c); }
// (non-negative doubles are ordered like their bits; nothing waits for the result)
__device__ __forceinline__ void conv_max(double* at, double v)
{
    atomicMax(reinterpret_cast<unsigned long long*>(at), (unsigned long long)__double_as_longlong(v));
}

// value of the next lane of a row of 16 lanes (the last lane gets the first one's)
__device__ __forceinline__ double row16_next(double v)
{
    const int2 u = __builtin_bit_cast(int2, v);
    int2 w;
    w.x = __builtin_amdgcn_update_dpp(u.x, u.x, 0x12f, 0xf, 0xf, false);  // row_ror:15
    w.y = __builtin_amdgcn_update_dpp(u.y, u.y, 0x12f, 0xf, 0xf, false);
    return __builtin_bit_cast(double, w);
}

__device__ __forceinline__ float row16_next(float v)
{
    const int u = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(u, u, 0x12f, 0xf, 0xf, false));
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <typename T> struct vec2;
template <> struct vec2<double> { typedef f64x2 type; };
template <> struct vec2<float> { typedef f32x2 type; };
constexpr int kJacLd = 2 * kJacB + 1;   // row pitch of a 32 x 32 matrix in LDS
constexpr int kJacLt = kJacB + 1;       // of a 16 x 16 tile

// The rotations of two small blocks A, B of rows: every row of A with every row of B, 16 rounds of 16 disjoint pairs on the
// blocks' Gram matrix, by two waves (jac_solve) while two more accumulate the rotations (jac_accumulate).
//
// Round t pairs row i of A with row i + t of B (mod 16).  Thread (i, m), m = 1 .. 8, keeps the 2 x 2 block of row pair i and
// column pair j = i + m in registers; the blocks of the other m are these transposed, and those of m = 0 are the pairs' own: the
// squared norms aa, bb and the inner product, zero after the rotation.  i is the lane of a row of 16 lanes, so the threads
// (i, 1), whose blocks hold the inner product of the pair that comes next, share one wave: it computes the next round's
// rotations right after its blocks' update.  Going to the next round, (B_i, B_j) moves by one lane (a lane rotation), (A_i, B_j)
// and (B_i, A_j) pass through LDS.  A round is one LDS round trip, a 2 x 2 block update, one rotation and one barrier: 0.27 us with
// two groups on a compute unit.  With all 256 blocks, and every wave computing rotations, it took 0.31 us for one group and 0.47
// for two (instruction issue); with every thread computing both rotations of its block from the whole matrix in LDS 0.6 for one.
template <typename T> struct JacRounds {
    typedef typename vec2<T>::type T2;
    T2 cs[kJacB + 1][kJacB];          // [round][pair]: cosine and sine
    T2 unused[3 * kJacB];             // (where the other lanes of the wave that computes rotations write)
    T cross[2][2][8][kJacB];        // [round parity][(A_i, B_j) | (B_i, A_j)][m - 1][i]
    T zero[2][2][8][kJacB];         // (first row: the product that a round's rotation made zero)
};
struct JacPlace { int i, j, m; bool rotates; };
__device__ __forceinline__ JacPlace jac_place(int w)  // w: the wave's number in its group
{
    JacPlace t;
    t.i = lane_id() & 15; t.m = 1 + w * 4 + (lane_id() >> 4); t.j = (t.i + t.m) & 15; t.rotates = w == 0;
    return t;
}
// In: thread (i, m)'s elements (A_i, A_j), (A_i, B_j), (B_i, A_j), (B_i, B_j) and pair i's squared norms aa, bb and inner product
// ab.  Out: b00, b11 and, in the threads (i, 1), aa and bb after the rounds (of row i of either block).  17 barriers.
template <typename T>
__device__ __forceinline__ void jac_solve(JacRounds<T>& L, const JacPlace& at, T& b00, T b01, T b10, T& b11, T& aa,
                                          T& bb, T ab)
{
    typedef typename vec2<T>::type T2;
    const int i = at.i, j = at.j, i1 = (i + 1) & 15, half = lane_id() >> 4;
    // where a round finds (A_i, B_j): thread (i, m + 1)'s, and for m = 8 thread (i + 9, 7)'s (B_i, A_j); and (B_i, A_j): thread
    // (i + 1, m - 1)'s (of m = 1 it is zero)
    T* const from01 = at.m < 8 ? &L.cross[0][0][at.m][i] : &L.cross[0][1][6][(i + 9) & 15];
    T* const from10 = at.m > 1 ? &L.cross[0][1][at.m - 2][i1] : &L.zero[0][0][0][i];
    T* const to = &L.cross[0][0][at.m - 1][i];
    constexpr int kParity = 2 * 8 * kJacB;
    const T2 *Ri = &L.cs[0][i], *Rj = &L.cs[0][j];
    T2* out = half == 0 ? &L.cs[0][i] : &L.unused[(half - 1) * kJacB + i];
    const int step = half == 0 ? kJacB : 0;
    auto rotation = [&](T abt) {
        T c, s, tan;
        jac_rotation(aa, bb, abt, &c, &s, &tan);
        *out = T2{c, s};
        out += step;
        aa = fma(-tan, abt, aa);
        bb = row16_next(fma(tan, abt, bb));   // (the next round's B row)
    };
    auto round = [&](auto parity, bool last) {
        constexpr int odd = decltype(parity)::value * kParity;
        const T c = Ri->x, s = Ri->y, cj = Rj->x, sj = Rj->y;
        Ri += kJacB; Rj += kJacB;
        b01 = from01[odd];
        b10 = from10[odd];
        const T r00 = c * b00 - s * b10, r01 = c * b01 - s * b11, r10 = s * b00 + c * b10, r11 = s * b01 + c * b11;
        const T n01 = sj * r00 + cj * r01;
        to[kParity - odd] = n01;
        to[kParity - odd + 8 * kJacB] = cj * r10 - sj * r11;
        if (at.rotates && !last) rotation(n01);  // uniform
        b00 = cj * r00 - sj * r01;
        b11 = row16_next(sj * r10 + cj * r11);
        __syncthreads();
    };
    // (the first round reads what its threads hold from where a round's threads read)
    *from01 = b01;
    if (at.m > 1) *from10 = b10;
    else from10[0] = b10, from10[kParity] = 0;
    if (at.rotates) rotation(ab);  // uniform
    __builtin_amdgcn_s_setprio(2);  // (the accumulating waves fill the gaps)
    __syncthreads();
#pragma unroll 1
    for (int t = 0; t < kJacB; t += 2) {  // (not unrolled further: every launch starts with cold instruction caches)
        round(std::integral_constant<int, 0>{}, false);
        if (t == 0 && at.m == 1) from10[0] = 0;
        round(std::integral_constant<int, 1>{}, t + 2 == kJacB);
    }
    __builtin_amdgcn_s_setprio(0);
}
// The largest |sin| of the 256 rotations among those that involved a row of squared norm >= lead (the rows that can still
// change a leading eigenvector), by the norms the rows of A and B have now (diagonals of pitch `ld`); one wave, every lane
// gets it.
__device__ __forceinline__ double jac_largest(const JacRounds<double>& L, const double* A, const double* B, int ld, double lead)
{
    const int l16 = lane_id() & 15, kg = lane_id() >> 4;
    double smax = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int t = k * 4 + kg;
        smax = fmax(A[l16 * (ld + 1)], B[((l16 + t) & 15) * (ld + 1)]) >= lead ? fmax(smax, fabs(L.cs[t][l16].y)) : smax;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) smax = fmax(smax, __shfl_xor(smax, o, kWave));
    return smax;
}
// lane l: rows l % 16 of A and B of the accumulated matrix, kJacNc columns; 17 barriers.  (Sixteen moves: every row of B ends
// in its place.)
constexpr int kJacNc = 2 * kJacB / 8;   // columns per lane
template <typename T>
__device__ __forceinline__ void jac_accumulate(const JacRounds<T>& L, T (&x)[kJacNc], T (&y)[kJacNc])
{
    const int l16 = lane_id() & 15;
    __syncthreads();
#pragma unroll 1
    for (int t = 0; t < kJacB; ++t) {
        const typename vec2<T>::type R = L.cs[t][l16];
        const T c = jac_unit(R.x, R.y), s = R.y;
#pragma unroll
        for (int e = 0; e < kJacNc; ++e) {
            const T xe = x[e], ye = y[e];
            x[e] = c * xe - s * ye;
            y[e] = row16_next(s * xe + c * ye);
        }
        __syncthreads();
    }
}

// The pairs of rows inside a 32-row block, by 256 threads (t): 15 rounds inside its two small blocks (side by side, on whole matrices
// in LDS) and the 16 rounds between them.  In: the Gram matrix in the first of W.  Out: the accumulated rotations, pitch kJacLd, in turned(), behind
// a barrier (W is free then).
// conv: not null: keeps the largest |sin| of a rotation (see jac_largest).
template <typename T> struct JacInside {
    static constexpr int N = 2 * kJacB * kJacLd;
    T W[2 * N], Q[2][N];   // Gram matrix (two of them) and accumulated rotations
    __device__ T* turned() { return Q[(kJacB - 1) & 1]; }
    T conv[sizeof(T) == 8 ? kJacB : 1];   // (in floats nobody asks whether the rows have converged)
};
template <typename T>
__device__ __forceinline__ void jac_inside(JacInside<T>& sh, JacRounds<T>& rounds, int t256, double lead, double* __restrict__ conv)
{
    constexpr bool kConv = sizeof(T) == 8;
    constexpr int B2 = 2 * kJacB, LD = kJacLd;
    const int lane = t256 & 63, wave = __builtin_amdgcn_readfirstlane(t256 >> 6), l16 = lane & 15, kg = lane >> 4;
    const int i = t256 >> 4, j = t256 & 15;
    for (int e = t256; e < B2 * B2; e += 256) sh.Q[0][(e >> 5) * LD + (e & 31)] = (e >> 5) == (e & 31) ? 1 : 0;
    __syncthreads();
    int cur = 0;
    {
        auto inside = [&](int t, int k, int* a, int* b) {  // pair k of round t: k < 8 inside the first small block, otherwise the second
            calib_pair(kJacB, t, k & 7, a, b);
            *a += k < 8 ? 0 : kJacB; *b += k < 8 ? 0 : kJacB;
        };
        T smax = 0;
#pragma unroll 1
        for (int t = 0; t < kJacB - 1; ++t) {
            {
                int pi, qi, pj, qj;
                inside(t, i, &pi, &qi);
                inside(t, j, &pj, &qj);
                const T* W = sh.W + cur * sh.N; const T* Q = sh.Q[cur];
                T* Wn = sh.W + (cur ^ 1) * sh.N; T* Qn = sh.Q[cur ^ 1];
                const T aa = W[pi * LD + pi], bb = W[qi * LD + qi];
                const T b00 = W[pi * LD + pj], b01 = W[pi * LD + qj], b10 = W[qi * LD + pj], b11 = W[qi * LD + qj];
                const T x0 = Q[pi * LD + j], y0 = Q[qi * LD + j], x1 = Q[pi * LD + j + kJacB], y1 = Q[qi * LD + j + kJacB];
                T c, s, cj, sj, tan;
                jac_rotation(aa, bb, W[pi * LD + qi], &c, &s, &tan);
                jac_rotation(W[pj * LD + pj], W[qj * LD + qj], W[pj * LD + qj], &cj, &sj, &tan);
                if (kConv) smax = fmax(aa, bb) >= (T)lead ? fmax(smax, fabs(s)) : smax;
                const T r00 = c * b00 - s * b10, r01 = c * b01 - s * b11, r10 = s * b00 + c * b10, r11 = s * b01 + c * b11;
                Wn[pi * LD + pj] = cj * r00 - sj * r01;
                Wn[pi * LD + qj] = sj * r00 + cj * r01;
                Wn[qi * LD + pj] = cj * r10 - sj * r11;
                Wn[qi * LD + qj] = sj * r10 + cj * r11;
                const T cu = jac_unit(c, s);
                Qn[pi * LD + j] = cu * x0 - s * y0; Qn[qi * LD + j] = s * x0 + cu * y0;
                Qn[pi * LD + j + kJacB] = cu * x1 - s * y1; Qn[qi * LD + j + kJacB] = s * x1 + cu * y1;
            }
            __syncthreads();
            cur ^= 1;
        }
        if (kConv && j == 0) sh.conv[i] = smax;
    }
    T* const Qo = sh.turned();   // (= Q[cur])
    if (wave < 2) {
        const T* W = sh.W + cur * sh.N;
        const JacPlace at = jac_place(wave);
        T b00 = W[at.i * LD + at.j], b11 = W[(kJacB + at.i) * LD + kJacB + at.j];
        T aa = W[at.i * (LD + 1)], bb = W[(kJacB + at.i) * (LD + 1)];
        jac_solve<T>(rounds, at, b00, W[at.i * LD + kJacB + at.j], W[at.j * LD + kJacB + at.i], b11, aa, bb,
                  W[at.i * LD + kJacB + at.i]);
        if (at.m == 1) { T* const Wn = sh.W + (cur ^ 1) * sh.N; Wn[at.i * (LD + 1)] = aa; Wn[(kJacB + at.i) * (LD + 1)] = bb; }
    } else {
        T x[kJacNc], y[kJacNc];
        const int c0 = ((wave & 1) * 4 + kg) * kJacNc;
#pragma unroll
        for (int e = 0; e < kJacNc; ++e) { x[e] = Qo[l16 * LD + c0 + e]; y[e] = Qo[(kJacB + l16) * LD + c0 + e]; }
        jac_accumulate<T>(rounds, x, y);
#pragma unroll
        for (int e = 0; e < kJacNc; ++e) { Qo[l16 * LD + c0 + e] = x[e]; Qo[(kJacB + l16) * LD + c0 + e] = y[e]; }
    }
    __syncthreads();
    if constexpr (kConv) if (conv && wave == 3) {
        const double* W = sh.W + (cur ^ 1) * sh.N;
        double smax = jac_largest(rounds, W, W + kJacB * (LD + 1), LD, lead);
#pragma unroll
        for (int k = 0; k < kJacB; ++k) smax = fmax(smax, sh.conv[k]);
        if (lane == 0 && smax > 0.0) conv_max(conv, smax);
    }
}

// First step of a sweep: the pairs of rows inside every 32-row block (jac_inside); workgroup (block, slice) applies the accumulated
// rotations to its slice of the columns on the matrix cores.  Every slice repeats the small problem (the same numbers).
// conv[block] keeps the largest |sin| of a rotation since the host cleared it.
constexpr int kJacInsideThreads = 4 * kWave;
__global__ __launch_bounds__(kJacInsideThreads) void calib_jacobi_inside_kernel(double* __restrict__ G, int pitch, int slice_cols,
                                                                                const double* __restrict__ part, int n_part,
                                                                                const double* __restrict__ lead_at, double* __restrict__ conv)
{
    typedef double T;
    typedef typename mma_tile<T>::acc V4;
    constexpr int LD = kJacLd;
    __shared__ JacInside<T> sh;
    __shared__ JacRounds<T> s_rounds;
    const double lead = *lead_at;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, kg = lane >> 4;
    T* const gp = G + (size_t)blockIdx.x * kJacBig * pitch + blockIdx.y * slice_cols + l16;
    {
        const int i = tid >> 4, j = tid & 15;
        T w8[3][8];
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int u = 0; u < 8; ++u)
                w8[t][u] = part[((size_t)min(u, n_part - 1) * gridDim.x + blockIdx.x) * kJacRec + t * kJacTile + tid];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            T v = 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) v += u < n_part ? w8[t][u] : (T)0;
            const int r = i + (t == 2 ? kJacB : 0), c = j + (t >= 1 ? kJacB : 0);
            sh.W[r * LD + c] = v;
            if (t == 1) sh.W[c * LD + r] = v;
        }
    }
    jac_inside<T>(sh, s_rounds, tid, lead, blockIdx.y == 0 ? conv + blockIdx.x : nullptr);
    const T* const Qo = sh.turned();
    auto row_of = [&](int s) { return 16 * (s >> 2) + mma_tile<T>::row(kg, s & 3); };   // of the block, in contraction step s
    T qa[2][8];  // the accumulated rotations as MFMA operand: rows m 16 .. +16, contraction step s
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int s = 0; s < 8; ++s) qa[m][s] = Qo[(m * 16 + l16) * LD + row_of(s)];
    for (int c = wave * 16; c < slice_cols; c += 64) {
        T x[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) x[s] = gp[(size_t)row_of(s) * pitch + c];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            V4 acc = V4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 8; ++s) acc = mma_step(qa[m][s], x[s], acc);
#pragma unroll
            for (int e = 0; e < 4; ++e) gp[(size_t)row_of(4 * m + e) * pitch + c] = acc[e];
        }
    }
}

// Rotates the rows of the step's pairs of blocks.  Workgroup (pair, slice) adds up the pair's partial Gram matrices (64 x 64)
// and rotates P0 with Q0 beside P1 with Q1 and then P0 with Q1 beside P1 with Q0 (jac_solve, a group of four waves each); in
// between it brings the tiles (P0, Q1) and (P1, Q0) up to date with the accumulated rotations, on the matrix cores, as it
// applies them to its slice of the columns in the end: two products with 32 x 32 matrices, the first one's result being the
// second one's operand as it lies in the registers.  Every slice repeats the small problem (the same numbers): a launch between
// the two would cost more than its 32 dependent rounds.
// At D = 1024 (256 workgroups of 64 columns) the kernel takes 19.9 us behind 5.7 for the Gram matrices: 8.7 for the rounds, 2.3 for
// the partial sums, 2.4 for the last products, 1.1 between the halves, the rest for the launch and the matrix's way back to memory.
// A call at D = 1024, r = 640: 15.4 ms with 16-row blocks, 11.6 with these; at D = 4096 239 and 155.
constexpr int kJacThreads = 8 * kWave;   // waves 0, 1 and 2, 3: the groups' rounds; 4, 5 and 6, 7: their accumulated rotations
// INSIDE: the pairs inside the blocks first, in the same launch (rows in floats): group g's 256 threads rotate the pairs inside its block
// (jac_inside), and the pair's Gram matrix W becomes J W J^T, so that one launch for Gram matrices and one passage of the rows less do: 30
// us at D = 1024 behind 4 for the Gram matrices, in place of 4.6 + 17 + 4 + 15 us in two launches each.  A call at D = 1024, r = 640 2996 ->
// 2936 us, 2048 14.49 -> 14.31 ms.
template <typename T, bool INSIDE = false>
__global__ __launch_bounds__(kJacThreads) void calib_jacobi_rotate_kernel(T* __restrict__ G, int D, int pitch, int step, int slice_cols,
                                                                          const T* __restrict__ part, int n_part,
                                                                          const double* __restrict__ lead_at, double* __restrict__ conv)
{
    constexpr int LD = kJacLd, LT = kJacLt;
    const double lead = sizeof(T) == 8 ? *lead_at : 0.0;
    typedef typename mma_tile<T>::acc V4;
    typedef typename vec2<T>::type V2;
    __shared__ T S[kJacTiles][kJacB * LT];          // Gram matrix
    __shared__ T J[2][2][2 * kJacB * LD];           // [half][group] accumulated rotations
    __shared__ T H[2][kJacB * LD];
    __shared__ JacRounds<T> s_rounds[2];
    __shared__ int s_any;
    int p, q;
    jac_pair(D / kJacBig, step, blockIdx.x, &p, &q);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, kg = lane >> 4;
    const bool solver = wave < 4;   // uniform
    const int grp = (wave >> 1) & 1;
    const JacPlace at = jac_place(wave & 1);
    const int i = at.i, j = at.j;

    // partial Gram matrices (at most 8), two elements per load, and this wave's first column tile, all requested together
    constexpr int NP = kJacBigRec / 2, NV = (NP + kJacThreads - 1) / kJacThreads;
    V2 w8[NV][8];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int u = 0; u < 8; ++u)
            w8[v][u] = *reinterpret_cast<const V2*>(part + ((size_t)min(u, n_part - 1) * gridDim.x + blockIdx.x) * kJacBigRec +
                                                       2 * min(tid + v * kJacThreads, NP - 1));
    T* g[4];   // small block u
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = G + (size_t)jac_row(p, q, u) * pitch + blockIdx.y * slice_cols + l16;
    T x[4][4];  // small block u, contraction step s: row mma_tile::row(kg, s)
    auto load_tile = [&](int c) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int s = 0; s < 4; ++s) x[u][s] = g[u][(size_t)mma_tile<T>::row(kg, s) * pitch + c];
    };
    if (wave * 16 < slice_cols) load_tile(wave * 16);  // uniform
    if (tid == 0) s_any = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int e = 2 * (tid + v * kJacThreads), tile = e / kJacTile, pos = e % kJacTile;
        V2 sum = V2{0, 0};
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            sum.x += u < n_part ? w8[v][u].x : (T)0;
            sum.y += u < n_part ? w8[v][u].y : (T)0;
        }
        if (e < kJacBigRec) {
            S[tile][(pos >> 4) * LT + (pos & 15)] = sum.x;
            S[tile][(pos >> 4) * LT + (pos & 15) + 1] = sum.y;
        }
    }
    __syncthreads();
    // tiles of small blocks P_a and Q_b
    auto tile_pp = [](int a) { return a ? kTile11 : kTile00; };
    auto tile_qq = [](int b) { return b ? kTile33 : kTile22; };
    auto tile_pq = [](int a, int b) { return (b ? kTile03 : kTile02) + a; };
    T* Jin[2] = {nullptr, nullptr};   // INSIDE: rotations inside P and Q
    if constexpr (INSIDE) {
        __shared__ JacInside<T> s_in[2];
        const int blk = tid >> 8;
        {   // small blocks 2 blk and 2 blk + 1
            const int r = (tid >> 4) & 15, c = l16;
            T* const W = s_in[blk].W;
            const T v01 = S[blk ? kTile23 : kTile01][r * LT + c];
            W[r * LD + c] = S[blk ? kTile22 : kTile00][r * LT + c];
            W[(kJacB + r) * LD + kJacB + c] = S[blk ? kTile33 : kTile11][r * LT + c];
            W[r * LD + kJacB + c] = v01;
            W[(kJacB + c) * LD + r] = v01;
        }
        jac_inside<T>(s_in[blk], s_rounds[blk], tid & 255, 0.0, nullptr);
        Jin[0] = s_in[0].turned();
        Jin[1] = s_in[1].turned();
        // rows of J W where the blocks' Gram matrices were (of Q's rows the columns of Q only) ...
        constexpr int LY = 2 * LD;
        static_assert(LY >= 4 * kJacB, "64 columns");
        auto rows_of = [&](int g, int m, int n) {
            V4 acc = V4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int k = 4 * s + kg, u = 2 * g + (s >> 2), r = k & 15;
                const int tile = u <= n ? jac_tile_of(u, n) : jac_tile_of(n, u);
                acc = mma_step(Jin[g][(m * 16 + l16) * LD + k], S[tile][u <= n ? r * LT + l16 : l16 * LT + r], acc);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) s_in[g].W[(m * 16 + mma_tile<T>::row(kg, e)) * LY + n * 16 + l16] = acc[e];
        };
        rows_of(0, wave >> 2, wave & 3);
        if (wave < 4) rows_of(1, wave >> 1, 2 + (wave & 1));
        __syncthreads();
        // ... and times J^T
        for (int tile = wave; tile < kJacTiles; tile += 8) {
            const int u = jac_tile_row(tile), v = jac_tile_col(tile), g = v >> 1;
            const T* const Y = s_in[u >> 1].W;
            V4 acc = V4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 8; ++s)
                acc = mma_step(Y[((u & 1) * 16 + l16) * LY + g * 32 + 4 * s + kg], Jin[g][((v & 1) * 16 + l16) * LD + 4 * s + kg], acc);
#pragma unroll
            for (int e = 0; e < 4; ++e) S[tile][mma_tile<T>::row(kg, e) * LT + l16] = acc[e];
        }
        __syncthreads();
    }
    // nothing to rotate (most pairs of the last sweeps): the rounds would leave everything as it is
    if constexpr (!INSIDE) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int a = wave >> 2, r = (tid >> 4) & 15, c = l16;
            if (jac_open(S[tile_pp(a)][r * (LT + 1)], S[tile_qq(b)][c * (LT + 1)], S[tile_pq(a, b)][r * LT + c])) s_any = 1;
        }
        __syncthreads();
        if (!s_any) return;  // uniform, and the same in every slice of the pair
    }

#pragma unroll 1
    for (int h = 0; h < 2; ++h) {
        const int b = h ? 1 - grp : grp;  // group's blocks: P_grp and Q_b
        T* const A = S[tile_pp(grp)]; T* const C = S[tile_qq(b)];
        const T* const B = S[tile_pq(grp, b)];
        if (solver) {
            T b00 = A[i * LT + j], b11 = C[i * LT + j], aa = A[i * (LT + 1)], bb = C[i * (LT + 1)];
            jac_solve<T>(s_rounds[grp], at, b00, B[i * LT + j], B[j * LT + i], b11, aa, bb, B[i * (LT + 1)]);
            A[i * LT + j] = A[j * LT + i] = b00;
            C[i * LT + j] = C[j * LT + i] = b11;
            if (at.m == 1) { A[i * (LT + 1)] = aa; C[i * (LT + 1)] = bb; }
        } else {
            T xr[kJacNc], yr[kJacNc];
            const int c0 = ((wave & 1) * 4 + kg) * kJacNc;
#pragma unroll
            for (int e = 0; e < kJacNc; ++e) { xr[e] = c0 + e == l16 ? 1 : 0; yr[e] = c0 + e == kJacB + l16 ? 1 : 0; }
            jac_accumulate<T>(s_rounds[grp], xr, yr);
            T* Jo = J[h][grp];
#pragma unroll
            for (int e = 0; e < kJacNc; ++e) { Jo[l16 * LD + c0 + e] = xr[e]; Jo[(kJacB + l16) * LD + c0 + e] = yr[e]; }
        }
        __syncthreads();
        if constexpr (sizeof(T) == 8) if (!solver && (wave & 1) && blockIdx.y == 0) {   // (in floats nobody asks)
            const double smax = jac_largest(s_rounds[grp], A, C, LT, lead);
            if (lane == 0 && smax > 0.0) conv_max(conv + blockIdx.x, smax);
        }
        if (h == 1) break;
        // (P0, Q1) and (Q0, P1) after the first half: rows of J1 W J2^T, W = the Gram matrix between (P0, Q0) and (P1, Q1).
        // First H[m] = rows m of J1 W, a 16 x 16 tile per wave, then H[m] times the other rows of J2.
        if (wave < 4) {
            const int m = wave >> 1, n = wave & 1;
            V4 acc = V4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 4; ++s)  // rows 4 s + kg of P0 ...
                acc = mma_step(J[0][0][(m * 16 + l16) * LD + 4 * s + kg], S[n ? kTile03 : kTile01][(4 * s + kg) * LT + l16], acc);
#pragma unroll
            for (int s = 0; s < 4; ++s)  // ... and of Q0 (the tile (P1, Q0) the other way round)
                acc = mma_step(J[0][0][(m * 16 + l16) * LD + kJacB + 4 * s + kg],
                              n ? S[kTile23][(4 * s + kg) * LT + l16] : S[kTile12][l16 * LT + 4 * s + kg], acc);
#pragma unroll
            for (int e = 0; e < 4; ++e) H[m][mma_tile<T>::row(kg, e) * LD + n * 16 + l16] = acc[e];
        }
        __syncthreads();
        if (wave < 2) {
            const int m = wave;
            V4 acc = V4{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 8; ++s)
                acc = mma_step(H[m][l16 * LD + 4 * s + kg], J[0][1][((1 - m) * 16 + l16) * LD + 4 * s + kg], acc);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (m == 0) S[kTile03][mma_tile<T>::row(kg, e) * LT + l16] = acc[e];
                else S[kTile12][l16 * LT + mma_tile<T>::row(kg, e)] = acc[e];
            }
        }
        __syncthreads();
    }
    // row of small block u of the result: J[h][group] times the group's two small blocks (A, B), half after half
    for (int c = wave * 16; c < slice_cols; c += 8 * 16) {
        if (c != wave * 16) load_tile(c);
        auto turn = [&](const T* Jt, T (&A)[4], T (&B)[4]) {
            asm volatile("" ::: "memory");  // (the operands of all products at once do not fit into the registers)
            V4 acc[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                acc[m] = V4{0, 0, 0, 0};
#pragma unroll
                for (int s = 0; s < 8; ++s)
                    acc[m] = mma_step(Jt[(m * 16 + l16) * LD + 16 * (s >> 2) + mma_tile<T>::row(kg, s & 3)], s < 4 ? A[s & 3] : B[s & 3], acc[m]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) { A[e] = acc[0][e]; B[e] = acc[1][e]; }
        };
        if constexpr (INSIDE) { turn(Jin[0], x[0], x[1]); turn(Jin[1], x[2], x[3]); }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int a = 0; a < 2; ++a) turn(J[h][a], x[a], x[2 + (h ? 1 - a : a)]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int s = 0; s < 4; ++s) g[u][(size_t)mma_tile<T>::row(kg, s) * pitch + c] = x[u][s];
    }
}

// norm of every row and the sign that makes the row's largest component positive
__global__ __launch_bounds__(kCalThreads) void calib_rownorm_kernel(const double* __restrict__ G, int D, double* __restrict__ lam,
                                                                    double* __restrict__ sgn)
{
    __shared__ double red[kCalThreads / kWave], bestv[kCalThreads / kWave], bests[kCalThreads / kWave];
    __shared__ int besti[kCalThreads / kWave];
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double acc = 0.0, bv = -1.0, bs = 1.0;
    int bi = 0;
    for (int d = tid; d < D; d += kCalThreads) {
        const double g = G[(size_t)i * D + d];
        acc += g * g;
        if (fabs(g) > bv) { bv = fabs(g); bi = d; bs = g < 0.0 ? -1.0 : 1.0; }
    }
    acc = wave_sum_f64(acc);
    // largest |component|, the first index among equals
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(bv, o, kWave), os = __shfl_xor(bs, o, kWave);
        const int oi = __shfl_xor(bi, o, kWave);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; bs = os; }
    }
    if (lane == 0) { red[wave] = acc; bestv[wave] = bv; besti[wave] = bi; bests[wave] = bs; }
    __syncthreads();
    if (tid == 0) {
        double sum = 0.0;
        for (int w = 0; w < kCalThreads / kWave; ++w) sum += red[w];
        int best = 0;
        for (int w = 1; w < kCalThreads / kWave; ++w)
            if (bestv[w] > bestv[best] || (bestv[w] == bestv[best] && besti[w] < besti[best])) best = w;
        lam[i] = sqrt(sum);
        sgn[i] = bests[best];
    }
}

// number of rows with a norm larger than row i's (equal ones by row index), by a whole workgroup
__device__ __forceinline__ int calib_rank(const double* __restrict__ norm, int D, int i, int (&cnt)[kCalThreads / kWave])
{
    const int tid = threadIdx.x;
    const double li = norm[i];
    int c = 0;
    for (int j = tid; j < D; j += kCalThreads) {
        const double lj = norm[j];
        c += (lj > li || (lj == li && j < i)) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
    if ((tid & 63) == 0) cnt[tid >> 6] = c;
    __syncthreads();
    int rank = 0;
#pragma unroll
    for (int w = 0; w < kCalThreads / kWave; ++w) rank += cnt[w];
    return rank;
}

// A little less than the square of the r-th largest norm (so that the r-th row itself is among the leading ones), a workgroup a row.  (5
// us at D = 1024; the host would have to wait for the norms, 22 us, and select among them, 10.)
__global__ __launch_bounds__(kCalThreads) void calib_lead_kernel(const double* __restrict__ norm, int D, int r, double* __restrict__ lead)
{
    __shared__ int cnt[kCalThreads / kWave];
    const int rank = calib_rank(norm, D, blockIdx.x, cnt);
    if (threadIdx.x == 0 && rank == r - 1) *lead = 0.999 * norm[blockIdx.x] * norm[blockIdx.x];
}
// the largest norm, between the largest diagonal entry and the largest eigenvalue of a covariance (not a number if one of them is not)
__global__ __launch_bounds__(kCalThreads) void calib_scale_kernel(const double* __restrict__ norm, int D, double* __restrict__ scale)
{
    __shared__ double s_most[kCalThreads / kWave];
    const int tid = threadIdx.x;
    auto larger = [](double a, double b) { return a != a || a > b ? a : b; };
    double most = 0.0;
    for (int i = tid; i < D; i += kCalThreads) most = larger(norm[i], most);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) most = larger(__shfl_xor(most, o, kWave), most);
    if ((tid & 63) == 0) s_most[tid >> 6] = most;
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < kCalThreads / kWave; ++w) most = larger(s_most[w], most);
        *scale = most;
    }
}

// Row i of G takes rank = number of rows with a larger norm (equal ones by row index); eigval[rank] = lambda_i and, for
// rank < r, column rank of U [D, r] = sgn_i * row i of G / |row i|, rounded to the storage type (a zero row gives a
// zero column); row i of C = lambda_i times the eigenvector.  ROOT: G is the rotated Cholesky factor (lambda = squared
// norm less the shift, at least zero); otherwise its rows are C's own, orthogonal as they came (lambda = norm).
template <typename T, bool ROOT>
__global__ __launch_bounds__(kCalThreads) void calib_select_kernel(const double* __restrict__ G, const double* __restrict__ norm,
                                                                   const double* __restrict__ sgn, int D, int r, double shift,
                                                                   double* __restrict__ eigval, T* __restrict__ U,
                                                                   double* __restrict__ C)
{
    __shared__ int cnt[kCalThreads / kWave];
    const int i = blockIdx.x, tid = threadIdx.x;
    const double li = norm[i];
    const int rank = calib_rank(norm, D, i, cnt);
    const double lam = ROOT ? fmax(li * li - shift, 0.0) : li;
    if (tid == 0) eigval[rank] = lam;
    const double s = li > 0.0 ? sgn[i] / li : 0.0, to_c = ROOT && li > 0.0 ? lam / li : 0.0;
    for (int d = tid; d < D; d += kCalThreads) {
        const double g = G[(size_t)i * D + d];
        if (rank < r) elem<T>::store(U + (size_t)d * r + rank, (float)(s * g));
        if (ROOT) C[(size_t)i * D + d] = to_c * g;
    }
}

}  // namespace sals
