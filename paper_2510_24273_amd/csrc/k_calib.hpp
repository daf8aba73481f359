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
//                A step takes D / 32 disjoint pairs of 16-row blocks: one launch forms the pairs' 32 x 32 Gram
//                matrices, a second one rotates them to orthogonality in LDS and applies the accumulated rotations to
//                the rows with the fp64 matrix instructions; D / 16 - 1 steps (round-robin over the blocks) rotate every
//                pair of rows once: one sweep.  One launch per row-pair step (D - 1 of them a sweep, each streaming the
//                whole matrix) was bound by its launches up to D = 1024 and by the stream above.
//                fp64 throughout.
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
// changed nothing).  With the addition below 636 to 650 us a call; a transposing copy of the keys, 256 x 128 tiles staged through
// registers and an addition per 4096 tokens took 1400 us.
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

__global__ __launch_bounds__(512, 2) void calib_cov_kernel(const bf16_t* __restrict__ X, long long n_tok, int D, int nt,
                                                           int slice_tok, int slices, float* __restrict__ P)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];  // [stage][A | B]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int wm = wave >> 2, wn = wave & 3;
    // consecutive ids go to different XCDs: each XCD takes a run of the list (slice slowest), so the tiles that share token
    // rows meet in its L2
    int tile, slice;
    {
        const int n_tiles = nt * (nt + 1) / 2, total = n_tiles * slices;
        const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds, qn = total / kXcds, rem = total % kXcds;
        const int w = (xcd < rem ? xcd * (qn + 1) : rem * (qn + 1) + (xcd - rem) * qn) + slot;
        slice = w / n_tiles; tile = w - slice * n_tiles;
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

// C[i, j] += sum over the slices of P[slice][tile][i, j] in slice order, in fp64, for i <= j, and the same value to C[j, i].
// One workgroup per 32 x 32 block of the upper triangle's tiles; grid (64, tiles).  A stream: 486 MB in 101 us at D = 4096
// and eight slices.
__global__ __launch_bounds__(256) void calib_cov_reduce_kernel(double* __restrict__ C, const float* __restrict__ P, int D, int nt,
                                                               int slices)
{
    __shared__ double t[32][33];
    int tr, tc;
    cov_tile(blockIdx.y, nt, &tr, &tc);
    const int bi = blockIdx.x >> 3, bj = blockIdx.x & 7;
    const int i0 = tr * kCovTile + bi * 32, j0 = tc * kCovTile + bj * 32;
    if (i0 >= D || j0 >= D || j0 < i0) return;  // uniform
    const int tx = threadIdx.x & 7, ty = threadIdx.x >> 3;  // four columns of one row per thread
    const float* src = P + (size_t)blockIdx.y * (kCovTile * kCovTile) + (bi * 32 + ty) * kCovTile + bj * 32 + tx * 4;
    const size_t stride = (size_t)gridDim.y * (kCovTile * kCovTile);
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
        t[ty][tx * 4 + e] = c;
        if (i0 < j0 || ty <= tx * 4 + e) dst[e] = c;
    }
    __syncthreads();
    double* mir = C + (size_t)(j0 + ty) * D + i0 + tx * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (i0 < j0 || ty > tx * 4 + e) mir[e] = t[tx * 4 + e][ty];
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

// Panel at row k0: every workgroup factors the 64 x 64 diagonal block by itself (a row of it per four threads, the pivot
// row passed through LDS, one barrier per pivot: 64 dependent steps are what the kernel takes, so repeating them beats
// another launch) and then carries 64 columns of the panel through the triangular solve, one column per thread of its first
// wave (with a column on every thread the four waves' broadcast reads of the factor are bound by the LDS).  The
// factored block goes to `diag` (other workgroups still read the original).  grid max(1, (D - k0 - 64) / 64).
__global__ __launch_bounds__(256) void calib_chol_panel_kernel(double* __restrict__ G, int D, int k0, double shift,
                                                               double* __restrict__ diag, int* __restrict__ fail)
{
    __shared__ double row[2][kCalPanel];
    __shared__ double Rk[kCalPanel][kCalPanel + 1];
    __shared__ double invd[kCalPanel];
    const int tid = threadIdx.x, i = tid >> 2, j0 = (tid & 3) * 16;
    const int c = k0 + kCalPanel + blockIdx.x * 64 + tid;
    double a[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) a[e] = G[(size_t)(k0 + i) * D + k0 + j0 + e] + (j0 + e == i ? shift : 0.0);
    double pv_i = 0.0;
    for (int k = 0; k < kCalPanel; ++k) {
        double* rk = row[k & 1];
        if (i == k) {
#pragma unroll
            for (int e = 0; e < 16; ++e) rk[j0 + e] = a[e];
        }
        __syncthreads();
        const double pv = rk[k];
        if (i == k) pv_i = pv;
        if (i > k) {
            const double f = pv > 0.0 ? rk[i] / pv : 0.0;
#pragma unroll
            for (int e = 0; e < 16; ++e) a[e] -= f * rk[j0 + e];
        }
    }
    const double inv = pv_i > 0.0 ? rsqrt(pv_i) : 0.0;
    if (!(pv_i > 0.0) && blockIdx.x == 0) *fail = 1;
    if ((tid & 3) == 0) invd[i] = inv;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        a[e] = j0 + e >= i ? a[e] * inv : 0.0;
        Rk[i][j0 + e] = a[e];
        if (blockIdx.x == 0) diag[(size_t)(k0 + i) * kCalPanel + j0 + e] = a[e];
    }
    __syncthreads();
    if (tid >= 64 || c >= D) return;
    // forward substitution R_kk^T x = a, the column's values in registers
    double x[kCalPanel];
#pragma unroll
    for (int k = 0; k < kCalPanel; ++k) x[k] = G[(size_t)(k0 + k) * D + c];
#pragma unroll
    for (int k = 0; k < kCalPanel; ++k) {
        x[k] *= invd[k];
#pragma unroll
        for (int m = k + 1; m < kCalPanel; ++m) x[m] -= Rk[k][m] * x[k];
    }
#pragma unroll
    for (int k = 0; k < kCalPanel; ++k) G[(size_t)(k0 + k) * D + c] = x[k];
}

typedef double f64x4 __attribute__((ext_vector_type(4)));
// v_mfma_f64_16x16x4: lane holds A[l % 16][l / 16] and B[l / 16][l % 16]; result element i is row l / 16 + 4 i, column l % 16
__device__ __forceinline__ f64x4 mma_f64(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Trailing update behind the panel at k0: A[i, j] -= sum_k R[k, i] R[k, j] over the panel's 64 rows, 64 x 64 tiles that
// reach the upper triangle.  grid (tiles, tiles)
__global__ __launch_bounds__(256) void calib_chol_update_kernel(double* __restrict__ G, int D, int k0)
{
    if (blockIdx.x < blockIdx.y) return;
    const int base = k0 + kCalPanel, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, kg = lane >> 4;
    const int i0 = base + blockIdx.y * 64 + (wave >> 1) * 32, c0 = base + blockIdx.x * 64 + (wave & 1) * 32;
    f64x4 acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int s = 0; s < kCalPanel / 4; ++s) {
        const double* r = G + (size_t)(k0 + 4 * s + kg) * D + l16;
        const double a0 = r[i0], a1 = r[i0 + 16], b0 = r[c0], b1 = r[c0 + 16];
        acc[0][0] = mma_f64(a0, b0, acc[0][0]); acc[0][1] = mma_f64(a0, b1, acc[0][1]);
        acc[1][0] = mma_f64(a1, b0, acc[1][0]); acc[1][1] = mma_f64(a1, b1, acc[1][1]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) G[(size_t)(i0 + u * 16 + kg + 4 * e) * D + c0 + v * 16 + l16] -= acc[u][v][e];
}

// the factored diagonal blocks into place, zeros below the diagonal
__global__ __launch_bounds__(256) void calib_chol_finish_kernel(double* __restrict__ G, int D, const double* __restrict__ diag)
{
    const int i = blockIdx.x, k0 = i / kCalPanel * kCalPanel;
    for (int j = threadIdx.x; j < k0 + kCalPanel; j += 256)
        G[(size_t)i * D + j] = j < k0 ? 0.0 : diag[(size_t)i * kCalPanel + j - k0];
}

// ---- Jacobi step over pairs of row blocks ----------------------------------------------------------------------------
constexpr int kJacB = 16;               // rows per block
constexpr int kJacRec = 3 * kJacB * kJacB;  // a pair's Gram matrix: blocks (P,P), (P,Q), (Q,Q)

// Partial Gram matrices of the step's block pairs over one slice of the columns: part[slice][pair][3][16][16].
// grid (slices, pairs); four waves, each taking every fourth group of 16 columns (a lane reads four consecutive columns
// of its row, which serve as four contraction steps of the fp64 MFMA for either operand).
__global__ __launch_bounds__(256) void calib_jacobi_gram_kernel(const double* __restrict__ G, int D, int step, int slice_cols,
                                                                double* __restrict__ part)
{
    __shared__ double red[3][kJacRec];
    int p, q;
    calib_pair(D / kJacB, step, blockIdx.y, &p, &q);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, kg = lane >> 4;
    const double* gp = G + (size_t)(p * kJacB + l16) * D + blockIdx.x * slice_cols + kg * 4;
    const double* gq = G + (size_t)(q * kJacB + l16) * D + blockIdx.x * slice_cols + kg * 4;
    f64x4 acc[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int c = wave * 16; c < slice_cols; c += 128) {  // two groups requested together, the second from a clamped column
        f64x4 a[2], b[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            a[u] = *reinterpret_cast<const f64x4*>(gp + min(c + 64 * u, slice_cols - 16));
            b[u] = *reinterpret_cast<const f64x4*>(gq + min(c + 64 * u, slice_cols - 16));
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (c + 64 * u < slice_cols) {  // uniform
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[0] = mma_f64(a[u][e], a[u][e], acc[0]);
                    acc[1] = mma_f64(a[u][e], b[u][e], acc[1]);
                    acc[2] = mma_f64(b[u][e], b[u][e], acc[2]);
                }
            }
        }
    }
    // the waves' sums, added in wave order
    if (wave > 0) {
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave - 1][t * 256 + (kg + 4 * e) * 16 + l16] = acc[t][e];
    }
    __syncthreads();
    if (wave == 0) {
        double* out = part + ((size_t)blockIdx.x * gridDim.y + blockIdx.y) * kJacRec;
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int at = t * 256 + (kg + 4 * e) * 16 + l16;
                out[at] = acc[t][e] + red[0][at] + red[1][at] + red[2][at];
            }
    }
}

// 1 / sqrt(x) for normal x: the hardware's estimate and one third-order step (full precision)
__device__ __forceinline__ double jac_rsqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
// cosine and sine of the rotation (g_p, g_q) -> (c g_p - s g_q, s g_p + c g_q) that makes two rows with squared norms aa,
// bb and inner product ab orthogonal, by the smaller angle: with h = sqrt((bb-aa)^2 + 4 ab^2) the double angle has
// cosine |bb-aa| / h and sine 2 |ab| / h, so two reciprocal square roots do.  Rows orthogonal to working precision are left
// alone.  (No row is too small to count: beside a large one, a row of squared norm w left as it is moves the large one's
// eigenvector by up to w over its eigenvalue.)
__device__ __forceinline__ bool jac_open(double aa, double bb, double ab) { return ab * ab > 1e-30 * (aa * bb); }
__device__ __forceinline__ bool jac_rotation(double aa, double bb, double ab, double* c, double* s)
{
    const bool ok = jac_open(aa, bb, ab);
    const double d = bb - aa, hi = jac_rsqrt(fma(d, d, 4.0 * ab * ab));
    const double c2 = fma(0.5 * fabs(d), hi, 0.5), ci = jac_rsqrt(c2);
    *c = ok ? c2 * ci : 1.0;
    *s = ok ? (d >= 0.0 ? ab : -ab) * hi * ci : 0.0;
    return ok;
}
// (non-negative doubles are ordered like their bits; nothing waits for the result)
__device__ __forceinline__ void conv_max(double* at, double v)
{
    atomicMax(reinterpret_cast<unsigned long long*>(at), (unsigned long long)__double_as_longlong(v));
}

// Rotates the rows of the step's block pairs.  Workgroup (slice, pair) adds up the pair's partial Gram matrices, runs the
// rotations on the 32 x 32 Gram matrix (16 rounds of 16 disjoint pairs: every row of P with every row of Q; in the
// sweep's first step 15 rounds more, the pairs inside the blocks) while accumulating them into a 32 x 32 matrix, and
// applies that to its slice of the columns on the matrix cores.  Every slice repeats the small problem (the same
// numbers): a launch between the two would cost more than its 16 dependent rounds.  In a round thread (i, j) rotates the
// 2 x 2 block of row pair i and column pair j; what the next round's threads need passes through one of two LDS buffers
// (one barrier per round), what belongs to a row of P stays with its thread.  A round is a chain of LDS reads, two
// reciprocal square roots and LDS writes, bound by instruction issue of the one wave per SIMD.
// (The rounds in fp32, with the accumulated matrix re-orthogonalised in fp64, were no faster: 0.5 against 0.6 us a round.)
// conv[pair] keeps the largest |sin| of a rotation, since the host cleared it, that involved a row of squared norm >=
// lead (the rows that can still change a leading eigenvector).
__global__ __launch_bounds__(256) void calib_jacobi_rotate_kernel(double* __restrict__ G, int D, int step, int slice_cols,
                                                                  const double* __restrict__ part, int n_part, double lead,
                                                                  double* __restrict__ conv)
{
    constexpr int B2 = 2 * kJacB, LD = B2 + 1, LB = kJacB + 1;
    __shared__ double Wb[2][B2 * LD], Qb[2][B2 * LD];   // Gram matrix and accumulated rotations
    __shared__ double s_diag[B2], s_conv[kJacB];
    __shared__ int s_any[2];
    int p, q;
    calib_pair(D / kJacB, step, blockIdx.y, &p, &q);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15, kg = lane >> 4;

    // partial Gram matrices (at most 8) and the first two column tiles of this wave, all requested together
    double w8[3][8];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int u = 0; u < 8; ++u)
            w8[t][u] = part[((size_t)min(u, n_part - 1) * gridDim.y + blockIdx.y) * kJacRec + t * 256 + tid];
    double* const gp = G + (size_t)(p * kJacB + kg) * D + blockIdx.x * slice_cols + l16;
    double* const gq = G + (size_t)(q * kJacB + kg) * D + blockIdx.x * slice_cols + l16;
    double x[2][8];  // tile u, contraction step s: row 4 s + kg of (P, Q)
    auto load_tiles = [&](int c0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = min(c0 + 64 * u, slice_cols - 16);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                x[u][s] = gp[(size_t)(4 * s) * D + c];
                x[u][4 + s] = gq[(size_t)(4 * s) * D + c];
            }
        }
    };
    load_tiles(wave * 16);
    const int i = tid >> 4, j = tid & 15;
    if (tid < 2) s_any[tid] = 0;
    double v[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        v[t] = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) v[t] += u < n_part ? w8[t][u] : 0.0;
        const int r = i + (t == 2 ? kJacB : 0), c = j + (t >= 1 ? kJacB : 0);
        Wb[0][r * LD + c] = v[t];
        if (t == 1) Wb[0][c * LD + r] = v[t];
        if (r == c) s_diag[r] = v[t];
    }
    for (int e = tid; e < B2 * B2; e += 256) Qb[0][(e >> 5) * LD + (e & 31)] = (e >> 5) == (e & 31) ? 1.0 : 0.0;
    __syncthreads();
    // nothing to rotate (most pairs of the last sweeps): the rounds would leave everything as it is
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const int r = i + (t == 2 ? kJacB : 0), c = j + (t >= 1 ? kJacB : 0);
        if (r != c && (t == 1 || step == 0) && jac_open(s_diag[r], s_diag[c], v[t])) s_any[0] = 1;
    }
    __syncthreads();
    if (!s_any[0]) return;  // uniform, and the same in every slice of the pair

    double smax = 0.0;
    bool any = false;
    int cur = 0;
    if (step == 0) {  // the pairs inside the blocks, on whole matrices
        auto inside = [&](int t, int k, int* a, int* b) {  // pair k of round t: k < 8 inside P, otherwise inside Q
            calib_pair(kJacB, t, k & 7, a, b);
            *a += k < 8 ? 0 : kJacB; *b += k < 8 ? 0 : kJacB;
        };
        for (int t = 0; t < kJacB - 1; ++t) {
            int pi, qi, pj, qj;
            inside(t, i, &pi, &qi);
            inside(t, j, &pj, &qj);
            const double* W = Wb[cur]; const double* Q = Qb[cur];
            double* Wn = Wb[cur ^ 1]; double* Qn = Qb[cur ^ 1];
            const double aa = W[pi * LD + pi], bb = W[qi * LD + qi];
            const double b00 = W[pi * LD + pj], b01 = W[pi * LD + qj], b10 = W[qi * LD + pj], b11 = W[qi * LD + qj];
            const double x0 = Q[pi * LD + j], y0 = Q[qi * LD + j], x1 = Q[pi * LD + j + kJacB], y1 = Q[qi * LD + j + kJacB];
            double c, s, cj, sj;
            const bool ok = jac_rotation(aa, bb, W[pi * LD + qi], &c, &s);
            jac_rotation(W[pj * LD + pj], W[qj * LD + qj], W[pj * LD + qj], &cj, &sj);
            any |= ok;
            smax = fmax(aa, bb) >= lead ? fmax(smax, fabs(s)) : smax;
            const double r00 = c * b00 - s * b10, r01 = c * b01 - s * b11, r10 = s * b00 + c * b10, r11 = s * b01 + c * b11;
            Wn[pi * LD + pj] = cj * r00 - sj * r01;
            Wn[pi * LD + qj] = sj * r00 + cj * r01;
            Wn[qi * LD + pj] = cj * r10 - sj * r11;
            Wn[qi * LD + qj] = sj * r10 + cj * r11;
            Qn[pi * LD + j] = c * x0 - s * y0; Qn[qi * LD + j] = s * x0 + c * y0;
            Qn[pi * LD + j + kJacB] = c * x1 - s * y1; Qn[qi * LD + j + kJacB] = s * x1 + c * y1;
            __syncthreads();
            cur ^= 1;
        }
    }
    // every row of P with every row of Q: round t pairs row i of P with row (i + t) mod 16 of Q
    const double* Qd;
    {
        double b00 = Wb[cur][i * LD + j];
        double x0 = Qb[cur][i * LD + j], x1 = Qb[cur][i * LD + j + kJacB];
        const double b01 = Wb[cur][i * LD + kJacB + j], b11 = Wb[cur][(kJacB + i) * LD + kJacB + j];
        const double y0 = Qb[cur][(kJacB + i) * LD + j], y1 = Qb[cur][(kJacB + i) * LD + j + kJacB];
        // the two buffers: (P,Q) block [16][17], (Q,Q) block [16][17], diagonal of P [16], accumulated rows of Q [16][33]
        constexpr int kPQ = 0, kQQ = kJacB * LB, kDP = 2 * kJacB * LB, kAcc = kDP + kJacB, kBuf = kAcc + kJacB * LD;
        __shared__ double buf0[2 * kBuf];
        buf0[kPQ + i * LB + j] = b01;
        buf0[kQQ + i * LB + j] = b11;
        if (i == j) buf0[kDP + i] = b00;
        buf0[kAcc + i * LD + j] = y0; buf0[kAcc + i * LD + j + kJacB] = y1;
        __syncthreads();
#pragma unroll 2
        for (int t = 0; t < kJacB; ++t) {
            const double* R = buf0 + (t & 1) * kBuf;
            double* N = buf0 + ((t & 1) ^ 1) * kBuf;
            const int qi = (i + t) & 15, qj = (j + t) & 15;
            const double aa = R[kDP + i], bb = R[kQQ + qi * (LB + 1)], ab = R[kPQ + i * LB + qi];
            const double aj = R[kDP + j], bj = R[kQQ + qj * (LB + 1)], abj = R[kPQ + j * LB + qj];
            const double w01 = R[kPQ + i * LB + qj], w10 = R[kPQ + j * LB + qi], w11 = R[kQQ + qi * LB + qj];
            const double v0 = R[kAcc + qi * LD + j], v1 = R[kAcc + qi * LD + j + kJacB];
            double c, s, cj, sj;
            any |= jac_rotation(aa, bb, ab, &c, &s);
            jac_rotation(aj, bj, abj, &cj, &sj);
            smax = fmax(aa, bb) >= lead ? fmax(smax, fabs(s)) : smax;
            const double r00 = c * b00 - s * w10, r01 = c * w01 - s * w11, r10 = s * b00 + c * w10, r11 = s * w01 + c * w11;
            b00 = cj * r00 - sj * r01;
            N[kPQ + i * LB + qj] = sj * r00 + cj * r01;
            N[kQQ + qi * LB + qj] = sj * r10 + cj * r11;
            if (i == j) N[kDP + i] = b00;
            N[kAcc + qi * LD + j] = s * x0 + c * v0; N[kAcc + qi * LD + j + kJacB] = s * x1 + c * v1;
            x0 = c * x0 - s * v0; x1 = c * x1 - s * v1;
            __syncthreads();
        }
        // the accumulated rotations as one 32 x 32 matrix
        double* const Qo = &Qb[0][0];
        const double* R = buf0;  // (an even number of rounds)
        static_assert(kJacB % 2 == 0, "the last round wrote the first buffer");
        Qo[i * LD + j] = x0; Qo[i * LD + j + kJacB] = x1;
        Qo[(kJacB + i) * LD + j] = R[kAcc + i * LD + j]; Qo[(kJacB + i) * LD + j + kJacB] = R[kAcc + i * LD + j + kJacB];
        Qd = Qo;
    }
    if (j == 0) s_conv[i] = smax;
    if (any) s_any[1] = 1;
    __syncthreads();
    if (!s_any[1]) return;  // uniform
    if (tid == 0 && blockIdx.x == 0) {
        double m = 0.0;
        for (int k = 0; k < kJacB; ++k) m = fmax(m, s_conv[k]);
        conv_max(conv + blockIdx.y, m);
    }
    double qa[2][8];  // the accumulated rotations as MFMA operand: rows m 16 .. +16, contraction step s
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int s = 0; s < 8; ++s) qa[m][s] = Qd[(m * 16 + l16) * LD + 4 * s + kg];
    for (int c0 = wave * 16; c0 < slice_cols; c0 += 128) {
        if (c0 != wave * 16) load_tiles(c0);
        f64x4 acc[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                acc[u][m] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 8; ++s) acc[u][m] = mma_f64(qa[m][s], x[u][s], acc[u][m]);
            }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = c0 + 64 * u;
            if (c < slice_cols) {  // uniform
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    gp[(size_t)(4 * e) * D + c] = acc[u][0][e];
                    gq[(size_t)(4 * e) * D + c] = acc[u][1][e];
                }
            }
        }
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
    const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double li = norm[i];
    int c = 0;
    for (int j = tid; j < D; j += kCalThreads) {
        const double lj = norm[j];
        c += (lj > li || (lj == li && j < i)) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
    if (lane == 0) cnt[wave] = c;
    __syncthreads();
    int rank = 0;
#pragma unroll
    for (int w = 0; w < kCalThreads / kWave; ++w) rank += cnt[w];
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
