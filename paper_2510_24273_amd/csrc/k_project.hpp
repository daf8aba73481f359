// Latent projection  x~ = U^T x  (Sec. 4.3; Algorithm 1, projection step) and the one-time
// repacking of the projectors.
//
// The projection reads the TRANSPOSED projector U^T [r x D] (made once by pack_weights),
// so each output coordinate is a dot product along a contiguous row: a workgroup owns 16
// latent coordinates and one slice of the D axis (the slices' partial sums are added by
// the score kernel, in slice order), its 4 waves split the slice, and every wave keeps all
// of its 16-byte row pieces in flight at once.  The products run on 16x16 MFMA tiles whose
// columns are the (sequence, query head of the KV group) pairs, so a whole batch costs
// one pass over U^T; the heads of a group are added in fp32 afterwards, which equals
// projecting their sum.  Single pass, fixed summation order, bit-reproducible.
#pragma once
#include "common.hpp"

namespace sals {

typedef float f32x4v __attribute__((ext_vector_type(4)));

template <typename T> struct mma16_op;
template <> struct mma16_op<bf16_t> {  // v_mfma_f32_16x16x32_bf16
    static __device__ __forceinline__ void run(const u32x4& a, const u32x4& b, f32x4v& c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                    c, 0, 0, 0);
    }
};
template <> struct mma16_op<float> {   // four v_mfma_f32_16x16x4_f32
    static __device__ __forceinline__ void run(const u32x4& a, const u32x4& b, f32x4v& c)
    {
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    }
};

constexpr int kScoreMaxParts = 8;   // slices of the D axis the projection may split into
constexpr int kProjWaves = 4;       // waves of a query projection workgroup
constexpr int kProjThreads = 64 * kProjWaves;
constexpr int kAppendWaves = 8;     // ... and at most of an append workgroup, which owns the whole D axis
constexpr int kProjMaxCols = 128;  // B * (H_q / H_kv) handled per call
constexpr int kProjBatch = 8;      // row pieces a wave of a query projection keeps in flight per round

struct ProjArgs {  // (what the first loads need comes first: those 14 words arrive preloaded in scalar registers)
    const void* UT[2];   // transposed projectors [r, D]
    const void* X[2];    // QUERY: q [B,H,d] (X[0]); else new key / value [B,D]
    int D, np, B, H, H_kv, r;
    int d, S_max, nproj;
    int ring;            // append: > 0 = the cache is a ring of this many rows, token t in row t mod ring
    void* cache[2];      // append: [B,S_max,r], or [B,ring,r] when ring > 0
    float* out_f32;      // QUERY: partial q~ [np,B,r], one slice of the D axis each; append with np > 1: [nproj,np,B,r]
    const int32_t* seq_len;  // append: [B] row to write
    uint32_t* arrived;       // append: not null = the last of its n_wg workgroups to arrive here advances the lengths
    uint32_t n_wg;
};

// One wave, lane l with the lengths of sequences l and 64 + l and (lane 0) the workgroup's arrival: the last workgroup advances them.
__device__ __forceinline__ void append_advance(const ProjArgs& a, uint32_t order, int32_t len0, int32_t len1)
{
    if ((uint32_t)wave_uniform((int)order) != a.n_wg - 1) return;
    int32_t* const seq_len = const_cast<int32_t*>(a.seq_len);
    const int lane = lane_id();
    if (lane < a.B && len0 < a.S_max) seq_len[lane] = len0 + 1;
    if (lane + kWave < a.B && len1 < a.S_max) seq_len[lane + kWave] = len1 + 1;
}

// workgroup of NW waves, HB column blocks in a round, of which a wave has NBATCH row pieces of LB at a time in flight; i0: first latent
// coordinate
//
// Code size counts here as in every kernel of a decode step: the instruction caches (64 KB for two CUs) keep code from one
// launch to the next (measured: a launch's first pass through 32 KB is as fast as its second), so a step whose kernels fit
// together runs from them, and one that exceeds them fetches lines from L2 or, behind large caches, from memory (20-30 ns a line) on
// every pass: the same kernels of a small step linked in nine orders took 27.7 to 29.1 us.  So the column blocks are a loop and
// not unrolled over registers of their own (a slice of one round still keeps U^T's pieces for all of them), 12.0 -> 2.4 KB for
// up to 16 columns.  With the value sum's shorter code, whole steps: 1 x (512 of 4096) 28.0 -> 27.4 us, 12 ragged sequences
// of 8 KV heads 65.1 -> 62.2 (the projection 5.9 -> 4.8), 32 x 2048 the same way 84 -> 79.5, 64 x 2048 of 32 KV heads 263 -> 255.
template <typename T, bool QUERY, int NW, int NBATCH, int HB, int LB>
__device__ __forceinline__ void project_block(const ProjArgs& a, int i0, int slice, int proj)
{
    constexpr int VEC = elem<T>::vec;
    constexpr int KS = 4 * VEC;  // elements of the D axis per MFMA step
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int G = QUERY ? idiv(a.H, a.H_kv) : 1;
    const int ncols = a.B * G, n_nblk = (ncols + 15) >> 4;
    const int nks = idiv((unsigned)a.D / KS, a.np);  // steps of this workgroup's slice
    const int ks_first = slice * nks;
    const T* UT = static_cast<const T*>(a.UT[proj]);
    const T* X = static_cast<const T*>(a.X[proj]);
    const T* arow = UT + (size_t)(i0 + l16) * a.D + kg * VEC;

    __shared__ __attribute__((aligned(16))) float red[HB][NW][64][4];
    __shared__ float colsum[kProjMaxCols][16];
    // Append: the first wave requests all lengths ahead of its other loads, for the workgroup's stores, and says that it has them.
    __shared__ int32_t length[QUERY ? 1 : kProjMaxCols];
    static_assert(kProjMaxCols == 2 * kWave, "two lengths a lane");
    int32_t len0 = 0, len1 = 0;
    uint32_t order = 0;
    if (!QUERY && wave == 0) { len0 = a.seq_len[min(lane, a.B - 1)]; len1 = a.seq_len[min(lane + kWave, a.B - 1)]; }

    u32x4 af[NBATCH];
    for (int nb0 = 0; nb0 < n_nblk; nb0 += HB) {
        const T* xrow[HB];
#pragma unroll
        for (int h = 0; h < HB; ++h) {  // (columns past the last one repeat it)
            const int n = min((nb0 + h) * 16 + l16, ncols - 1), b = QUERY ? idiv(n, G) : n;
            xrow[h] = X + (QUERY ? ((size_t)b * a.H + n - b * G) * kHeadDim : (size_t)n * a.D) + kg * VEC;
        }
        f32x4v acc[HB];
#pragma unroll
        for (int h = 0; h < HB; ++h) acc[h] = f32x4v{0.f, 0.f, 0.f, 0.f};

        // this wave's steps: wave, wave+NW, ... ; NBATCH steps of loads per round, those of LB column blocks requested
        // together, ahead of their products: they cost one memory round trip.  Branches are wave-uniform (a step that is not
        // there costs no load: clamped instead, 24 columns of 64 steps took 12.4 us where 8.1 do).
        for (int ks0 = wave; ks0 < nks; ks0 += NW * NBATCH) {
            if (nb0 == 0 || nks > NW * NBATCH) {
#pragma unroll
                for (int u = 0; u < NBATCH; ++u)
                    if (ks0 + u * NW < nks) af[u] = ld16(arow + (size_t)(ks_first + ks0 + u * NW) * KS);
            }
#pragma unroll
            for (int h0 = 0; h0 < HB; h0 += LB) {
                if (nb0 + h0 >= n_nblk) continue;
                u32x4 bf[LB][NBATCH];
#pragma unroll
                for (int h = 0; h < LB; ++h) {
                    if (nb0 + h0 + h < n_nblk) {
#pragma unroll
                        for (int u = 0; u < NBATCH; ++u)
                            if (ks0 + u * NW < nks) {
                                const unsigned c = (unsigned)(ks_first + ks0 + u * NW) * KS;  // (a step lies within one head)
                                bf[h][u] = ld16(xrow[h0 + h] + (QUERY ? c / kHeadDim * G * kHeadDim + c % kHeadDim : c));
                            }
                    }
                }
                asm volatile("" ::: "memory");  // (keeps the loads above from sinking towards their products)
                if (!QUERY && wave == 0 && nb0 + h0 + ks0 == 0) {  // uniform
                    length[lane] = len0; length[lane + kWave] = len1;
                    asm volatile("" ::"v"(len0), "v"(len1) : "memory");
                    if (a.arrived && lane == 0) order = arrive(a.arrived, a.n_wg);
                }
#pragma unroll
                for (int h = 0; h < LB; ++h) {
                    if (nb0 + h0 + h < n_nblk) {
#pragma unroll
                        for (int u = 0; u < NBATCH; ++u)
                            if (ks0 + u * NW < nks) mma16_op<T>::run(af[u], bf[h][u], acc[h0 + h]);
                    }
                }
            }
        }

        // fold the waves' sums in wave order; acc[h][v] is (coordinate 4*kg+v, column (nb0+h)*16+l16)
        if (nb0 > 0) __syncthreads();
#pragma unroll
        for (int h = 0; h < HB; ++h) *reinterpret_cast<f32x4v*>(red[h][wave][lane]) = acc[h];
        __syncthreads();
        if (tid < 256) {
            const int col = tid & 15, rr = tid >> 4;
            const int src_lane = (rr >> 2) * 16 + col, v = rr & 3;
#pragma unroll
            for (int h = 0; h < HB; ++h) {
                float s = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) s += red[h][w][src_lane][v];
                if (nb0 + h < n_nblk) colsum[(nb0 + h) * 16 + col][rr] = s;
            }
        }
    }
    __syncthreads();
    // add the heads of each group and write
    for (int t = tid; t < a.B * 16; t += 64 * NW) {
        int b = t >> 4, rr = t & 15;
        float s = 0.f;
        for (int m = 0; m < G; ++m) s += colsum[b * G + m][rr];
        if (QUERY || a.np > 1) {
            a.out_f32[((size_t)(proj * a.np + slice) * a.B + b) * a.r + i0 + rr] = s;
        } else {
            const int t_new = length[b];
            const int rows = a.ring > 0 ? a.ring : a.S_max;
            if (t_new >= 0 && t_new < a.S_max) {
                const int row = a.ring > 0 ? (unsigned)t_new % (unsigned)a.ring : t_new;
                elem<T>::store(static_cast<T*>(a.cache[proj]) + ((size_t)b * rows + row) * a.r + i0 + rr, s);
            }
        }
    }
    if (!QUERY && a.arrived && wave == 0) append_advance(a, order, len0, len1);
}

// HB: as many column blocks as there are (1, 2, 4 or 8), so that all their operands arrive in one round trip (1 x 48 columns, r = 640,
// D = 1024: 5.6 us unrolled over all blocks, 7.6 in rounds of two, 5.4 in one of four; 128 columns, whole steps of 32 sequences of 8 KV
// heads, r = 512, behind a copy that empties the caches: two rounds of four 65.0, eight at once 63.4, eight in pairs 64.2)
template <typename T, int HB>
__global__ __launch_bounds__(kProjThreads) void project_kernel(ProjArgs a)
{
    project_block<T, true, kProjWaves, kProjBatch, HB, HB>(a, blockIdx.x * 16, blockIdx.y, blockIdx.z);
}

// Append in slices of the D axis: adds up the slices' partial sums (in slice order) into the new rows and advances the lengths.
// One workgroup per sequence, which thus reads its length before it advances it.
template <typename T>
__global__ __launch_bounds__(256) void append_finish_kernel(ProjArgs a)
{
    const int b = blockIdx.x, t_new = a.seq_len[b];
    if (t_new >= a.S_max) return;  // uniform
    for (int e = threadIdx.x; e < a.nproj * a.r / 4; e += 256) {
        const int proj = e / (a.r / 4), i = (e - proj * (a.r / 4)) * 4;
        f32x4 x[kScoreMaxParts];
#pragma unroll
        for (int p = 0; p < kScoreMaxParts; ++p)
            x[p] = *reinterpret_cast<const f32x4*>(a.out_f32 + ((size_t)(proj * a.np + min(p, a.np - 1)) * a.B + b) * a.r + i);
        f32x4 s = x[0];
#pragma unroll
        for (int p = 1; p < kScoreMaxParts; ++p) {
            const bool use = p < a.np;
            s.x += use ? x[p].x : 0.f; s.y += use ? x[p].y : 0.f; s.z += use ? x[p].z : 0.f; s.w += use ? x[p].w : 0.f;
        }
        if (t_new >= 0) {
            T* dst = static_cast<T*>(a.cache[proj]) + ((size_t)b * a.S_max + t_new) * a.r + i;
            elem<T>::store(dst, s.x); elem<T>::store(dst + 1, s.y); elem<T>::store(dst + 2, s.z); elem<T>::store(dst + 3, s.w);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) const_cast<int32_t*>(a.seq_len)[b] = t_new + 1;
}

// after an append of a context without a count of arrivals (see arrival_count): advance the sequence lengths
__global__ void bump_seq_len_kernel(int32_t* __restrict__ seq_len, int B, int S_max)
{
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B && seq_len[b] < S_max) seq_len[b] += 1;
}

// ---------------------------------------------------------------------------------
// one-time weight repacking (model-load time; not on the decode path)
// ---------------------------------------------------------------------------------
// section 0: UkT [r, D]      section 1: UvT [r, D]
// section 2: Uk in reconstruction order: [H_kv][r/KE][128 slots][KE] (KE = 64 bytes of the latent
//            axis) with the head dims in RoPE pair order (slot p < 64: first element of pair p; 64+p: its partner)
// section 3: Uv [D, r] unchanged
template <typename T>
__global__ __launch_bounds__(256) void pack_weights_kernel(const T* __restrict__ Uk, const T* __restrict__ Uv,
                                                           T* __restrict__ packed, size_t section_elems,
                                                           int D, int r, int style)
{
    constexpr int KE = 64 / (int)sizeof(T);
    const int sec = blockIdx.y;
    T* dst = packed + (size_t)sec * section_elems;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < section_elems; e += (size_t)gridDim.x * 256) {
        T v;
        if (sec == 0 || sec == 1) {
            size_t i = e / D, c = e - i * D;
            v = (sec == 0 ? Uk : Uv)[c * r + i];
        } else if (sec == 2) {
            size_t per_head = (size_t)kHeadDim * r;
            size_t g = e / per_head, rem = e - g * per_head;
            size_t kc = rem / ((size_t)kHeadDim * KE), rem2 = rem - kc * kHeadDim * KE;
            int slot = (int)(rem2 / KE), ke = (int)(rem2 - (size_t)slot * KE);
            int dim = slot < kPairs ? (style ? 2 * slot : slot) : (style ? 2 * (slot - kPairs) + 1 : slot);
            v = Uk[(g * kHeadDim + dim) * r + kc * KE + ke];
        } else {
            v = Uv[e];
        }
        dst[e] = v;
    }
}

}  // namespace sals
