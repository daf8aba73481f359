// Selective reconstruction, RoPE and sparse attention (Sec. 4.4, Eq. 5;
// Algorithm 1, reconstruction to output steps).
//
//   attend_logits  K_C = K~_C U_k^T on the matrix cores; RoPE and q.K in the epilogue, so the
//                  reconstructed keys never leave registers.  Also rotates the query in its
//                  prologue and leaves, per (head, token tile), the softmax maximum and
//                  normaliser of the tile.
//   attend_pv      combines the tile statistics into the softmax of Eq. 5 and forms
//                  T[h,:] = sum_j p_hj V~_C[j,:]                 (latent-space value sum)
//   attend_out     y[h] = T[h,:] U_v[g(h) block]^T               (one pass over U_v)
//
// The value product uses  p (V~_C U_v^T) = (p V~_C) U_v^T : the same sum in another
// order, which avoids reconstructing V_C.
//
// Head dims are handled in "pair order": slot p < 64 is the first element of RoPE pair
// p, slot 64+p its partner, for either pairing style; the packed U_k panel (see
// pack_weights_kernel) already has its rows in that order, so both elements of a pair land
// in the same lane of the MFMA result.
//
// RoPE angles.  The angle of token position t and pair p is t * theta^(-2p/d), evaluated in
// fp64.  The query's cos/sin are computed in the logits kernel; those of the cached tokens
// come from a table over the positions 0 .. S_max that is filled once per context.
#pragma once
#include "common.hpp"

namespace sals {

__device__ __forceinline__ int pair_first(int p, int style) { return style ? 2 * p : p; }
__device__ __forceinline__ int pair_second(int p, int style) { return style ? 2 * p + 1 : p + kPairs; }
__device__ __forceinline__ int slot_to_dim(int slot, int style)
{
    return slot < kPairs ? pair_first(slot, style) : pair_second(slot - kPairs, style);
}

struct InvFreq { double f[kPairs]; };  // theta^(-2p/d), computed on the host in fp64

// cos/sin of every (position, pair): tab[t][p] = (cos, sin)(t * f_p)
// (and zero in `count`, unless null, for what counts arrivals)
__global__ __launch_bounds__(256) void rope_table_kernel(float2* __restrict__ tab, InvFreq inv, int rows, uint32_t* count)
{
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e == 0 && count) *count = 0u;
    if (e >= (size_t)rows * kPairs) return;
    double sn, c;
    sincos((double)(e / kPairs) * inv.f[e % kPairs], &sn, &c);
    tab[e] = make_float2((float)c, (float)sn);
}

constexpr int kMaxGroup = 8;                 // query heads per KV head

// The logits kernels exist in many instantiations, and a whole step promises the bits that the staged calls leave, whichever of
// them either runs: which of two products is rounded by itself and which is fused with the addition is written out below, not left
// to the compiler (which had chosen otherwise from one instantiation to another: 1.4e-4 of a bf16 output, with the same accuracy).
__device__ __forceinline__ void rotate_key(float y1, float y2, float c, float s, float& k1, float& k2)
{
    k1 = fmaf(y1, c, -(y2 * s));
    k2 = fmaf(y1, s, y2 * c);
}
__device__ __forceinline__ void rotate_query(float x1, float x2, float2 cs, float scale, float& q1, float& q2)
{
    q1 = fmaf(x1, cs.x, -(x2 * cs.y)) * scale;
    q2 = fmaf(x2, cs.x, x1 * cs.y) * scale;
}
// four pairs' share of q . k
__device__ __forceinline__ float dot_pairs(const f32x4& q1, const f32x4& q2, const float (&k1)[4], const float (&k2)[4])
{
    float t = fmaf(q1.x, k1[0], q1.y * k1[1]);
    t = fmaf(q1.z, k1[2], t);
    t = fmaf(q1.w, k1[3], t);
    t = fmaf(q2.x, k2[0], t);
    t = fmaf(q2.y, k2[1], t);
    t = fmaf(q2.z, k2[2], t);
    return fmaf(q2.w, k2[3], t);
}

// softmax statistics of a set of logits: maximum m and sum of exp(x - m)
__device__ __forceinline__ float2 stat_merge(float2 a, float2 b)
{
    const float m = fmaxf(a.x, b.x);
    if (m == -INFINITY) return make_float2(-INFINITY, 0.f);
    return make_float2(m, fmaf(a.y, __expf(a.x - m), b.y * __expf(b.x - m)));
}

// Logits whose latent axis was split over workgroups (64-token tiles): a slice's workgroup left its partial logits; the sum in
// slice order and the tile's softmax statistics are one wave's job per (token tile, head).
constexpr int kLsTok = 64;       // tokens per tile
constexpr int kLsMaxSplit = 8;   // slices at most
struct SplitLogits {
    const float* plogits;    // [ksplit][rows][lk]
    const int32_t* n_sel;    // [B] tokens of a sequence
    float* logits;           // [rows][lk]
    float2* stats;           // [rows][stats_stride], this pass's tiles from record 0 on
    int ksplit, n_parts, rows, H, lk, stats_stride;   // rows = B * H
};
// The job in two halves, so that a kernel that does it on the side requests what it needs early and uses it late.
struct SplitLogitsJob {
    float v[kLsMaxSplit];
    int n, slot, row, part;
    __device__ __forceinline__ void request(const SplitLogits& f, int row_, int part_)
    {
        row = row_; part = part_;
        slot = part * kLsTok + lane_id();
#pragma unroll
        for (int u = 0; u < kLsMaxSplit; ++u)  // all slices requested together, from clamped addresses
            v[u] = f.plogits[((size_t)min(u, f.ksplit - 1) * f.rows + row) * f.lk + min(slot, f.lk - 1)];
        n = f.n_sel[row / f.H];
    }
    __device__ __forceinline__ void finish(const SplitLogits& f) const
    {
        float d = 0.f;
#pragma unroll
        for (int u = 0; u < kLsMaxSplit; ++u) d += u < f.ksplit ? v[u] : 0.f;
        const bool valid = slot < n;
        if (slot < f.lk) f.logits[(size_t)row * f.lk + slot] = valid ? d : -INFINITY;
        const float mx = wave_max(valid ? d : -INFINITY);
        const float se = wave_sum(valid ? __expf(d - mx) : 0.f);
        if (lane_id() == 0) f.stats[(size_t)row * f.stats_stride + part] = make_float2(mx, se);
    }
};

// The recent window's tokens by the sequence length alone: the last min(w, min(length, k_tot)) tokens of the sequence, w the
// window's own selection size (see write_window_lists, which writes the same list).
struct WindowByLength { const int32_t* seq_len; int k_tot; };

template <typename T> struct mma_op;
template <> struct mma_op<bf16_t> {  // one v_mfma_f32_32x32x16_bf16 per 16-byte fragment pair
    static __device__ __forceinline__ void run(const u32x4& a, const u32x4& b, f32x16& c)
    {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                    __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct mma_op<float> {   // four v_mfma_f32_32x32x2_f32 per 16-byte fragment pair
    static __device__ __forceinline__ void run(const u32x4& a, const u32x4& b, f32x16& c)
    {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
    }
};

}  // namespace sals
