// Mixed-precision recent window (Sec. 5.1): the most recent w tokens, which the selection always keeps
// (Sec. 5.2), live in a second latent cache of higher rank, a ring of w rows with its own projectors.
// Attention over the union of both caches is one softmax (Eq. 5).  It runs as two passes of the sparse-attention
// kernels, the low-rank pass over the sinks and critical tokens and the window pass over the ring: both logits
// kernels leave their tile statistics in one array, so each value kernel weights its tokens with the maximum and
// normaliser of the whole selection, and one output projection adds the two passes' latent value sums through
// their projectors.
//
// The window's tokens follow from the sequence lengths, so its logits need no selection: in a decode step the window's logits
// pass and the selection of the critical tokens, which fills one compute unit per sequence, are one launch (window_select_*).
// Where the window's latent axis is split, the low-rank logits kernel adds the slices up on the side (SplitLogits).
#pragma once
#include "common.hpp"
#include "k_attend.hpp"
#include "k_logits.hpp"
#include "k_logits_small.hpp"
#include "k_topk.hpp"

namespace sals {

// The selection lists the recent tokens last.  With n = n_sel[b] and n_w = min(w, n):
//   idx_hi[b, :n_w] = idx[b, n - n_w : n] (zero beyond), n_hi[b] = n_w, n_lo[b] = n - n_w.
// grid (B), 256 threads.
__global__ __launch_bounds__(256) void window_split_kernel(const int32_t* __restrict__ idx,
                                                           const int32_t* __restrict__ n_sel, int k_tot, int w,
                                                           int32_t* __restrict__ idx_hi, int32_t* __restrict__ n_lo,
                                                           int32_t* __restrict__ n_hi)
{
    const int b = blockIdx.x;
    const int n = min(max(n_sel[b], 0), k_tot);
    const int nw = min(w, n);
    const int32_t* ib = idx + (size_t)b * k_tot;
    for (int i = threadIdx.x; i < w; i += 256) {
        const int v = ib[min(n - nw + i, k_tot - 1)];
        idx_hi[(size_t)b * w + i] = i < nw ? v : 0;
    }
    if (threadIdx.x == 0) { n_lo[b] = n - nw; n_hi[b] = nw; }
}

// Selection of a step's critical tokens (topk_window_kernel's arguments and results) by the launch's first `n_blocks` (B, rounded up
// to a whole number per die) workgroups; the others form the window's logits.
struct StepSelect {
    const float* scores;
    const int32_t* seq_len;
    int32_t* idx;
    int32_t* n_sel;
    int n_blocks, B, S_max, top_k, n_sink, n_recent;
    WindowLists wl;
};
constexpr int kWsMaxS = 8192;  // longer sequences keep the selection kernel of 1024 threads, whose own launch then takes longer than the window pass
// `lds`: at least sizeof(TopkShared) bytes.  The list is the selection kernel's, entry by entry (see topk_select_sequence).
template <int NTH> __device__ __forceinline__ void step_select(const StepSelect& a, unsigned char* lds)
{
    static_assert(kWsMaxS % (4 * NTH) == 0, "whole groups of four keys per thread");
    const int b = blockIdx.x;
    if (b >= a.B) return;
    TopkShared& sh = *reinterpret_cast<TopkShared*>(lds);
    write_window_lists(a.wl, a.seq_len, b, a.S_max, a.top_k + a.n_sink + a.n_recent, NTH);
    if (a.S_max <= kWsMaxS / 2)
        topk_select_sequence<kWsMaxS / 2 / (4 * NTH), NTH>(sh, a.scores, a.seq_len, a.idx, a.n_sel, b, a.S_max, a.top_k, a.n_sink,
                                                                 a.n_recent);
    else
        topk_select_sequence<kWsMaxS / (4 * NTH), NTH>(sh, a.scores, a.seq_len, a.idx, a.n_sel, b, a.S_max, a.top_k, a.n_sink,
                                                             a.n_recent);
}

// One sequence (few tiles): the window's logits in the 64-token form.
// Step of one sequence, 32 heads, 4096 tokens, w = 64, r_hi = 2048: the two launches took 5.1 + 7.4 us and the
// addition of the slices 2.4, this one 10.0: the step 44.4 -> 38.4.
template <typename T, int NST>
__global__ __launch_bounds__(kLsThreads) void window_select_small_kernel(
    StepSelect sel, const T* __restrict__ UkP, int B, int H_kv, int n_parts, int heads_fastest, int ksplit, int w, int r, int H,
    const T* __restrict__ Kw, const T* __restrict__ q, const int32_t* __restrict__ q_pos, const float2* __restrict__ rope, InvFreq inv,
    float* __restrict__ logits, float2* __restrict__ stats, int S_max, int lk, int style, float scale, float* __restrict__ plogits,
    int stats_stride)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    if ((int)blockIdx.x < sel.n_blocks) { step_select<kLsThreads>(sel, lds); return; }  // uniform
    logits_small_tile<T, NST, false, true, false>((int)blockIdx.x - sel.n_blocks, nullptr, nullptr, UkP, B, H_kv, n_parts, heads_fastest, ksplit,
                                           w, r, H, Kw, q, q_pos, rope, inv, logits, stats, S_max, lk, style, scale, w, plogits,
                                           stats_stride, FusedSelect{},
                                           WindowByLength{sel.seq_len, sel.top_k + sel.n_sink + sel.n_recent}, SplitLogits{});
}

// A batch: tiles of one head and two sequences' windows, or (WIDE) of two heads and four sequences'.
// Bound by the operands a compute unit draws, which the wide tiles halve per product.  Step of 16 sequences, 32 heads, 4096 tokens, w =
// 64, r_hi = 2048: the two launches took 6.7 + 23.0 us (the window's in two slices, 4.7 more to add them up), this one 30 in tiles of a
// head (one slice) and 23 in wide ones (three slices, which the low-rank logits kernel adds up on the side): 109.3 -> 104.2 us a step.
template <typename T, int GB, int GFIX, bool WIDE>
__global__ __launch_bounds__(WIDE ? 512 : 256, WIDE ? 2 : 1) void window_select_kernel(
    StepSelect sel, const T* __restrict__ Kw, const T* __restrict__ UkP, const T* __restrict__ q, const int32_t* __restrict__ q_pos,
    const float2* __restrict__ rope, InvFreq inv, float* __restrict__ logits, float2* __restrict__ stats, int B, int S_max, int r, int H,
    int H_kv, int w, int lk, int style, float scale, int stats_stride, float* __restrict__ plogits, int ksplit)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    if ((int)blockIdx.x < sel.n_blocks) { step_select<WIDE ? 512 : 256>(sel, lds); return; }  // uniform
    logits_tile<T, WIDE ? 2 : 1, 4, WIDE ? 2 : 1, GB, GFIX, true, true, false, false>(
        (int)blockIdx.x - sel.n_blocks, Kw, UkP, nullptr, nullptr, q, q_pos, rope, inv, logits, stats, B, S_max, r, H, H_kv, w, lk, 1, 0, style,
        scale, w, stats_stride, plogits, ksplit, WindowByLength{sel.seq_len, sel.top_k + sel.n_sink + sel.n_recent}, SplitLogits{},
        TopkResolve{});
}

}  // namespace sals
