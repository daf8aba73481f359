// Critical-token selection for long sequences (Algorithm 1, TopK step; Sec. 5.2 composition),
// spread over many workgroups.
//
// One workgroup walks a compute unit's worth of instructions per key and pass, so beyond a few
// ten thousand scores a single workgroup per sequence is the bottleneck.  Here a sequence is cut
// into chunks of 8192 scores, one workgroup each, and the selection runs as a chain of small
// kernels that exchange a few kilobytes:
//   range    per chunk: minimum and maximum candidate key
//   hist     per chunk: histogram over 2048 linear bins of the sequence's [min, max], 16-bit counts from the top bin down
//   place    per chunk: the bin holding the top_k-th score, how many of its members are selected and
//            where the chunk's output starts (every workgroup of the sequence derives the same
//            numbers: a thread adds up two bins over the chunks, all its loads in flight together, and one block scan
//            of the totals and of the earlier chunks' counts settles everything); then the indices of the scores in
//            higher bins go to their final positions (chunk order, then the order of a chunk's threads) and the
//            members of the threshold bin to a candidate list
//   finish   per sequence: ranks the candidates (ties towards the smaller index), writes the
//            selected ones in token order, the sink / recent entries and n_sel
// The result is the same set as topk_kernel's, a deterministic function of the scores; only
// the order inside the top_k block differs (bins above the threshold first).  Cases this chain
// does not cover (a cache no longer than the selection, a degenerate or non-finite score range,
// more than 512 members in the threshold bin) raise a flag, and the finish kernel's workgroup
// then selects that sequence from scratch the way topk_kernel does.
// A decode step whose logits kernel has tiles of one sequence needs no finish launch (3.9 us with the gap before it): the first
// chunk's place workgroup does all but the ranking (topk_place_kernel<true>), and the logits workgroups whose tiles reach the
// entries to be ranked do that for themselves, beside the loads of their first panels (TopkResolve; 0.5 - 1 us of theirs).
#pragma once
#include "common.hpp"
#include "k_topk.hpp"

namespace sals {

constexpr int kTmChunk = 8192;            // scores per workgroup
constexpr int kTmF4 = kTmChunk / (4 * kTopkThreads);  // float4 groups per thread: 2
constexpr int kTmBins = 2048;
constexpr int kTmMaxChunks = 128;         // S_max <= 2^20
constexpr int kTmCand = 512;              // candidates the finish kernel ranks
constexpr int kTmRow = kTmBins / 2;       // 32-bit words of a chunk's histogram: two 16-bit counts each (a chunk has 8192 scores)
static_assert(kTmChunk < 65536, "a chunk's counts fit in 16 bits");

struct TopkMeta {        // per sequence, written by the place kernel
    uint32_t fallback;   // 1: topk_kernel must redo the sequence
    uint32_t t_slot;     // threshold bin (slot 0 = top of the range)
    uint32_t kk;         // members of the threshold bin that are selected
    uint32_t n_above;    // scores in higher bins
    uint32_t members;    // scores in the threshold bin
    float flo, scale;    // slot = kTmBins-1 - clamp(int((x - flo) * scale))
    uint32_t pad;
};

// workspace of the chain, per sequence (the kernels take its members as arguments, those that their first loads need and the
// sizes first: these words arrive preloaded in scalar registers)
struct TopkMultiWs {
    const uint2* range;  // [B][n_range] (min key, max key) pairs that cover the sequence's candidates: `part`, or the
    int n_range;         //   pairs the score kernel left per workgroup (then over all scores below the length)
    uint2* part;         // [B][n_chunk] (min key, max key) of the chunk's candidates
    uint32_t* hist;      // [B][n_chunk][kTmRow]: the chunk's candidates in slots 2w (low half) and 2w + 1 (slot 0 = top bin)
    TopkMeta* meta;      // [B]
    uint2* cand;         // [B][kTmCand] (key, token index)
};

// keys of this thread's 8 scores of chunk `chunk`: tokens chunk*8192 + 4*(c*1024 + tid) + e;
// non-candidates (sink / recent tokens, positions past the sequence) carry key 0
__device__ __forceinline__ void tm_load_keys(const float* __restrict__ s, int S_max, int chunk, int lo, int hi,
                                            uint32_t* keys)
{
    const int tid = threadIdx.x;
    float f[4 * kTmF4];
    if ((S_max & 3) == 0 && S_max >= 4 && (reinterpret_cast<uintptr_t>(s) & 15) == 0) {  // uniform
        // both groups requested at once from clamped addresses (no load inside a branch)
        f32x4 v[kTmF4];
#pragma unroll
        for (int c = 0; c < kTmF4; ++c)
            v[c] = *reinterpret_cast<const f32x4*>(s + min(chunk * kTmChunk + ((c * kTopkThreads + tid) << 2), S_max - 4));
#pragma unroll
        for (int c = 0; c < kTmF4; ++c) { f[4 * c] = v[c].x; f[4 * c + 1] = v[c].y; f[4 * c + 2] = v[c].z; f[4 * c + 3] = v[c].w; }
    } else {
#pragma unroll
        for (int c = 0; c < kTmF4; ++c) {
            const int j = chunk * kTmChunk + ((c * kTopkThreads + tid) << 2);
#pragma unroll
            for (int e = 0; e < 4; ++e) f[4 * c + e] = 0.f;
            if (j + 3 < S_max && ((reinterpret_cast<uintptr_t>(s + j) & 15) == 0)) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(s + j);
                f[4 * c] = v.x; f[4 * c + 1] = v.y; f[4 * c + 2] = v.z; f[4 * c + 3] = v.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (j + e < S_max) f[4 * c + e] = s[j + e];
            }
        }
    }
    // (a group past the row read the row's last group: its tokens are at or past S_max >= hi, so their keys are 0)
#pragma unroll
    for (int c = 0; c < kTmF4; ++c) {
        const int j = chunk * kTmChunk + ((c * kTopkThreads + tid) << 2);
#pragma unroll
        for (int e = 0; e < 4; ++e) keys[4 * c + e] = (j + e >= lo && j + e < hi) ? score_key(f[4 * c + e]) : 0u;
    }
}
__device__ __forceinline__ int tm_token(int chunk, int i)
{
    return chunk * kTmChunk + ((((i >> 2) * kTopkThreads) + threadIdx.x) << 2) + (i & 3);
}

// the sequence's linear map from the (min key, max key) pairs of its parts (the chunks of the range kernel, or the
// workgroups of the score kernel): every workgroup derives the same numbers.  All threads of the workgroup must call
// (one barrier); `red` is LDS scratch of 2 * kTopkWaves words.
__device__ __forceinline__ bool tm_range(const uint2* __restrict__ part, int n_part, uint32_t* red, float* flo, float* scale)
{
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    for (int c0 = 0; c0 < n_part; c0 += 2 * kTopkThreads) {  // two loads per thread and trip, from clamped part numbers
        const uint2 a = part[min(c0 + tid, n_part - 1)], b = part[min(c0 + kTopkThreads + tid, n_part - 1)];
        kmin = min(kmin, min(a.x, b.x));
        kmax = max(kmax, max(a.y, b.y));
    }
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) { red[wave] = kmin; red[kTopkWaves + wave] = kmax; }
    __syncthreads();
    static_assert(kTopkWaves == 16, "one DPP row of wave results");
    kmin = wave_min_u32(red[lane & 15]);
    kmax = wave_max_u32(red[kTopkWaves + (lane & 15)]);
    if (kmax == 0u) return false;  // no candidate at all
    const float a = key_to_score(kmin), span = key_to_score(kmax) - a;
    const float sc = (span > 0.f && span < 3.0e38f) ? (float)kTmBins / span : 0.f;
    *flo = a;
    *scale = sc;
    return sc > 0.f && sc < 3.0e38f && fabsf(a * sc) < 3.0e38f;
}
__device__ __forceinline__ int tm_slot(uint32_t key, float flo, float scale)
{
    const int bin = (int)((key_to_score(key) - flo) * scale);
    return kTmBins - 1 - min(max(bin, 0), kTmBins - 1);
}

__global__ __launch_bounds__(kTopkThreads) void topk_range_kernel(const float* __restrict__ scores,
                                                                  const int32_t* __restrict__ seq_len, int S_max, int n_chunk,
                                                                  int n_sink, int n_recent, uint2* __restrict__ part)
{
    __shared__ uint32_t s_min[kTopkWaves], s_max[kTopkWaves];
    const int chunk = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int S = min(ld_uniform_i32(seq_len + b), S_max);  // (vector memory path: in flight with the scores)
    uint32_t keys[4 * kTmF4];
    tm_load_keys(scores + (size_t)b * S_max, S_max, chunk, n_sink, S - n_recent, keys);
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int i = 0; i < 4 * kTmF4; ++i)
        if (keys[i] != 0u) { kmin = min(kmin, keys[i]); kmax = max(kmax, keys[i]); }
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if ((tid & 63) == 0) { s_min[tid >> 6] = kmin; s_max[tid >> 6] = kmax; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 0; w < kTopkWaves; ++w) { kmin = min(kmin, s_min[w]); kmax = max(kmax, s_max[w]); }
        part[(size_t)b * n_chunk + chunk] = make_uint2(kmin, kmax);
    }
}

__global__ __launch_bounds__(kTopkThreads) void topk_hist_kernel(const float* __restrict__ scores,
                                                                 const int32_t* __restrict__ seq_len,
                                                                 const uint2* __restrict__ range, int n_range, int S_max, int n_chunk,
                                                                 int n_sink, int n_recent, uint32_t* __restrict__ hist_out)
{
    __shared__ TopkShared sh;  // (its histogram array and scan buffers)
    static_assert(kTmBins == 2 * kTopkThreads && kTmBins <= kTopkBins, "two bins per thread");
    uint32_t* hist = sh.hist;
    const int chunk = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int S = min(ld_uniform_i32(seq_len + b), S_max);  // (vector memory path: in flight with the scores)
    uint32_t keys[4 * kTmF4];
    tm_load_keys(scores + (size_t)b * S_max, S_max, chunk, n_sink, S - n_recent, keys);
    for (int t = tid; t < kTmBins; t += kTopkThreads) hist[t] = 0u;
    float flo, scale;
    const bool ok = tm_range(range + (size_t)b * n_range, n_range, sh.cand, &flo, &scale);  // (barrier inside)
    if (ok) {
#pragma unroll
        for (int i = 0; i < 4 * kTmF4; ++i)
            if (keys[i] != 0u) atomicAdd(&hist[tm_slot(keys[i], flo, scale)], 1u);
    }
    __syncthreads();
    const uint2 c = *reinterpret_cast<const uint2*>(&hist[2 * tid]);
    hist_out[((size_t)b * n_chunk + chunk) * kTmRow + tid] = c.x | (c.y << 16);
}

// The sequence-level decisions, taken identically by every workgroup of the sequence from the chunks' histograms: threshold
// bin, selected members, and the first output position / candidate slot of chunk `chunk`.
// Returns the meta record (fallback set if the chain does not apply).
struct TmResolveLds {
    uint32_t red[2 * kTopkWaves];
    uint32_t found, t_slot, n_above, members, base_above, base_cand;
};
__device__ __forceinline__ TopkMeta tm_resolve(TmResolveLds& L, TopkShared& sh, int& phase, const uint2* __restrict__ range,
                                               int n_range, const uint32_t* __restrict__ hist, int b, int chunk,
                                               int S, int n_chunk, int top_k, int n_sink, int n_recent, uint32_t* base_above,
                                               uint32_t* base_cand)
{
    const int tid = threadIdx.x;
    TopkMeta m{};
    const uint32_t* h = hist + (size_t)b * n_chunk * kTmRow + tid;
    // this thread's two bins over all chunks and over the chunks before this one, 16 loads in flight per trip
    uint32_t tot[2] = {0u, 0u}, bef[2] = {0u, 0u};
    if (tid == 0) L.found = 0u;
    uint32_t v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = h[(size_t)min(u, n_chunk - 1) * kTmRow];
    const bool ok = tm_range(range + (size_t)b * n_range, n_range, L.red, &m.flo, &m.scale) &&  // (barrier inside)
                    S > top_k + n_sink + n_recent && top_k > 0;
    if (!ok) {  // uniform
        m.fallback = 1u;
        return m;
    }
    for (int c0 = 0;;) {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int c = c0 + u;
            const uint32_t x = c < n_chunk ? v[u] : 0u, y = c < chunk ? x : 0u;
            tot[0] += x & 0xffffu; tot[1] += x >> 16;
            bef[0] += y & 0xffffu; bef[1] += y >> 16;
        }
        c0 += 16;
        if (c0 >= n_chunk) break;
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = h[(size_t)min(c0 + u, n_chunk - 1) * kTmRow];
    }
    uint32_t above = tot[0] + tot[1], before = bef[0] + bef[1], sum_a, sum_b;
    block_excl_scan2(above, before, sh, phase, &sum_a, &sum_b);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (above < (uint32_t)top_k && (uint32_t)top_k <= above + tot[i]) {  // (one thread at most)
            L.found = 1u; L.t_slot = (uint32_t)(2 * tid + i); L.n_above = above; L.members = tot[i];
            L.base_above = before; L.base_cand = bef[i];
        }
        above += tot[i];
        before += bef[i];
    }
    __syncthreads();
    if (!L.found) {  // uniform: fewer candidates than top_k in the histograms (cannot happen for a valid range)
        m.fallback = 1u;
        return m;
    }
    m.t_slot = L.t_slot;
    m.n_above = L.n_above;
    m.members = L.members;
    m.kk = (uint32_t)top_k - m.n_above;
    // candidates in the threshold bin of earlier chunks, and in the bins above it
    *base_above = L.base_above;
    *base_cand = L.base_cand;
    m.fallback = m.members > (uint32_t)kTmCand ? 1u : 0u;
    return m;
}

// LAST: no finish kernel follows.  The first chunk's workgroup also writes the sink and recent entries, the count and the window
// lists, and selects a flagged sequence from scratch; the members of the threshold bin are ranked by the logits kernel (TopkResolve).
template <bool LAST>
__global__ __launch_bounds__(kTopkThreads) void topk_place_kernel(const float* __restrict__ scores,
                                                                  const int32_t* __restrict__ seq_len,
                                                                  const uint2* __restrict__ range,
                                                                  const uint32_t* __restrict__ hist, int n_range, int S_max,
                                                                  int n_chunk, int top_k, int n_sink, int n_recent,
                                                                  int32_t* __restrict__ idx, TopkMeta* __restrict__ meta,
                                                                  uint2* __restrict__ cand_out, int32_t* __restrict__ n_sel,
                                                                  WindowLists wl)
{
    __shared__ TopkShared sh;
    __shared__ TmResolveLds rl;
    const int chunk = blockIdx.x, b = blockIdx.y;
    const int S = min(ld_uniform_i32(seq_len + b), S_max);  // (vector memory path: in flight with the scores)
    uint32_t keys[4 * kTmF4];
    tm_load_keys(scores + (size_t)b * S_max, S_max, chunk, n_sink, S - n_recent, keys);
    uint32_t base_above = 0u, base_cand = 0u;
    int phase = 0;
    const TopkMeta m = tm_resolve(rl, sh, phase, range, n_range, hist, b, chunk, wave_uniform(S), n_chunk, top_k, n_sink, n_recent, &base_above,
                                  &base_cand);
    if (chunk == 0 && threadIdx.x == 0) meta[b] = m;  // for the finish kernel, or the logits kernel
    if (LAST && chunk == 0) {  // uniform
        write_window_lists(wl, seq_len, b, S_max, top_k + n_sink + n_recent, kTopkThreads);
        if (m.fallback) {
            __syncthreads();  // (sh is used anew)
            topk_select_sequence<0>(sh, scores, seq_len, idx, n_sel, b, S_max, top_k, n_sink, n_recent);
            return;
        }
        int32_t* all = idx + (size_t)b * (top_k + n_sink + n_recent);
        const int len = wave_uniform(S);
        for (int t = threadIdx.x; t < n_sink; t += kTopkThreads) all[t] = t;
        for (int t = threadIdx.x; t < n_recent; t += kTopkThreads) all[n_sink + top_k + t] = len - n_recent + t;
        if (threadIdx.x == 0) n_sel[b] = top_k + n_sink + n_recent;
    }
    if (m.fallback) return;
    int slot[4 * kTmF4];
    uint32_t n_ab = 0u, n_eq = 0u;
#pragma unroll
    for (int i = 0; i < 4 * kTmF4; ++i) {
        slot[i] = keys[i] != 0u ? tm_slot(keys[i], m.flo, m.scale) : kTmBins;  // non-candidates: below every bin
        n_ab += slot[i] < (int)m.t_slot;
        n_eq += slot[i] == (int)m.t_slot;
    }
    uint32_t tot_ab, tot_eq;
    block_excl_scan2(n_ab, n_eq, sh, phase, &tot_ab, &tot_eq);
    int32_t* out = idx + (size_t)b * (top_k + n_sink + n_recent) + n_sink;
    uint2* cand = cand_out + (size_t)b * kTmCand;
    uint32_t pa = base_above + n_ab, pc = base_cand + n_eq;
#pragma unroll
    for (int i = 0; i < 4 * kTmF4; ++i) {
        const int j = tm_token(chunk, i);
        if (slot[i] < (int)m.t_slot) { if (pa < (uint32_t)top_k) out[pa] = j; ++pa; }
        else if (slot[i] == (int)m.t_slot) { if (pc < (uint32_t)kTmCand) cand[pc] = make_uint2(keys[i], (uint32_t)j); ++pc; }
    }
}

// What a kernel needs that reads a selection whose threshold bin has not been ranked (topk_place_kernel<true>): the entries
// n_sink + n_above .. n_sink + top_k of a sequence's list are the kk first of its `members` candidates, in token order.
struct TopkResolve {
    const TopkMeta* meta;    // [B]
    const uint2* cand;       // [B][kTmCand]
    int32_t* idx;            // [B][k_tot], the list to complete
    int n_sink, top_k;
};
constexpr int kTmResolveLds = kTmCand * (8 + 4 + 4);
// Ranks the candidates of a sequence (NT threads; raw[u]: candidate threadIdx.x + u NT) in `lds` (kTmResolveLds bytes, 16-byte
// aligned); returns the selected tokens in token order, in LDS, readable by all threads.
template <int NT>
__device__ __forceinline__ const int* tm_rank(unsigned char* lds, const uint2 (&raw)[(kTmCand + NT - 1) / NT], uint32_t nm, uint32_t kk)
{
    constexpr int NC = (kTmCand + NT - 1) / NT;
    uint64_t* s_c = reinterpret_cast<uint64_t*>(lds);  // key, then the token's complement: a larger number goes first
    uint32_t* s_sel = reinterpret_cast<uint32_t*>(lds + kTmCand * 8);
    int* s_tok = reinterpret_cast<int*>(lds + kTmCand * 12);
    const int tid = threadIdx.x;
    uint64_t me[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u) {
        me[u] = (uint64_t)raw[u].x << 32 | (uint32_t)~raw[u].y;
        if (tid + u * NT < kTmCand) s_c[tid + u * NT] = (uint32_t)(tid + u * NT) < nm ? me[u] : 0u;
    }
    __syncthreads();
    // rank among the members: larger key first, equal keys by smaller token index (slots past the members carry key 0 and
    // rank behind everything); eight members read together
    const uint32_t nm8 = (nm + 7u) & ~7u;
    bool sel[NC];
#pragma unroll
    for (int u = 0; u < NC; ++u) {
        const uint32_t e = tid + u * NT;
        uint32_t before = 0u;
        if (e < nm)
            for (uint32_t c = 0; c < nm8; c += 8) {
                uint64_t o[8];
#pragma unroll
                for (int v = 0; v < 8; ++v) o[v] = s_c[c + v];
#pragma unroll
                for (int v = 0; v < 8; ++v) before += o[v] > me[u];
            }
        sel[u] = e < nm && before < kk;
        // selected members in token order: the others' indices are replaced by the largest number
        if (e < (uint32_t)kTmCand) s_sel[e] = sel[u] ? raw[u].y : 0xffffffffu;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NC; ++u)
        if (sel[u]) {
            uint32_t pos = 0u;
            for (uint32_t c = 0; c < nm8; c += 8) {
                const u32x4 o0 = *reinterpret_cast<const u32x4*>(&s_sel[c]), o1 = *reinterpret_cast<const u32x4*>(&s_sel[c + 4]);
                pos += (o0.x < raw[u].y) + (o0.y < raw[u].y) + (o0.z < raw[u].y) + (o0.w < raw[u].y);
                pos += (o1.x < raw[u].y) + (o1.y < raw[u].y) + (o1.z < raw[u].y) + (o1.w < raw[u].y);
            }
            s_tok[pos] = (int)raw[u].y;
        }
    __syncthreads();
    return s_tok;
}

// finish: ranks the candidates; a flagged sequence is selected from scratch by this workgroup
__global__ __launch_bounds__(kTopkThreads) void topk_finish_kernel(const uint2* __restrict__ cand,
                                                                   const TopkMeta* __restrict__ meta,
                                                                   const int32_t* __restrict__ seq_len, int S_max, int top_k,
                                                                   int n_sink, int n_recent, int32_t* __restrict__ idx,
                                                                   int32_t* __restrict__ n_sel, const float* __restrict__ scores,
                                                                   WindowLists wl)
{
    __shared__ TopkShared sh;
    __shared__ __attribute__((aligned(16))) unsigned char s_rank[kTmResolveLds];
    const int b = blockIdx.x, tid = threadIdx.x;
    write_window_lists(wl, seq_len, b, S_max, top_k + n_sink + n_recent, kTopkThreads);
    // (the candidate pair, the length and the meta record are requested together; slots past the member count hold
    // stale pairs and are masked)
    const uint2 raw[1] = {cand[(size_t)b * kTmCand + min(tid, kTmCand - 1)]};
    const int S_v = ld_uniform_i32(seq_len + b);
    const TopkMeta m = meta[b];
    if (m.fallback) {  // uniform
        topk_select_sequence<0>(sh, scores, seq_len, idx, n_sel, b, S_max, top_k, n_sink, n_recent);
        return;
    }
    const int S = min(wave_uniform(S_v), S_max);
    const int k_tot = top_k + n_sink + n_recent;
    int32_t* out = idx + (size_t)b * k_tot;
    for (int t = tid; t < n_sink; t += kTopkThreads) out[t] = t;
    for (int t = tid; t < n_recent; t += kTopkThreads) out[n_sink + top_k + t] = S - n_recent + t;
    if (tid == 0) n_sel[b] = k_tot;
    const int* tok = tm_rank<kTopkThreads>(s_rank, raw, m.members, m.kk);
    if ((uint32_t)tid < m.kk) out[n_sink + m.n_above + tid] = tok[tid];
}

}  // namespace sals
