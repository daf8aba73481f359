// The value path of the sparse attention (Eq. 5; Algorithm 1, output step), evaluated as
// y_h = ((p_h V~_C) U_v[g(h) block]^T) : the same sum as p_h (V~_C U_v^T) in another order,
// so the selected values are never reconstructed.
//
//   attend_pv   per (sequence, token range, 64 latent columns):
//               T[h,:] = sum_j p_hj V~[C_j,:]  on the matrix cores, tokens being the
//               contraction axis (dealt in groups to the workgroup's four or eight waves); the gathered
//               rows are transposed in registers on the way.  The softmax weights are formed
//               on the fly, p = exp(logit - m_h) / Z_h, with m_h and Z_h merged in the prologue
//               from the per-tile statistics the logits kernel left.  Each token range writes an
//               fp32 partial sum.
//   attend_out  y[(b,h), c] = sum_i T[(b,h), i] U_v[g*128 + c, i]  on the matrix cores, after
//               adding the range partials (fp32, in a fixed order).
//
// bf16 storage: the fp32 weights p and the fp32 T are split into a bf16 head and a bf16
// remainder (two MFMAs each), which keeps about 16 mantissa bits.  fp32 storage: fp32 MFMAs.
#pragma once
#include "common.hpp"
#include "k_attend.hpp"
#include "k_project.hpp"

namespace sals {

constexpr int kPvTJ = 64;          // token ranges are whole multiples of this
constexpr int kPvCols = 64;        // latent columns per workgroup
constexpr int kPvMaxHeads = 64;    // H_q limit of these kernels
constexpr int kMaxRanges = 8;      // token ranges per sequence (the output projection adds them up)
constexpr int kPvMaxTok = 4096;    // tokens per workgroup, at most (their cache rows sit in LDS)

// The output projection that follows reads all of U_v once, in a launch of a few microseconds that mostly wait for it.  The
// value sum leaves many compute units idle: extra workgroups there touch every 64 bytes of U_v (its head blocks dealt to the
// XCDs as that launch deals them), so the projection finds it in its L2.
template <typename T>
__device__ __forceinline__ void warm_projector(const T* __restrict__ Uv, int r, int H_kv, int id, int n, int xcd, int n_threads)
{
    const int n_slots = (unsigned)n / kXcds, slot = (unsigned)id / kXcds;  // (n is a multiple of kXcds)
    const int per_head = kHeadDim * r * (int)sizeof(T) / 64;  // 64-byte pieces
    const int pieces = (H_kv - xcd + kXcds - 1) / kXcds * per_head;
    const unsigned char* base = reinterpret_cast<const unsigned char*>(Uv);
    for (int i0 = slot * n_threads + threadIdx.x; i0 < pieces; i0 += 4 * n_slots * n_threads) {
        uint32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // (from clamped addresses: requested together)
            const int i = min(i0 + u * n_slots * n_threads, pieces - 1), k = (unsigned)i / (unsigned)per_head;
            w[u] = *reinterpret_cast<const uint32_t*>(base + ((size_t)(xcd + k * kXcds) * per_head + (i - k * per_head)) * 64);
        }
        asm volatile("" :: "v"(w[0] ^ w[1] ^ w[2] ^ w[3]));  // (the values are of no use; the loads must stay)
    }
}

// NW waves (4 or 8), MB blocks of 32 heads.  The range's tokens are dealt to the waves in groups of one MFMA
// contraction step (16 tokens for bf16, 8 for fp32: half of them per half-wave); a wave works through its groups on
// its own, no barrier inside the loop, and keeps the loads of DEPTH groups in flight (the first are requested
// unconditionally, so that waiting for the statistics requested before them does not wait for them too).  DEPTH is small
// because the loop is unrolled that often and its code is fetched cold: the eight waves keep a CU's memory path busy by
// themselves.  bf16, r = 640, 32 heads, behind a copy that empties the caches, four | two | one group ahead: 16 sequences of
// 512 tokens in one range 8.9 | 7.9 | 7.8 us, 4 of 2048 in six 8.4 | 7.4 | 7.0; fp32 (groups half as long), 4 of 512 in four 6.4 |
// 5.9 | 5.8, 1 of 512 in two 7.5 | 7.3 | 7.6.  Four waves, one | two ahead: bf16, 256 tokens in two ranges 5.3 | 4.6, fp32, 64
// tokens 4.9 | 4.6.
//
// The MFMA's second operand wants, per lane, consecutive TOKENS of one column, while memory holds consecutive
// columns of one token.  bf16: lane l32 fetches the 32-bit word (columns 2 l32, 2 l32 + 1) of each of its eight
// tokens, a half-wave thus a whole 128-byte piece per token, and two byte permutes per token pair turn the eight words
// into the operand of the even column and the operand of the odd column: the transposition never leaves the
// registers.  fp32 (two tokens per MFMA, one per half-wave): the loaded words are the operands as they are.
//
// TWO: a second cache under the same softmax (the recent window beside the low-rank cache) takes the workgroups behind the
// first cache's: two launches of a few dozen workgroups each would follow one another for nothing (one sequence: 5.8 + 5.3 -> 5.3 us).
// Otherwise the workgroups behind warm the output projection's U_v.
template <typename T> struct PvSecond {
    const int32_t* idx; const int32_t* n_sel; const T* Vc; const float* logits; float* Tpart;
    int r, n_tr, tok_per_wg, k_tot, lk, S_max, ring;
};
// SPLIT: the logits are still partial sums over slices of the latent axis (`ksplit` of them).  Every workgroup adds up all of its
// sequence's (a thread has four tokens of a head at a time, all slices requested together), keeps its range's in LDS and
// takes maxima and normalisers on the way, under the gathered rows: the launch that would add them up before moves the same bytes, from
// L2, once, and costs 1 to 2 us of a small step (see value_adds_slices).
constexpr int kPvSplitTok = 128;                // tokens of a range, at most
constexpr size_t kPvSplitBytes = 128 << 10;     // partial logits of a sequence, at most (a workgroup reads them all)
template <typename T, int NW, int MB, bool TWO, bool SPLIT>
__device__ __forceinline__ void pv_block(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ n_sel, const float2* __restrict__ stats,
    int B, int r, int n_tr, int n_parts, int tok_per_wg, int k_tot, int H, int lk,
    const T* __restrict__ Vc, const float* __restrict__ logits, float* __restrict__ Tpart, int S_max, int ring,
    const T* __restrict__ Uv, int H_kv, PvSecond<T> second, int ksplit)
{
    static_assert((NW == 4 || NW == 8) && (MB == 1 || MB == 2), "four or eight waves, one or two head blocks");
    constexpr int kPvThreads = NW * 64;
    constexpr int ES = (int)sizeof(T);
    constexpr int VEC = elem<T>::vec;        // tokens per lane per group = elements per 16 bytes
    constexpr int KG = 2 * VEC;              // tokens per group (both half-waves)
    constexpr bool kSplit = ES == 2;
    constexpr int DEPTH = NW == 8 && kSplit ? 1 : 2;
    constexpr int ND = 8;                    // gathered words per lane and group: 8 tokens (bf16) | 4 tokens x 2 column blocks (fp32)

    __shared__ __attribute__((aligned(16))) int sRow[SPLIT ? kPvSplitTok : kPvMaxTok];  // cache row of every token of the nominal range
    constexpr int kLgRow = kPvSplitTok + 4;  // (16 heads' 16 bytes lie in different banks)
    __shared__ __attribute__((aligned(16))) float sLg[SPLIT ? MB * 32 : 1][SPLIT ? kLgRow : 4];  // the range's logits
    __shared__ float2 sMZ[kPvMaxHeads];      // per head: softmax maximum, 1 / normaliser
    constexpr int NBR = NW == 4 ? 2 : 1;     // column blocks per pass of the cross-wave sums
    __shared__ float red[NBR][NW][64][17];   // cross-wave sums, after the loop

    // Work items are ordered (sequence, token range, column block) with the column block fastest.
    // Workgroup ids are dealt round-robin to the XCDs; the map below gives each XCD a contiguous run of
    // the list, so the column blocks of one token range (same indices, logits and statistics, adjacent
    // 128-byte pieces of the same cache rows) meet in one L2.
    int n_cb = (unsigned)r / kPvCols, total = n_cb * n_tr * B, id = blockIdx.x;
    if (id >= total) {  // (uniform)
        if constexpr (TWO) {
            id -= total;
            idx = second.idx; n_sel = second.n_sel; Vc = second.Vc; logits = second.logits; Tpart = second.Tpart;
            r = second.r; n_tr = second.n_tr; tok_per_wg = second.tok_per_wg; k_tot = second.k_tot; lk = second.lk;
            S_max = second.S_max; ring = second.ring;
            n_cb = (unsigned)r / kPvCols; total = n_cb * n_tr * B;
        } else {
            warm_projector<T>(Uv, r, H_kv, id - total, gridDim.x - total, (unsigned)id % kXcds, kPvThreads);
            return;
        }
    }
    const int item = xcd_item(id, total);
    const int trb = idiv(item, n_cb), cb = item - trb * n_cb, b = idiv(trb, n_tr), tr = trb - b * n_tr;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int col0 = cb * kPvCols;
    const float* lg = logits + (size_t)b * H * lk;
    const int32_t* ib = idx + (size_t)b * k_tot;

    // everything that depends on nothing is requested at once: the count, the range's indices, the tile statistics
    const int n_v = ld_uniform_i32(n_sel + b);
    constexpr int LPH = kPvThreads / (SPLIT ? MB * 32 : kPvMaxHeads);   // lanes that share a head's tiles (SPLIT: tokens)
    const int sh = tid / LPH, sub = tid % LPH;
    float2 st8[8];
    constexpr int PU = 4;                     // SPLIT: groups of four tokens in flight
    f32x4 pl[SPLIT ? PU : 1][SPLIT ? kLsMaxSplit : 1];
    auto request_logits = [&](int j0) {       // groups j0, j0 + 1, ... of this lane: tokens 4 (sub + LPH j)
        const float* p[PU];
#pragma unroll
        for (int e = 0; e < PU; ++e)
            p[e] = logits + ((size_t)b * H + min(sh, H - 1)) * lk + min(4 * (sub + LPH * (j0 + e)), lk - 4);
#pragma unroll
        for (int u = 0; u < kLsMaxSplit; ++u)
            if (u < ksplit) {  // uniform
#pragma unroll
                for (int e = 0; e < PU; ++e)
                    pl[SPLIT ? e : 0][SPLIT ? u : 0] = *reinterpret_cast<const f32x4*>(p[e] + (size_t)u * B * H * lk);
            }
    };
    if constexpr (SPLIT) {
        const int v = ib[min(tr * tok_per_wg + min(tid, tok_per_wg - 1), k_tot - 1)];
        request_logits(0);
        const int pos = min(max(v, 0), S_max - 1);
        if (tid < tok_per_wg) sRow[tid] = ring > 0 ? (unsigned)pos % (unsigned)ring : pos;
    } else {
        for (int t = tid; t < tok_per_wg; t += kPvThreads) {
            const int j = tr * tok_per_wg + t;
            const int v = ib[min(j, k_tot - 1)];
            const int pos = min(max(v, 0), S_max - 1);
            sRow[t] = ring > 0 ? (unsigned)pos % (unsigned)ring : pos;  // ring cache: token t lies in row t mod ring
        }
        const float2* sp = stats + ((size_t)b * H + min(sh, H - 1)) * n_parts;
#pragma unroll
        for (int u = 0; u < 8; ++u) st8[u] = sp[min(sub + LPH * u, n_parts - 1)];  // (clamped: no load in a branch)
    }
    __syncthreads();  // rows of the range in LDS

    const unsigned char* vbytes =
        reinterpret_cast<const unsigned char*>(Vc + (size_t)b * (ring > 0 ? ring : S_max) * r + col0) + l32 * 4;
    const uint32_t row_bytes = (uint32_t)r * ES;
    const int g_last = tok_per_wg / KG - 1;  // (the range is a whole number of groups)
    // what a group needs from global memory: the gathered words and this lane's logits
    struct Stage { uint32_t R[ND]; f32x4 X[MB][VEC / 4]; };
    auto g_load = [&](Stage& S, int g) {
        const int t0 = min(g, g_last) * KG + hi * VEC;  // first of this lane's VEC tokens within the range
        int rows[VEC];
#pragma unroll
        for (int v = 0; v < VEC; v += 4) {
            const int4 r4 = *reinterpret_cast<const int4*>(&sRow[t0 + v]);
            rows[v] = r4.x; rows[v + 1] = r4.y; rows[v + 2] = r4.z; rows[v + 3] = r4.w;
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const unsigned char* src = vbytes + (uint64_t)(uint32_t)rows[v] * row_bytes;  // (one 32 x 32 + 64 bit instruction)
            S.R[v] = *reinterpret_cast<const uint32_t*>(src);
            if constexpr (!kSplit) S.R[VEC + v] = *reinterpret_cast<const uint32_t*>(src + 32 * 4);
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if constexpr (SPLIT) break;
            const int h = min(mb * 32 + l32, H - 1);  // (rows past the last head: any head's logits, never stored)
            const size_t off = (size_t)h * lk + tr * tok_per_wg + t0;
#pragma unroll
            for (int v = 0; v < VEC / 4; ++v) S.X[mb][v] = *reinterpret_cast<const f32x4*>(lg + off + 4 * v);
        }
    };
    Stage S[DEPTH];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) g_load(S[u], wave + NW * u);  // (the count is not known yet: nominal groups)

    // softmax maximum and normaliser of every head, merged in a fixed order (under the loads above)
    if constexpr (SPLIT) {
        const int n = n_v, r0 = tr * tok_per_wg;
        float2 st = make_float2(-INFINITY, 0.f);
        auto take = [&](int j0) {
            f32x4 d[PU];
            float m = -INFINITY, z = 0.f;
#pragma unroll
            for (int e = 0; e < PU; ++e) d[e] = pl[e][0];
#pragma unroll
            for (int u = 1; u < kLsMaxSplit; ++u)  // (in slice order)
                if (u < ksplit) {  // uniform
#pragma unroll
                    for (int e = 0; e < PU; ++e) d[e] += pl[SPLIT ? e : 0][SPLIT ? u : 0];
                }
#pragma unroll
            for (int e = 0; e < PU; ++e) {
                const int t = 4 * (sub + LPH * (j0 + e));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    d[e][i] = t + i < n ? d[e][i] : -INFINITY;
                    m = fmaxf(m, d[e][i]);
                }
                if (t >= r0 && t < r0 + tok_per_wg) *reinterpret_cast<f32x4*>(&sLg[sh][t - r0]) = d[e];
            }
            const float ref = m > -INFINITY ? m : 0.f;
#pragma unroll
            for (int e = 0; e < PU; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) z += d[e][i] > -INFINITY ? __expf(d[e][i] - ref) : 0.f;
            st = stat_merge(st, make_float2(m, z));
        };
        take(0);
        for (int j0 = PU; 4 * LPH * j0 < k_tot; j0 += PU) { request_logits(j0); take(j0); }
#pragma unroll
        for (int o = 1; o < LPH; o <<= 1) st = stat_merge(st, make_float2(__shfl_xor(st.x, o, kWave), __shfl_xor(st.y, o, kWave)));
        if (sub == 0) sMZ[sh] = make_float2(st.x > -INFINITY ? st.x : 0.f, st.y > 0.f ? 1.f / st.y : 0.f);
    } else {
        // (eight at a time: the maximum first, then eight exponentials that do not wait for each other)
        auto merge8 = [&](float2* e, int t0) {
            float m = -INFINITY, z = 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                e[u].x = t0 + LPH * u < n_parts ? e[u].x : -INFINITY;
                m = fmaxf(m, e[u].x);
            }
            const float ref = m > -INFINITY ? m : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) z += e[u].x > -INFINITY ? e[u].y * __expf(e[u].x - ref) : 0.f;
            return make_float2(m, z);
        };
        float2 st = merge8(st8, sub);
        const float2* sp = stats + ((size_t)b * H + min(sh, H - 1)) * n_parts;
        for (int t0 = sub + 8 * LPH; t0 - sub < n_parts; t0 += 8 * LPH) {  // (more tiles: further rounds of eight loads)
            float2 e[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = sp[min(t0 + LPH * u, n_parts - 1)];
            st = stat_merge(st, merge8(e, t0));
        }
#pragma unroll
        for (int o = 1; o < LPH; o <<= 1) st = stat_merge(st, make_float2(__shfl_xor(st.x, o, kWave), __shfl_xor(st.y, o, kWave)));
        if (sub == 0) sMZ[sh] = make_float2(st.x > -INFINITY ? st.x : 0.f, st.y > 0.f ? 1.f / st.y : 0.f);
    }
    __syncthreads();
    float2 mz[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) mz[mb] = sMZ[mb * 32 + l32];

    const int n = wave_uniform(n_v);
    const int j_begin = min(n, tr * tok_per_wg), j_end = min(n, j_begin + tok_per_wg);
    const int ntok = j_end - j_begin;        // (0 for a range past the selection: it still writes its zero sums)
    const int n_groups = (ntok + KG - 1) / KG;

    f32x16 acc[MB][2];  // [head block][column block]
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;

    auto do_group = [&](const Stage& S, int g) {
        const int t0 = g * KG + hi * VEC;
        // words of slots past the range count as zero (their rows may never have been written)
        uint32_t w[ND];
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const bool ok = t0 + v < ntok;
            w[v] = ok ? S.R[v] : 0u;
            if constexpr (!kSplit) w[VEC + v] = ok ? S.R[VEC + v] : 0u;
        }
        u32x4 vf[2];
        if constexpr (kSplit) {
            vf[0] = u32x4{__builtin_amdgcn_perm(w[1], w[0], 0x05040100u), __builtin_amdgcn_perm(w[3], w[2], 0x05040100u),
                          __builtin_amdgcn_perm(w[5], w[4], 0x05040100u), __builtin_amdgcn_perm(w[7], w[6], 0x05040100u)};
            vf[1] = u32x4{__builtin_amdgcn_perm(w[1], w[0], 0x07060302u), __builtin_amdgcn_perm(w[3], w[2], 0x07060302u),
                          __builtin_amdgcn_perm(w[5], w[4], 0x07060302u), __builtin_amdgcn_perm(w[7], w[6], 0x07060302u)};
        } else {
            vf[0] = u32x4{w[0], w[1], w[2], w[3]};
            vf[1] = u32x4{w[4], w[5], w[6], w[7]};
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            float pj[VEC];
#pragma unroll
            for (int v = 0; v < VEC; v += 4) {
                const f32x4 x = SPLIT ? *reinterpret_cast<const f32x4*>(&sLg[SPLIT ? mb * 32 + l32 : 0][SPLIT ? t0 + v : 0]) : S.X[mb][v / 4];
                // slots past the range carry no weight (their logits may be unwritten)
                const int jt = t0 + v;
                pj[v] = jt < ntok ? __expf(x.x - mz[mb].x) * mz[mb].y : 0.f;
                pj[v + 1] = jt + 1 < ntok ? __expf(x.y - mz[mb].x) * mz[mb].y : 0.f;
                pj[v + 2] = jt + 2 < ntok ? __expf(x.z - mz[mb].x) * mz[mb].y : 0.f;
                pj[v + 3] = jt + 3 < ntok ? __expf(x.w - mz[mb].x) * mz[mb].y : 0.f;
            }
            u32x4 ah, al;
            if constexpr (kSplit) {
                uint32_t ph[VEC], pl[VEC];
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    const bf16_t hb = f32_to_bf16(pj[v]);
                    ph[v] = hb;
                    pl[v] = f32_to_bf16(pj[v] - bf16_to_f32(hb));
                }
                ah = u32x4{ph[0] | (ph[1] << 16), ph[2] | (ph[3] << 16), ph[4] | (ph[5] << 16), ph[6] | (ph[7] << 16)};
                al = u32x4{pl[0] | (pl[1] << 16), pl[2] | (pl[3] << 16), pl[4] | (pl[5] << 16), pl[6] | (pl[7] << 16)};
            } else {
                ah = u32x4{__float_as_uint(pj[0]), __float_as_uint(pj[1]), __float_as_uint(pj[2]), __float_as_uint(pj[3])};
            }
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                mma_op<T>::run(ah, vf[nb], acc[mb][nb]);
                if constexpr (kSplit) mma_op<T>::run(al, vf[nb], acc[mb][nb]);
            }
        }
    };
    for (int i0 = 0; wave + NW * i0 < n_groups; i0 += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int g = wave + NW * (i0 + u);  // wave-uniform
            if (g < n_groups) do_group(S[u], g);
            if (g + NW * DEPTH < n_groups) g_load(S[u], g + NW * DEPTH);
        }
    }

    // The waves' sums, NBR column blocks of a head block at a time, added in wave order; wave w finishes 16 / NW of a
    // lane's 16 values.  acc[mb][nb][4a+c] is head mb*32 + 8a + 4hi + c; its column is 2 l32 + nb (bf16: even / odd
    // operand) or nb*32 + l32 (fp32).
    float* out_t = Tpart + (((size_t)tr * B + b) * H) * r;
    constexpr int PER = 16 / NW;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb0 = 0; nb0 < 2; nb0 += NBR) {
            if (mb + nb0 > 0) __syncthreads();
#pragma unroll
            for (int k = 0; k < NBR; ++k)
#pragma unroll
                for (int v = 0; v < 16; ++v) red[k][wave][lane][v] = acc[mb][nb0 + k][v];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < NBR; ++k) {
                const int col = col0 + (kSplit ? 2 * l32 + nb0 + k : (nb0 + k) * 32 + l32);
#pragma unroll
                for (int c = 0; c < PER; ++c) {
                    const int v = wave * PER + c;
                    const int h = mb * 32 + (v >> 2) * 8 + hi * 4 + (v & 3);
                    float sum = red[k][0][lane][v];
#pragma unroll
                    for (int w = 1; w < NW; ++w) sum += red[k][w][lane][v];
                    if (h < H) out_t[(size_t)h * r + col] = sum;
                }
            }
        }
}

template <typename T, int NW, int MB, bool TWO>
__global__ __launch_bounds__(NW * 64) void attend_pv_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ n_sel, const float2* __restrict__ stats,
    int B, int r, int n_tr, int n_parts, int tok_per_wg, int k_tot, int H, int lk,
    const T* __restrict__ Vc, const float* __restrict__ logits, float* __restrict__ Tpart, int S_max, int ring,
    const T* __restrict__ Uv, int H_kv, PvSecond<T> second)
{
    pv_block<T, NW, MB, TWO, false>(idx, n_sel, stats, B, r, n_tr, n_parts, tok_per_wg, k_tot, H, lk, Vc, logits, Tpart, S_max, ring, Uv,
                                    H_kv, second, 1);
}
template <typename T, int NW, int MB>
__global__ __launch_bounds__(NW * 64) void attend_pv_split_kernel(
    const int32_t* __restrict__ idx, const int32_t* __restrict__ n_sel, const float* __restrict__ plogits,
    int B, int r, int n_tr, int ksplit, int tok_per_wg, int k_tot, int H, int lk,
    const T* __restrict__ Vc, float* __restrict__ Tpart, int S_max, int ring, const T* __restrict__ Uv, int H_kv)
{
    pv_block<T, NW, MB, false, true>(idx, n_sel, nullptr, B, r, n_tr, 1, tok_per_wg, k_tot, H, lk, Vc, plogits, Tpart, S_max, ring, Uv,
                                     H_kv, PvSecond<T>{}, ksplit);
}

// ---------------------------------------------------------------------------------
// output projection: y[(b,h), c] = sum_i T[(b,h), i] U_v[g*128 + c, i]
//
// One workgroup per (KV head, 16 output channels, tile of up to 16 rows): 8 x H_kv x ceil(B*G/16)
// workgroups, so that the pass over U_v is spread over the whole chip.  16x16 MFMA tiles, columns the channels; the latent
// axis is dealt to the eight waves.  A row is a (sequence, head of the group) pair; with fewer than 16 of them (R = 1, 2, 4, 8)
// the lanes of the other rows load the pairs of 16 / R token ranges, so that one load serves that many ranges.  The ranges'
// sums are added in fp32 across those lanes (DPP shifts, one per halving of the ranges) before T is split into bf16 head and
// remainder: neighbouring ranges may cancel, which the 16 bits of a split range would not survive (products of the ranges,
// split one by one and added behind the MFMA: 1 % error where ranges cancel to 1e-4).
//
// A few KB per workgroup: the kernel is one memory round trip if every load is requested before the first is used, and
// little code (each launch starts with cold instruction caches).  So a wave requests BATCH latent steps of U_v with RPR
// loads of T each in one batch, from clamped addresses and without a branch (predicated loads were waited for one by one).
// Launch durations (kernel trace) before -> now: one sequence, 32 heads, r = 640, 4 ranges 5.9 -> 3.7 us (0.8 of it by
// warm_projector); 16 sequences, one range 5.4 -> 4.7; one sequence, 8 KV heads, 8 ranges 6.8 -> 4.0; 4 sequences, 6 ranges
// 7.7 -> 5.1; one sequence with a window of rank 2048 11.7 -> 7.9.
// ---------------------------------------------------------------------------------
constexpr int kOutWaves = 8;
// one cache's share of the contraction, as a wave walks it
template <typename T, int BATCH, int RPR> struct OutPass {
    static constexpr int VEC = elem<T>::vec, KS = 4 * VEC;  // latent coordinates per MFMA step
    const T* U;           // the workgroup's first channel row (scalar)
    const float* Tp;      // range 0 (scalar)
    uint32_t lane_u, lane_t, tstride;
    int nks, n_tr, q, sub, ks0;  // q ranges per load; this lane's is number sub of them
    u32x4 bf[BATCH];
    f32x4 x[BATCH][RPR][VEC / 4];

    __device__ void start(const T* U_, const float* Tp_, int r, int bh, int BH, int n_tr_, int q_, int sub_, int l16, int kg,
                          int wave)
    {
        U = U_; Tp = Tp_; nks = r / KS; n_tr = n_tr_; q = q_; sub = sub_; ks0 = wave;
        lane_u = l16 * r + kg * VEC; lane_t = bh * r + kg * VEC; tstride = (uint32_t)BH * r;
        load();
    }
    // latent coordinates of step u, from a clamped step
    __device__ int at(int u) const { return min(ks0 + kOutWaves * u, nks - 1) * KS; }
    __device__ void load()
    {
        size_t t_at[RPR];
#pragma unroll
        for (int w = 0; w < RPR; ++w) t_at[w] = (size_t)min(w * q + sub, n_tr - 1) * tstride + lane_t;
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            bf[u] = ld16(U + at(u) + lane_u);
#pragma unroll
            for (int w = 0; w < RPR; ++w)
#pragma unroll
                for (int v = 0; v < VEC / 4; ++v)
                    x[u][w][v] = *reinterpret_cast<const f32x4*>(Tp + at(u) + 4 * v + t_at[w]);
        }
    }
    // s += the value `DIST` lanes further on in the 16-lane row (zero past its end)
    template <int DIST> static __device__ void add_lanes(f32x4 (&s)[VEC / 4])
    {
#pragma unroll
        for (int v = 0; v < VEC / 4; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s[v][e] += __int_as_float(
                    __builtin_amdgcn_update_dpp(0, __float_as_int(s[v][e]), 0x100 + DIST, 0xf, 0xf, true));  // row_shl
    }
    static __device__ void add(f32x4& s, const f32x4& v, bool use)
    {
        s.x += use ? v.x : 0.f; s.y += use ? v.y : 0.f; s.z += use ? v.z : 0.f; s.w += use ? v.w : 0.f;
    }
    // the loaded batch, step by step, so that a step does not wait for the loads of the next
    template <bool FOLD> __device__ void steps(f32x4 (&s)[BATCH][VEC / 4], f32x4v& acc)
    {
        const int R = 16 >> __builtin_ctz(q), used = min(n_tr, q) * R;  // lanes of a 16-lane row that hold ranges
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            if (ks0 + kOutWaves * u < nks) {  // uniform
#pragma unroll
                for (int v = 0; v < VEC / 4; ++v)
#pragma unroll
                    for (int w = 0; w < RPR; ++w) add(s[u][v], x[u][w][v], w * q + sub < n_tr);
                if constexpr (FOLD) {
                    // the sum of all ranges in the lanes of the tile's first R rows (the others are not used): lane l + R
                    // holds the range after lane l's
                    if (used > 8 && R <= 8) add_lanes<8>(s[u]);
                    if (used > 4 && R <= 4) add_lanes<4>(s[u]);
                    if (used > 2 && R <= 2) add_lanes<2>(s[u]);
                    if (used > 1 && R == 1) add_lanes<1>(s[u]);
                }
                if constexpr (sizeof(T) == 2) {
                    uint32_t hw[8], lw[8];
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        const float t = s[u][v / 4][v % 4];
                        hw[v] = f32_to_bf16(t);
                        lw[v] = f32_to_bf16(t - bf16_to_f32((bf16_t)hw[v]));
                    }
                    mma16_op<T>::run(u32x4{hw[0] | (hw[1] << 16), hw[2] | (hw[3] << 16), hw[4] | (hw[5] << 16),
                                           hw[6] | (hw[7] << 16)}, bf[u], acc);
                    mma16_op<T>::run(u32x4{lw[0] | (lw[1] << 16), lw[2] | (lw[3] << 16), lw[4] | (lw[5] << 16),
                                           lw[6] | (lw[7] << 16)}, bf[u], acc);
                } else {
                    mma16_op<T>::run(u32x4{__float_as_uint(s[u][0].x), __float_as_uint(s[u][0].y),
                                           __float_as_uint(s[u][0].z), __float_as_uint(s[u][0].w)}, bf[u], acc);
                }
            }
        }
    }
    // every batch of this pass; the first has been loaded
    __device__ void run(f32x4v& acc)
    {
        for (;;) {
            f32x4 s[BATCH][VEC / 4];
#pragma unroll
            for (int u = 0; u < BATCH; ++u)
#pragma unroll
                for (int v = 0; v < VEC / 4; ++v) s[u][v] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (n_tr == 1) {  // uniform: one range, no code to jump over between the steps
                steps<false>(s, acc);
            } else {
                // more ranges than one load takes: the further ones first, through registers of their own (reloading x would
                // cost the usual case, without them, a wait for all of x)
                for (int t = RPR * q + sub; t - sub < n_tr; t += q) {  // uniform
                    f32x4 y[BATCH][VEC / 4];
                    const size_t t_at = (size_t)min(t, n_tr - 1) * tstride + lane_t;
#pragma unroll
                    for (int u = 0; u < BATCH; ++u)
#pragma unroll
                        for (int v = 0; v < VEC / 4; ++v) y[u][v] = *reinterpret_cast<const f32x4*>(Tp + at(u) + 4 * v + t_at);
#pragma unroll
                    for (int u = 0; u < BATCH; ++u)
#pragma unroll
                        for (int v = 0; v < VEC / 4; ++v) add(s[u][v], y[u][v], t < n_tr);
                }
                steps<true>(s, acc);
            }
            ks0 += kOutWaves * BATCH;
            if (ks0 >= nks) break;
            load();
            asm volatile("" ::: "memory");
        }
    }
};

// BATCH2 > 0: two caches of different rank share the output (recent window beside the low-rank cache); the first loads of
// both are in flight together
template <typename T, int BATCH, int RPR, int BATCH2>
__global__ __launch_bounds__(64 * kOutWaves) void attend_out_kernel(const T* __restrict__ Uv, const float* __restrict__ Tpart,
                                                                    int B, int r, int H, int H_kv, int n_tr, int R, int r2,
                                                                    int n_tr2, const T* __restrict__ Uv2,
                                                                    const float* __restrict__ Tpart2, T* __restrict__ out)
{
    constexpr int NW = kOutWaves;
    __shared__ float red[NW][16][17];  // [wave][row of the tile][channel]

    // KV head fastest: workgroup ids are dealt round-robin to the XCDs, so the eight channel blocks of
    // a head (which read the same value sums) share one XCD's L2 whenever H_kv is a multiple of 8
    const int g = blockIdx.x, cb = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kg = lane >> 4;
    const int G = idiv(H, H_kv);
    const int n_rows = B * G;  // (sequence, head of this group) pairs
    const int row0 = blockIdx.z * R;  // this workgroup's rows: R = 1, 2, 4, 8 or 16 of them
    const int row = min(row0 + (l16 & (R - 1)), n_rows - 1);  // (rows past the last one repeat it and are not stored)
    const int rb = idiv(row, G), bh = rb * H + g * G + row - rb * G;
    const int lr = __builtin_ctz(R), q = 16 >> lr, sub = l16 >> lr;  // (R is a power of two)
    const size_t c0 = (size_t)g * kHeadDim + cb * 16;

    f32x4v acc = {0.f, 0.f, 0.f, 0.f};
    OutPass<T, BATCH, RPR> p1;
    p1.start(Uv + c0 * r, Tpart, r, bh, B * H, n_tr, q, sub, l16, kg, wave);
    if constexpr (BATCH2 > 0) {
        OutPass<T, BATCH2, 1> p2;
        p2.start(Uv2 + c0 * r2, Tpart2, r2, bh, B * H, n_tr2, q, sub, l16, kg, wave);
        asm volatile("" ::: "memory");  // (keeps the loads above from being sunk towards their first use)
        p1.run(acc);
        p2.run(acc);
    } else {
        asm volatile("" ::: "memory");
        p1.run(acc);
    }
    // the waves' latent shares, in order: acc[v] is tile row 4*kg+v, channel l16
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][kg * 4 + v][l16] = acc[v];
    __syncthreads();
    if (tid < R * 16) {
        const int m = tid >> 4, c = tid & 15, orow = row0 + m;
        float y = red[0][m][c];
#pragma unroll
        for (int w = 1; w < NW; ++w) y += red[w][m][c];
        if (orow < n_rows) {
            const int ob = idiv(orow, G), oh = g * G + orow - ob * G;
            elem<T>::store(out + ((size_t)ob * H + oh) * kHeadDim + cb * 16 + c, y);
        }
    }
}

}  // namespace sals
