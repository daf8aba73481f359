// Selective key reconstruction with fused RoPE and query dot product
// (Algorithm 1, reconstruction / RoPE / logit steps; Sec. 4.4):
//   logits[b, h, j] = RoPE(q[b,h], q_pos[b]) . RoPE(U_k[g(h) block] K~[b, C_j], C_j) / sqrt(d)
//
// A gathered-row GEMM on the matrix cores: for one sequence, HEADS KV heads and a tile of
// selected tokens, D[dim, token] = sum_i U_k[dim, i] K~[C_token, i].  Both operands come straight from memory into LDS
// in 64-byte steps of the latent axis (16 bytes per lane, no registers in between): the packed U_k panel (shared by
// the waves of a head) and the gathered latent rows (shared by the heads), in a swizzled layout that the MFMA
// fragment reads hit without bank conflicts.  Four LDS stages; while the MFMAs of one half step run, the fragments of the
// next are read and a share of the loads of the step three ahead is issued between them (a load is held at issue while
// the path from the L2 is busy: issued together in front of the MFMAs, they keep the matrix cores waiting).
//
// The reconstructed keys stay in the accumulators.  The epilogue needs the tokens' cos/sin rows, 16 RoPE pairs per pass:
// each pass is one stage of LDS, loaded through the same ring as four more steps behind the latent axis.  It rotates the
// accumulators and dots them with the rotated query, so only logits are written, plus each (head, token
// tile)'s softmax maximum and normaliser for the value kernel.  The query itself is rotated
// (fp64-accurate angles) and scaled by 1/sqrt(d) in the prologue, while the first tile loads
// are in flight.
//
// Wave tile: 128 head dims (4 MFMA row blocks, in RoPE pair order) x 32*NB tokens.
// Workgroup: HEADS x NTG waves, i.e. HEADS heads x (NTG*32*NB) tokens.  Two shapes: two heads x 256 tokens (8 waves) where that
// fills the chip: the least operand traffic per product, the matrix cores' power is the bound; one head x 128 tokens
// (4 waves, two workgroups per compute unit) for the launches in between that and the 64-token kernel, where idle compute
// units and the feed from the L2 are the bound.  Attention in all (sals_sparse_attend), 256-token tiles / these / the 64-token
// kernel: one sequence, 32 heads, 1024 tokens, r = 640: 26.3 / 20 / 24.5 us; one sequence, 8 KV heads, 4160 tokens, r = 512:
// 30.3 / 25.4 / 37.3; 12 sequences, 8 KV heads, 512 tokens, r = 640: 31.1 / 26.3 / 38.2; and 16 sequences, 32 heads, 512 tokens:
// 54.2 / 69.3 / 156.
#pragma once
#include "common.hpp"
#include "k_attend.hpp"
#include "k_gemm.hpp"
#include "k_topk_multi.hpp"

namespace sals {

constexpr int kLgChunk = 128;  // bytes per row of a [rows][128 B] swizzled LDS tile
constexpr int kLgStep = 64;    // bytes of the latent axis per pipeline step (= one packed U_k block)

// LDS tiles are read and written 16 bytes per lane; such an access is conflict-free when each
// group of 16 consecutive lanes covers all 16 bank groups (address / 16 mod 16).  A fragment read
// takes one piece index from 16 consecutive rows, a staging write takes consecutive pieces, so
// the piece index is XOR-ed with row bits.
// byte offset of 16-byte piece `pc` of row `row` inside a [rows][128 B] tile
__device__ __forceinline__ int swz(int row, int pc) { return row * kLgChunk + ((pc ^ ((row >> 1) & 7)) << 4); }
// the same for a [rows][64 B] tile
__device__ __forceinline__ int swz64(int row, int pc) { return row * kLgStep + ((pc ^ ((row >> 2) & 3)) << 4); }

template <int HEADS, int NTG, int NB> struct logits_cfg {
    static constexpr int NT = 64 * HEADS * NTG;            // threads
    static constexpr int TOK = NTG * NB * 32;              // tokens per workgroup
    static constexpr int A_BYTES = HEADS * 128 * kLgStep;  // U_k panel per step
    static constexpr int B_BYTES = TOK * kLgStep;          // gathered rows per step
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int NA = A_BYTES / 16 / NT;           // 16-byte pieces per thread per step
    static constexpr int NBP = B_BYTES / 16 / NT;
    static constexpr int CS_BYTES = TOK * kLgChunk;        // cos/sin of 16 pairs for every token
    static constexpr int NCS = CS_BYTES / 16 / NT;
    static constexpr int SLOT = STAGE > CS_BYTES ? STAGE : CS_BYTES;
    static constexpr size_t LDS = 4 * (size_t)SLOT;
};

// GB: query heads of a KV head handled as one block of straight-line code (1, or 4 when the group size is a multiple
// of 4): the LDS reads and the reductions of a block's heads are in flight together instead of one head after the other.
// GFIX: the group size when it is known at compile time (1 and 4, the common ones; 0: read from the arguments), which
// takes the per-block branches out of the epilogue.
// MULTI: a tile is made of the (at most 64 token) selections of consecutive SEQUENCES, 64 slots each, instead of as many
// tokens of one sequence: short selections such as a recent window then share one pass over the head's projector among
// the sequences of a tile.  Each sequence has its own query, count, index list and cache;
// the latent axis may be cut into `ksplit` slices of whole steps (the logit is additive over latent coordinates), whose partial
// logits go to `plogits` for logits_finish_kernel.
// BYLEN (MULTI only): the selections are recent windows given by the sequence lengths (`win`; idx and n_sel are not read).
// SIDE: `split` names the logits of another pass whose slices are still to be added up, on the side (one job per wave).
// RESOLVE: the selection's threshold bin is still to be ranked (`res`): by every workgroup whose tile reaches those entries, those
// of the first heads leave them in the list.
template <typename T, int HEADS, int NTG, int NB, int GB, int GFIX, bool MULTI, bool BYLEN, bool SIDE, bool RESOLVE>
__device__ __forceinline__ void logits_tile(
    int block, const T* __restrict__ Kc, const T* __restrict__ UkP, const int32_t* __restrict__ idx,
    const int32_t* __restrict__ n_sel, const T* __restrict__ q, const int32_t* __restrict__ q_pos,
    const float2* __restrict__ rope, const InvFreq& inv,
    float* __restrict__ logits, float2* __restrict__ stats, int B, int S_max, int r, int H, int H_kv,
    int k_tot, int lk, int n_parts, int heads_fastest, int style, float scale, int ring, int stats_stride,
    float* __restrict__ plogits, int ksplit, const WindowByLength& win, const SplitLogits& split, const TopkResolve& res)
{
    typedef logits_cfg<HEADS, NTG, NB> C;
    static_assert(!BYLEN || MULTI, "a window by length fills tiles of several sequences");
    static_assert(!MULTI || NB <= 2, "a sequence's 64 slots are those of one or two waves");
    constexpr int SQ = MULTI ? C::TOK / 64 : 1;   // sequences per tile
    constexpr int WT = NB * 32;                   // tokens per wave
    constexpr int NT = C::NT, NA = C::NA, NBP = C::NBP, NCS = C::NCS;
    constexpr int ES = (int)sizeof(T);
    static_assert(C::A_BYTES % (16 * NT) == 0 && C::B_BYTES % (16 * NT) == 0 && C::CS_BYTES % (16 * NT) == 0,
                  "tile / thread mismatch");
    static_assert(kMaxGroup % GB == 0 && (GFIX == 0 || (GFIX % GB == 0 && GFIX <= kMaxGroup)), "head blocks tile the group");
    constexpr int kGroupEnd = GFIX > 0 ? GFIX : kMaxGroup;

    // Workgroup id -> (sequence, token tile, head block).  Consecutive ids are dispatched to
    // different XCDs, each with its own L2, so every XCD gets one contiguous range of the work
    // list; the list is ordered so that a range shares the larger operand: heads fastest keeps
    // the gathered rows of a few token tiles in that L2 (U_k is re-read per XCD), tiles fastest
    // keeps the U_k panels of a few heads there (the rows are re-read per XCD).
    int b, g0, part, kz = 0;   // MULTI: b is the first sequence of the tile
    if constexpr (MULTI) {
        // list order (head, sequence group, latent slice): an XCD's range keeps a few heads' projector slices
        const int nsg = (unsigned)(B + SQ - 1) / SQ, N = nsg * ((unsigned)H_kv / HEADS) * ksplit;
        const int w = xcd_item(block, N);
        const int hb = idiv(w, nsg * ksplit), rest = w - hb * (nsg * ksplit), sg = idiv(rest, ksplit);
        g0 = hb * HEADS;
        b = sg * SQ; kz = rest - sg * ksplit; part = 0;
    } else {
        const int n_y = (unsigned)H_kv / HEADS, N = n_parts * n_y * B;
        const int w = xcd_item(block, N);
        if (heads_fastest) {
            const int bt = idiv(w, n_y);
            g0 = (w - bt * n_y) * HEADS; b = idiv(bt, n_parts); part = bt - b * n_parts;
        } else {
            const int hb = idiv(w, n_parts * B), bt = w - hb * (n_parts * B);
            g0 = hb * HEADS; b = idiv(bt, n_parts); part = bt - b * n_parts;
        }
    }
    const int tok0 = part * C::TOK;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int hh = wave / NTG, tg = wave % NTG;   // head of the tile, token group
    // sequence of tile token t (MULTI: sequence b + t / 64; sequences past the batch repeat the last one and get no weight)
    const int sw = MULTI ? tg * WT / 64 : 0;  // this wave's sequence within the tile
    auto seq_of = [&](int t) { return MULTI ? min(b + (t >> 6), B - 1) : b; };
    // count and query position: of this wave's sequence (MULTI: the position is needed per thread
    // for the thread's share of the cos/sin rows, see rotate_queries)
    const int n_v = ld_uniform_i32((BYLEN ? win.seq_len : n_sel) + (MULTI ? seq_of(tg * WT) : b));
    const int qpos_v = MULTI ? q_pos[seq_of(tid & ~63)] : ld_uniform_i32(q_pos + b);  // in flight with the loads below
    const int G = GFIX > 0 ? GFIX : idiv(H, H_kv);
    const int g = g0 + hh;
    static_assert(!RESOLVE || !MULTI, "a tile of one sequence");
    uint2 cand[(kTmCand + NT - 1) / NT];
    u32x4 meta = {1u, 0u, 0u, 0u};   // fallback, threshold slot, selected members, scores above
    uint32_t members = 0u;
    if constexpr (RESOLVE) {
        int zero;
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));  // (through the vector memory path, see ld_uniform_i32)
        const uint32_t* mp = reinterpret_cast<const uint32_t*>(res.meta + b) + zero;
        meta = ld16(mp);
        members = mp[4];
#pragma unroll
        for (int u = 0; u < (kTmCand + NT - 1) / NT; ++u) cand[u] = res.cand[(size_t)b * kTmCand + min(tid + u * NT, kTmCand - 1)];
    }

    // Everything the prologue needs from memory is requested before anything is waited for, from clamped
    // addresses so that no load sits in a branch: the tile's token rows (slots at or past the selection count
    // read whatever the index array holds there, clamped to a valid row; they get no weight), the raw query
    // pairs of the tile's heads and the query position.
    const int rows_per_seq = ring > 0 ? ring : S_max;
    SplitLogitsJob job;
    const int job_id = block * (NT / 64) + wave;
    const bool has_job = SIDE && job_id < split.rows * split.n_parts;  // uniform
    auto request_job = [&](int j) { const int row = idiv(j, split.n_parts); job.request(split, row, j - row * split.n_parts); };
    if (has_job) request_job(job_id);
    // cache row (= RoPE position) of tile token t: slot t of the one sequence, or slot t % 64 of sequence b + t / 64
    auto window_of = [&](int len, int* S) {  // tokens of a window by length
        *S = min(max(len, 0), S_max);
        return min(k_tot, min(*S, win.k_tot));
    };
    auto row_of = [&](int t) {
        if constexpr (BYLEN) {
            int S;
            const int nw = window_of(win.seq_len[seq_of(t)], &S);
            return min(max(S - nw + ((t & 63) < nw ? t & 63 : 0), 0), S_max - 1);
        }
        const int32_t* ib = idx + (size_t)seq_of(t) * k_tot;
        return min(max(ib[min(MULTI ? (t & 63) : tok0 + t, k_tot - 1)], 0), S_max - 1);
    };
    // this lane's row in each of the wave's 1 KB pieces (16 rows of 64 bytes) of the gathered side
    constexpr int NW = NT / 64;
    int b_row[NBP];
#pragma unroll
    for (int i = 0; i < NBP; ++i) {
        const int t = (wave + i * NW) * 16 + (lane >> 2);
        b_row[i] = row_of(t);
        if (ring > 0) b_row[i] %= ring;  // ring cache: token t lies in row t mod ring
        if (MULTI) b_row[i] += (seq_of(t) - b) * rows_per_seq;  // (rows counted from the tile's first sequence)
    }
    constexpr int NSP = (C::TOK + NT - 1) / NT;
    int pos_reg[NSP];
#pragma unroll
    for (int u = 0; u < NSP; ++u) pos_reg[u] = row_of(min(tid + u * NT, C::TOK - 1));
    constexpr int QP = (SQ * HEADS * (GFIX > 0 ? GFIX : kMaxGroup) * kPairs + NT - 1) / NT;
    float qa[QP], qb[QP];
#pragma unroll
    for (int u = 0; u < QP; ++u) {
        // query pair t: (sequence of the tile, query head of the tile's heads, pair)
        const int t = min(tid + u * NT, SQ * HEADS * G * kPairs - 1), p = t & (kPairs - 1);
        const int hq = t >> 6, sq = MULTI ? idiv(hq, HEADS * G) : 0, hm = MULTI ? hq - sq * (HEADS * G) : hq;
        const T* qrow = q + ((size_t)seq_of(sq * 64) * H + (size_t)g0 * G + hm) * kHeadDim;
        qa[u] = elem<T>::load(qrow + pair_first(p, style));
        qb[u] = elem<T>::load(qrow + pair_second(p, style));
    }
    // ---- global sources ----------------------------------------------------------------
    // U_k panel: the packed layout is [head][step][128 slots][64 B], so a step of a head is 8 KB in one piece and a wave's
    // load takes 16 slots.  In LDS the 16-byte piece of slot (row) r at position p is piece p ^ ((r >> 2) & 3).
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];  // [4 slots]: [A | B], later cos/sin passes
    const uint32_t lds0 = lds_offset(lds);
    const int prow = lane >> 2, ppos = lane & 3;
    const uint32_t a_off = (uint32_t)(prow * kLgStep + ((ppos ^ ((prow >> 2) & 3)) << 4));
    const unsigned char* a_base = reinterpret_cast<const unsigned char*>(UkP + (size_t)g0 * kHeadDim * r);
    const size_t head_bytes = (size_t)kHeadDim * r * ES;
    // steps of the latent axis: all of them, or this workgroup's slice
    const int kc_base = MULTI ? r * ES / kLgStep * kz / ksplit : 0;
    const int nkc = MULTI ? r * ES / kLgStep * (kz + 1) / ksplit - kc_base : r * ES / kLgStep;
    auto slot_at = [&](int step) { return lds0 + (uint32_t)(step & 3) * C::SLOT; };
    auto load_a = [&](int i, int step) {
        const int piece = wave + i * NW;  // 8 pieces per head
        load_lds16(a_base + (size_t)(piece >> 3) * head_bytes + (size_t)(kc_base + step) * (128 * kLgStep) + (piece & 7) * 1024,
                   a_off, slot_at(step) + piece * 1024);
    };
    // the panels of the first three steps depend on nothing
#pragma unroll
    for (int st = 0; st < 3; ++st)
        if (st < nkc) {  // uniform
#pragma unroll
            for (int i = 0; i < NA; ++i) load_a(i, st);
        }
    // MULTI: a sequence past the batch has no tokens
    int n = wave_uniform(n_v);
    if constexpr (BYLEN) { int S; n = window_of(n, &S); }
    if (MULTI && b + sw >= B) n = 0;
    if (has_job) {
        job.finish(split);
        // (the rest, where there are more than waves)
        for (int j = job_id + (int)gridDim.x * (NT / 64); j < split.rows * split.n_parts; j += (int)gridDim.x * (NT / 64)) {
            request_job(j);
            job.finish(split);
        }
    }
    const int qpos = MULTI ? qpos_v : wave_uniform(qpos_v);
    if (!MULTI && tok0 >= n) {  // no selected token in this tile: neutral statistics
        if (tid < HEADS * G)
            stats[((size_t)b * H + (size_t)g0 * G + tid) * stats_stride + part] = make_float2(-INFINITY, 0.f);
        vm_wait<0>();  // (no load may land in LDS that another workgroup has been given)
        return;
    }

    if constexpr (RESOLVE) {
        static_assert(C::SLOT >= kTmResolveLds, "the last stage is free until the main loop");
        const int lo = res.n_sink + wave_uniform((int)meta.w), up = res.n_sink + res.top_k;
        if (!wave_uniform((int)meta.x) && lo < tok0 + C::TOK && up > tok0) {  // uniform
            const int* tok = tm_rank<NT>(lds + 3 * C::SLOT, cand, (uint32_t)wave_uniform((int)members), (uint32_t)wave_uniform((int)meta.z));
            auto entry = [&](int t, int row) {
                const int slot = tok0 + t;
                return slot >= lo && slot < up ? min(max(tok[slot - lo], 0), S_max - 1) : row;
            };
#pragma unroll
            for (int i = 0; i < NBP; ++i) b_row[i] = entry((wave + i * NW) * 16 + (lane >> 2), b_row[i]);
#pragma unroll
            for (int u = 0; u < NSP; ++u) pos_reg[u] = entry(min(tid + u * NT, C::TOK - 1), pos_reg[u]);
            if (g0 == 0) {
                for (int t = tid; t < C::TOK; t += NT)
                    if (tok0 + t >= lo && tok0 + t < up) res.idx[(size_t)b * k_tot + tok0 + t] = tok[tok0 + t - lo];
            }
        }
    }
    constexpr int GQ = MULTI && GFIX > 0 ? GFIX : kMaxGroup;   // (eight heads' worth would not fit beside tiles of four sequences)
    __shared__ __attribute__((aligned(16))) float sQ[SQ * HEADS][GQ][kHeadDim];
    __shared__ float2 sCS[SQ][kPairs];
    __shared__ float2 sStat[HEADS][NTG][kMaxGroup];
    __shared__ int sPos[C::TOK];  // cache row (= RoPE position) of every token of the tile

#pragma unroll
    for (int u = 0; u < NSP; ++u)
        if (tid + u * NT < C::TOK) sPos[tid + u * NT] = pos_reg[u];
    // cos/sin of the query position: thread -> (sequence tid / 64, pair tid % 64); qpos is that sequence's.  Requested
    // here, ahead of the first operand loads, so that the wait for it does not include theirs.
    const bool q_in_table = qpos >= 0 && qpos <= S_max;  // the table holds exactly these positions
    float2 qcs = make_float2(1.f, 0.f);
    if (tid < SQ * kPairs) qcs = rope[(size_t)(q_in_table ? qpos : 0) * kPairs + (tid & (kPairs - 1))];
    auto rotate_queries = [&]() {
        if (tid < SQ * kPairs) {
            const int pr = tid & (kPairs - 1);
            if (!q_in_table) {
                double sn, c;
                sincos((double)qpos * inv.f[pr], &sn, &c);
                qcs = make_float2((float)c, (float)sn);
            }
            sCS[tid >> 6][pr] = qcs;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < QP; ++u) {
            const int t = tid + u * NT;
            if (t < SQ * HEADS * G * kPairs) {
                // (t / 64 = (sequence * heads of the tile + head) * G + head of the group)
                const int p = t & (kPairs - 1), hm = t >> 6;
                const float2 c = sCS[MULTI ? idiv(hm, HEADS * G) : 0][p];
                const int hd = idiv(hm, G);
                float* dst = &sQ[0][0][0] + (size_t)(hd * GQ + hm - hd * G) * kHeadDim;
                rotate_query(qa[u], qb[u], c, scale, dst[p], dst[kPairs + p]);
            }
        }
    };

    // gathered rows and, behind the latent axis, the cos/sin passes: token rows of 128 bytes, piece p of row r at position
    // p ^ ((r >> 1) & 7)
    const unsigned char* b_src[NBP];
#pragma unroll
    for (int i = 0; i < NBP; ++i)
        b_src[i] = reinterpret_cast<const unsigned char*>(Kc + ((size_t)b * rows_per_seq + b_row[i]) * r) +
                   (size_t)kc_base * kLgStep + ((ppos ^ ((prow >> 2) & 3)) << 4);
    auto load_b = [&](int i, int step) {
        load_lds16(b_src[i] + (size_t)step * kLgStep, slot_at(step) + C::A_BYTES + (wave + i * NW) * 1024);
    };
    const unsigned char* rope_b = reinterpret_cast<const unsigned char*>(rope);
    uint32_t cs_off[NCS];
    auto load_cs = [&](int i, int ps) {
        load_lds16(rope_b + ps * kLgChunk, cs_off[i], slot_at(nkc + ps) + (wave + i * NW) * 1024);
    };
    // load i of NL (or NCS) of virtual step `step`
    constexpr int NL = NA + NBP;
    auto load_piece = [&](int i, int step) {
        if (step < nkc) {  // uniform
            if (i < NA) load_a(i, step); else if (i < NL) load_b(i - NA, step);
        } else if (i < NCS) {
            load_cs(i, step - nkc);
        }
    };

    f32x16 acc[4][NB];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;

    // MFMA fragments of one half step (32 latent bytes): NB token blocks, 4 head-dim blocks
    struct Frags { u32x4 b[NB]; u32x4 a[4]; };
    const uint32_t f_at[2] = {(uint32_t)swz64(l32, hi), (uint32_t)swz64(l32, 2 + hi)};
    const unsigned char* pa = lds + hh * 128 * kLgStep;
    const unsigned char* pb = lds + C::A_BYTES + tg * NB * 32 * kLgStep;
    auto read_frag = [&](Frags& F, int i, uint32_t slot, int ks) {
        if (i < NB) F.b[i] = *reinterpret_cast<const u32x4*>(pb + slot + f_at[ks] + i * 32 * kLgStep);
        else F.a[i - NB] = *reinterpret_cast<const u32x4*>(pa + slot + f_at[ks] + (i - NB) * 32 * kLgStep);
    };
    // One half step: the MFMAs of `F`, between them the reads of the next half step's fragments into `N` and half of this
    // wave's loads of the step three ahead, in this order.
    constexpr int NLM = NL > NCS ? NL : NCS;
    auto half_step = [&](const Frags& F, Frags& N, uint32_t n_slot, int n_ks, int step, auto half) {
        constexpr int NM = 4 * NB, NR = 4 + NB, H2 = decltype(half)::value;
        constexpr int L0 = H2 ? (NLM + 1) / 2 : 0, L1 = H2 ? NLM : (NLM + 1) / 2;
#pragma unroll
        for (int j = 0; j < NM; ++j) {
            mma_op<T>::run(F.a[j / NB], F.b[j % NB], acc[j / NB][j % NB]);
#pragma unroll
            for (int i = j * NR / NM; i < (j + 1) * NR / NM; ++i) read_frag(N, i, n_slot, n_ks);
#pragma unroll
            for (int i = L0 + j * (L1 - L0) / NM; i < L0 + (j + 1) * (L1 - L0) / NM; ++i) load_piece(i, step);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    {
#pragma unroll
        for (int st = 0; st < 3; ++st)
            if (st < nkc) {  // uniform
#pragma unroll
                for (int i = 0; i < NBP; ++i) load_b(i, st);
            }
        rotate_queries();  // (its barrier also publishes sPos)
#pragma unroll
        for (int i = 0; i < NCS; ++i) {
            const int row = (wave + i * NW) * 8 + (lane >> 3);
            cs_off[i] = (uint32_t)sPos[row] * (uint32_t)(kPairs * sizeof(float2)) + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) << 4);
        }
        for (int st = nkc; st < 3; ++st) {  // (fewer than three latent steps)
#pragma unroll
            for (int i = 0; i < NCS; ++i) load_cs(i, st - nkc);
        }
        Frags F0, F1;
        vm_wait<(NBP < NCS ? NBP : NCS)>();  // steps 0 and 1 have landed
        wg_barrier();
#pragma unroll
        for (int i = 0; i < 4 + NB; ++i) read_frag(F0, i, 0, 0);
        for (int kc = 0; kc < nkc; ++kc) {
            // steps up to kc + 1 have landed, everywhere; every wave is done with step kc - 1
            if (kc + 2 < nkc) vm_wait<NL>(); else vm_wait<NCS>();
            wg_barrier();
            const uint32_t cur = (uint32_t)(kc & 3) * C::SLOT, nxt = (uint32_t)((kc + 1) & 3) * C::SLOT;
            half_step(F0, F1, cur, 1, kc + 3, std::integral_constant<int, 0>{});
            half_step(F1, F0, nxt, 0, kc + 3, std::integral_constant<int, 1>{});
        }
    }

    // ---- epilogue.  A lane holds, for token l32 of each block, slots mb*32 + 8a + 4hi + c; slot < 64
    // is the first element of pair (slot), slot+64 its partner (mb+2).  Pass ps = 2*ml + ah covers
    // the pairs ml*32 + ah*16 .. +16; the tokens' 128-byte cos/sin pieces of a pass are one slot of LDS, the last of
    // them loaded once the main loop has left its slot. ------------------------------------------
    float dot[kMaxGroup][NB];
#pragma unroll
    for (int m = 0; m < kMaxGroup; ++m)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) dot[m][nb] = 0.f;
    {
        wg_barrier();  // every wave is done with the last step
#pragma unroll
        for (int i = 0; i < NCS; ++i) load_cs(i, 3);
#pragma unroll
        for (int ps = 0; ps < 4; ++ps) {
            const int ml = ps >> 1, ah = ps & 1;
            if (ps == 1) { vm_wait<NCS>(); wg_barrier(); }  // passes 1 and 2 (pass 0 landed before the last step)
            if (ps == 3) { vm_wait<0>(); wg_barrier(); }
            const unsigned char* cb = lds + (size_t)((nkc + ps) & 3) * C::SLOT;
#pragma unroll
            for (int al = 0; al < 2; ++al) {
                const int a = 2 * ah + al;
                const int p0 = ml * 32 + a * 8 + hi * 4;
                // the rotated key elements of this lane's NB tokens first, then every query head's pieces are read
                // from LDS once and used for all NB tokens
                float k1[NB][4], k2[NB][4];
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int row = (tg * NB + nb) * 32 + l32;
                    const f32x4 t0 = *reinterpret_cast<const f32x4*>(cb + swz(row, al * 4 + hi * 2));      // pairs p0, p0+1
                    const f32x4 t1 = *reinterpret_cast<const f32x4*>(cb + swz(row, al * 4 + hi * 2 + 1));  // p0+2, p0+3
                    const float cc[4] = {t0.x, t0.z, t1.x, t1.z}, ss[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        rotate_key(acc[ml][nb][a * 4 + c], acc[ml + 2][nb][a * 4 + c], cc[c], ss[c], k1[nb][c], k2[nb][c]);
                }
#pragma unroll
                for (int m0 = 0; m0 < kGroupEnd; m0 += GB) {
                    if (GFIX > 0 || m0 < G) {  // uniform; G is a multiple of GB
                        f32x4 q1[GB], q2[GB];
#pragma unroll
                        for (int mi = 0; mi < GB; ++mi) {
                            q1[mi] = *reinterpret_cast<const f32x4*>(&sQ[MULTI ? sw * HEADS + hh : hh][m0 + mi][p0]);
                            q2[mi] = *reinterpret_cast<const f32x4*>(&sQ[MULTI ? sw * HEADS + hh : hh][m0 + mi][kPairs + p0]);
                        }
#pragma unroll
                        for (int mi = 0; mi < GB; ++mi)
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb) dot[m0 + mi][nb] += dot_pairs(q1[mi], q2[mi], k1[nb], k2[nb]);
                    }
                }
            }
        }
    }

    bool ok[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) ok[nb] = (MULTI ? (tg * WT & 63) + nb * 32 + l32 : tok0 + (tg * NB + nb) * 32 + l32) < n;
    const int bs = MULTI ? seq_of(tg * WT) : b;          // sequence of this wave's tokens
    const bool seq_real = !MULTI || b + sw < B;          // (a sequence past the batch writes nothing)
    const bool partial = MULTI && (HEADS > 1 || ksplit > 1);  // (tiles of several heads and sequences always have slices)
#pragma unroll
    for (int m0 = 0; m0 < kGroupEnd; m0 += GB) {
        if (GFIX > 0 || m0 < G) {  // uniform
#pragma unroll
            for (int mi = 0; mi < GB; ++mi)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) dot[m0 + mi][nb] += __shfl_xor(dot[m0 + mi][nb], 32, kWave);
#pragma unroll
            for (int mi = 0; mi < GB; ++mi)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int slot = MULTI ? (tg * WT & 63) + nb * 32 + l32 : tok0 + (tg * NB + nb) * 32 + l32;
                    const size_t at = ((size_t)bs * H + g * G + m0 + mi) * lk + slot;
                    if (partial) {  // uniform: this slice's share of the logit
                        if (hi == 0 && slot < lk && seq_real) plogits[(size_t)kz * B * H * lk + at] = dot[m0 + mi][nb];
                    } else if (hi == 0 && slot < lk && seq_real) {
                        logits[at] = ok[nb] ? dot[m0 + mi][nb] : -INFINITY;
                    }
                }
            if (partial) continue;  // (statistics are taken when the slices are added up)
            // softmax statistics of this tile, per head: the waves' (max, sum exp) merged in wave order below
            float mx[GB], se[GB];
#pragma unroll
            for (int mi = 0; mi < GB; ++mi) {
                mx[mi] = -INFINITY;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) mx[mi] = ok[nb] ? fmaxf(mx[mi], dot[m0 + mi][nb]) : mx[mi];
            }
#pragma unroll
            for (int mi = 0; mi < GB; ++mi) mx[mi] = wave_max(mx[mi]);
#pragma unroll
            for (int mi = 0; mi < GB; ++mi) {
                se[mi] = 0.f;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) se[mi] += (ok[nb] && hi == 0) ? __expf(dot[m0 + mi][nb] - mx[mi]) : 0.f;
            }
#pragma unroll
            for (int mi = 0; mi < GB; ++mi) se[mi] = wave_sum(se[mi]);
            if (lane == 0) {
#pragma unroll
                for (int mi = 0; mi < GB; ++mi) sStat[hh][tg][m0 + mi] = make_float2(mx[mi], se[mi]);
            }
        }
    }
    if (partial) return;  // uniform
    __syncthreads();
    // the waves' statistics, merged in wave order: those of a head, or (MULTI) of a sequence, whose single tile this is
    constexpr int WS = MULTI ? 64 / WT : NTG;  // waves to merge
    if (tid < (MULTI ? SQ : HEADS) * G) {
        const int u = idiv(tid, G), m = tid - u * G, bt = MULTI ? b + u : b, h2 = MULTI ? 0 : u;
        float2 st = sStat[h2][MULTI ? u * WS : 0][m];
#pragma unroll
        for (int t = 1; t < WS; ++t) st = stat_merge(st, sStat[h2][(MULTI ? u * WS : 0) + t][m]);
        if (!MULTI || bt < B) stats[((size_t)bt * H + (size_t)(g0 + h2) * G + m) * stats_stride + part] = st;
    }
}

#define SALS_LG_ARGS                                                                                                     \
    const T *__restrict__ Kc, const T *__restrict__ UkP, const int32_t *__restrict__ idx, const int32_t *__restrict__ n_sel, \
        const T *__restrict__ q, const int32_t *__restrict__ q_pos, const float2 *__restrict__ rope, InvFreq inv,         \
        float *__restrict__ logits, float2 *__restrict__ stats, int B, int S_max, int r, int H, int H_kv, int k_tot,      \
        int lk, int n_parts, int heads_fastest, int style, float scale, int ring, int stats_stride,                       \
        float *__restrict__ plogits, int ksplit
template <typename T, int HEADS, int NTG, int NB, int GB, int GFIX, bool MULTI = false>
__global__ __launch_bounds__(64 * HEADS * NTG, HEADS * NTG >= 8 ? 2 : 1) void attend_logits_kernel(SALS_LG_ARGS)
{
    logits_tile<T, HEADS, NTG, NB, GB, GFIX, MULTI, false, false, false>((int)blockIdx.x, Kc, UkP, idx, n_sel, q, q_pos, rope, inv, logits, stats,
                                                                  B, S_max, r, H, H_kv, k_tot, lk, n_parts, heads_fastest, style, scale,
                                                                  ring, stats_stride, plogits, ksplit, WindowByLength{}, SplitLogits{},
                                                                  TopkResolve{});
}
// with another pass's split logits on the side
template <typename T, int HEADS, int NTG, int NB, int GB, int GFIX>
__global__ __launch_bounds__(64 * HEADS * NTG, HEADS * NTG >= 8 ? 2 : 1) void attend_logits_side_kernel(SALS_LG_ARGS, SplitLogits split)
{
    logits_tile<T, HEADS, NTG, NB, GB, GFIX, false, false, true, false>((int)blockIdx.x, Kc, UkP, idx, n_sel, q, q_pos, rope, inv, logits, stats,
                                                                 B, S_max, r, H, H_kv, k_tot, lk, n_parts, heads_fastest, style, scale,
                                                                 ring, stats_stride, plogits, ksplit, WindowByLength{}, split,
                                                                 TopkResolve{});
}
// on a selection whose threshold bin is still to be ranked
template <typename T, int HEADS, int NTG, int NB, int GB, int GFIX>
__global__ __launch_bounds__(64 * HEADS * NTG, HEADS * NTG >= 8 ? 2 : 1) void attend_logits_resolve_kernel(SALS_LG_ARGS, TopkResolve res)
{
    logits_tile<T, HEADS, NTG, NB, GB, GFIX, false, false, false, true>((int)blockIdx.x, Kc, UkP, idx, n_sel, q, q_pos, rope, inv, logits,
                                                                        stats, B, S_max, r, H, H_kv, k_tot, lk, n_parts, heads_fastest,
                                                                        style, scale, ring, stats_stride, plogits, ksplit,
                                                                        WindowByLength{}, SplitLogits{}, res);
}
#undef SALS_LG_ARGS

}  // namespace sals
