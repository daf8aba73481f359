// Prefill-time bulk compression (Eq. 1; Algorithm 1, projection and append steps, applied to a whole
// prompt at once):  K~ = K U_k,  V~ = V U_v  for n_tok new tokens per sequence, written to the
// cache rows seq_len[b] .. seq_len[b] + n_new[b] - 1.
//
// A plain GEMM on the matrix cores, [tokens x D_kv] . [D_kv x r], both operands read along their contiguous axis: the token
// rows as they lie in memory and the TRANSPOSED projector U^T [r x D_kv] (section 0 / 1 of the packed weights, the same rows
// the one-token projection reads).  fp32 accumulation, one rounding to the storage type at the store, so a row equals the
// one-token projection of the same token up to the order of the fp32 sum.
//   prefill_tile_kernel       bf16: both operands straight into LDS, tiles of up to 256 x 320, a list of tiles over the batch
//   prefill_compress_kernel   fp32: operands staged through registers, tiles of up to 256 x 128 of one sequence; also the
//                             symmetric product of the calibration for fp32 keys
#pragma once
#include <type_traits>

#include "common.hpp"
#include "k_attend.hpp"
#include "k_gemm.hpp"
#include "k_logits.hpp"

namespace sals {

constexpr int kPfThreads = 512;
constexpr size_t prefill_lds_bytes(int tok, int nl) { return 3 * (size_t)(tok + nl) * kLgStep; }

struct PrefillArgs {
    const void* X[2];        // new keys / values [B, n_tok, D]
    const void* UT[2];       // transposed projectors [r, D]
    void* cache[2];          // [B, S_max, r]
    const int32_t* seq_len;  // [B] first row to write
    const int32_t* n_new;    // [B] tokens of each sequence (<= n_tok), or nullptr: n_tok everywhere
    int n_tok, D, r, S_max, B, nproj;
    uint32_t* arrived;       // not null: the last of the launch's n_wg workgroups to arrive here advances the lengths
    uint32_t n_wg;
    float* pacc;             // SYRK form only: [slices][n_tok, r] fp32 tile sums of each slice of the contraction axis
    int kslice_steps;        // SYRK form only: 64-byte steps of the contraction axis per slice (blockIdx.y = slice)
};

// a sequence's length behind the prompt
__device__ __forceinline__ void pf_advance(int32_t* seq_len, const int32_t* n_new, int n_tok, int b, int S_max)
{
    const int n = n_new ? min(max(n_new[b], 0), n_tok) : n_tok;
    const int s = seq_len[b];
    if (s >= 0) seq_len[b] = (int)min((long long)s + n, (long long)S_max);
}
// thread 0 of a workgroup arrives behind every read of the lengths; the last workgroup advances them before it ends (6 ragged prompts
// of up to 4001 tokens, D = 1024, r = 640 62.9 us a call with a launch for that behind the stores, 61.8 so)
__device__ __forceinline__ uint32_t pf_arrive(const PrefillArgs& a) { return a.arrived && threadIdx.x == 0 ? arrive(a.arrived, a.n_wg) : 0u; }
__device__ __forceinline__ void pf_leave(const PrefillArgs& a, uint32_t order)
{
    if (!a.arrived || threadIdx.x >= kWave || (uint32_t)wave_uniform((int)order) != a.n_wg - 1) return;
    for (int b = lane_id(); b < a.B; b += kWave) pf_advance(const_cast<int32_t*>(a.seq_len), a.n_new, a.n_tok, b, a.S_max);
}

// fp32 prompts.  One workgroup owns TOK tokens x NL latent coordinates of one sequence and one projection; its eight waves
// are 4 token groups x 2 latent groups (NL = 128) or 8 token groups (NL = 64), a wave tile being TOK/4 (TOK/8) tokens x 64
// latent coordinates.  TOK = 256, or 128 when the larger tile would leave most of the chip without a workgroup.  Both operand
// tiles walk the D axis in 64-byte steps through three swizzled LDS stages: the fragments of the next half step are read
// under the MFMAs of the current one, and the step after next moves from registers to the third stage.  Bound by the fp32
// matrix instructions.
//
// SYRK: the same tiles and pipeline as a plain product of two row-major operands, out[t, l] = sum_c X[t, c] UT[l, c],
// whose fp32 tile sums are stored as they are instead of becoming cache rows (the covariance of the offline
// calibration, Sec. 4.2, with X = UT = the transposed keys and c running over the calibration tokens).  The
// contraction axis is cut into slices (blockIdx.y), each with its own output matrix, so that narrow matrices still
// fill the chip; a second kernel adds the slices to the fp64 covariance.
template <int TOK, int NL, bool SYRK = false>
__global__ __launch_bounds__(kPfThreads, 2) void prefill_compress_kernel(PrefillArgs a)
{
    typedef float T;
    static_assert((NL == 128 || NL == 64) && (TOK == 256 || (TOK == 128 && NL == 128)), "tile");
    constexpr int kPfTok = TOK;
    constexpr int ES = (int)sizeof(T);
    constexpr int WN = NL / 64;                 // latent groups of 64 among the waves
    constexpr int WM = 8 / WN;                  // token groups
    constexpr int MB = kPfTok / WM / 32;        // 32-token MFMA blocks per wave: 2 | 1
    constexpr int A_BYTES = kPfTok * kLgStep, B_BYTES = NL * kLgStep, STAGE = A_BYTES + B_BYTES;
    constexpr int NA = A_BYTES / 16 / kPfThreads;                       // 2
    constexpr int NBP = (B_BYTES / 16 + kPfThreads - 1) / kPfThreads;   // 1
    constexpr bool kBAll = B_BYTES / 16 >= kPfThreads;                   // every thread has a piece of the B tile
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];  // [3][A | B]

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;
    const int b = blockIdx.z / a.nproj, proj = blockIdx.z - b * a.nproj;
    int tile_x = blockIdx.x, tile_y = blockIdx.y;
    if constexpr (SYRK) {
        // The result is symmetric: only the tiles that reach the upper triangle (column tile >= row tile, in units of
        // NL columns) are computed, the rest is mirrored afterwards.  blockIdx.x numbers those tiles row by row.
        constexpr int RPT = kPfTok / NL;                // column tiles a row tile spans: 2 | 1
        const int ncol = a.r / NL;
        int id = blockIdx.x, row = 0;
        while (id >= ncol - row * RPT) { id -= ncol - row * RPT; ++row; }   // (at most n_tok / TOK rounds, uniform)
        tile_x = row; tile_y = row * RPT + id;
    }
    const int tok0 = tile_x * kPfTok, lat0 = tile_y * NL;
    const int n_b = (!SYRK && a.n_new) ? min(max(ld_uniform_i32(a.n_new + b), 0), a.n_tok) : a.n_tok;
    const int row0_v = SYRK ? 0 : ld_uniform_i32(a.seq_len + b);
    const T* X = static_cast<const T*>(a.X[proj]) + (size_t)b * a.n_tok * a.D;
    const T* UT = static_cast<const T*>(a.UT[proj]);

    // global sources of this thread's 16-byte pieces: piece q -> row q/4, column q%4 of the tile
    const unsigned char* a_src[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = tid + i * kPfThreads;
        const int t = min(tok0 + (q >> 2), a.n_tok - 1);  // rows past the prompt re-read its last token; never stored
        a_src[i] = reinterpret_cast<const unsigned char*>(X + (size_t)t * a.D) + (q & 3) * 16;
    }
    const unsigned char* b_src;
    {
        const int q = kBAll ? tid : (tid & (B_BYTES / 16 - 1));
        b_src = reinterpret_cast<const unsigned char*>(UT + (size_t)(lat0 + (q >> 2)) * a.D) + (q & 3) * 16;
    }
    auto a_dst = [&](int i) { const int q = tid + i * kPfThreads; return swz64(q >> 2, q & 3); };
    const int b_dst = A_BYTES + swz64((tid & (B_BYTES / 16 - 1)) >> 2, tid & 3);
    const bool b_mine = kBAll || tid < B_BYTES / 16;

    f32x16 acc[MB][2];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;

    const int nkc_all = a.D * ES / kLgStep;
    const int kc_base = SYRK ? (int)blockIdx.y * a.kslice_steps : 0;
    const int nkc = SYRK ? min(a.kslice_steps, nkc_all - kc_base) : nkc_all;  // (the host gives every slice >= 1 step)
    struct Regs { u32x4 a[NA]; u32x4 b[NBP]; };
    auto g_load = [&](Regs& R, int kc) {
#pragma unroll
        for (int i = 0; i < NA; ++i) R.a[i] = ld16(a_src[i] + (size_t)(kc_base + kc) * kLgStep);
        R.b[0] = ld16(b_src + (size_t)(kc_base + kc) * kLgStep);
    };
    auto l_store = [&](const Regs& R, int buf) {
        unsigned char* base = lds + (size_t)buf * STAGE;
#pragma unroll
        for (int i = 0; i < NA; ++i) *reinterpret_cast<u32x4*>(base + a_dst(i)) = R.a[i];
        if (b_mine) *reinterpret_cast<u32x4*>(base + b_dst) = R.b[0];
    };
    struct Frags { u32x4 a[MB]; u32x4 b[2]; };
    auto read_frags = [&](Frags& F, int buf, int ks) {
        const unsigned char* pa = lds + (size_t)buf * STAGE + wm * MB * 32 * kLgStep;
        const unsigned char* pb = lds + (size_t)buf * STAGE + A_BYTES + wn * 64 * kLgStep;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) F.a[mb] = *reinterpret_cast<const u32x4*>(pa + swz64(mb * 32 + l32, ks * 2 + hi));
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) F.b[nb] = *reinterpret_cast<const u32x4*>(pb + swz64(nb * 32 + l32, ks * 2 + hi));
    };
    auto mma_frags = [&](const Frags& F) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) mma_op<T>::run(F.a[mb], F.b[nb], acc[mb][nb]);
    };

    {
        Regs R, R1;
        Frags F0, F1;
        g_load(R, 0);
        g_load(R1, min(1, nkc - 1));
        l_store(R, 0);
        l_store(R1, 1);
        g_load(R, min(2, nkc - 1));
        __syncthreads();
        read_frags(F0, 0, 0);
        int cur = 0, nxt = 1, third = 2;  // stage of step kc, kc+1, kc+2
        for (int kc = 0; kc < nkc; ++kc) {
            read_frags(F1, cur, 1);
            mma_frags(F0);
            l_store(R, third);                       // step kc+2 (a copy of the last step past the end)
            g_load(R, min(kc + 3, nkc - 1));
            read_frags(F0, nxt, 0);
            mma_frags(F1);
            __syncthreads();
            const int t = cur; cur = nxt; nxt = third; third = t;
        }
    }

    // acc[mb][nb][4a+c] is token wm*MB*32 + mb*32 + 8a + 4hi + c of the tile, latent coordinate wn*64 + nb*32 + l32:
    // for fixed (a, c) the 32 lanes of a half wave write 32 consecutive elements of one cache row
    if constexpr (SYRK) {
        float* pout = a.pacc + (size_t)blockIdx.y * a.n_tok * a.r;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = tok0 + (wm * MB + mb) * 32 + (v >> 2) * 8 + hi * 4 + (v & 3);
                if (t < n_b) {
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) pout[(size_t)t * a.r + lat0 + wn * 64 + nb * 32 + l32] = acc[mb][nb][v];
                }
            }
        return;
    }
    const int row0 = wave_uniform(row0_v);
    const uint32_t order = pf_arrive(a);  // (every wave's length came before its last operands)
    T* cache = static_cast<T*>(a.cache[proj]) + (size_t)b * a.S_max * a.r;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int t = tok0 + (wm * MB + mb) * 32 + (v >> 2) * 8 + hi * 4 + (v & 3);
            const long long row = (long long)row0 + t;
            if (t < n_b && row0 >= 0 && row < a.S_max) {
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    cache[(size_t)row * a.r + lat0 + wn * 64 + nb * 32 + l32] = acc[mb][nb][v];
            }
        }
    pf_leave(a, order);
}

// bf16 prompts: tiles of 128 NBT tokens x 64 NBW latent coordinates (NBT 1 | 2, NBW 1 .. 5), one workgroup per compute unit.
// Both operands come straight from memory into LDS (64-byte steps of the D axis, four stages, 16-byte pieces at their index
// XOR row bits) and eight waves of 32 NBT tokens x 32 NBW coordinates read the next half step's fragments under the current
// one's MFMAs, one barrier per step.  The latent coordinates are the MFMA's rows, so a lane ends up with four consecutive
// coordinates of a token; the stores go through LDS.
// Matrix-bound while the whole chip works (22 ns per MFMA and SIMD at the clock its power leaves, 13.4 with few workgroups);
// what is lost to it is the last round of tiles and 2 (smallest tile) to about 9 us (largest) per round to start and store.  Whole
// calls, with the launch that advances the lengths, against the 256 x 128 and 128 x 128 tiles staged through registers, two
// workgroups per compute unit, that this replaced: 6 ragged prompts of up to 4001 tokens, D = 1024, r = 640 91 -> 78 us;
// 6000 tokens, D = 4096, r = 1024 125 -> 99 us; 64 tokens, D = 4096 44 -> 20 us.
// Tiles: without n_new the prompts of a batch are one run of B n_tok rows (a tile may span sequences); with n_new every
// sequence has tiles of its own and only those that hold tokens are in the list (its length is known on the device only, so
// the launch covers n_tok everywhere and the workgroups past the end leave at once).
// All tiles alike, or two kinds in a launch (prefill_split_kernel): the first workgroups (kPfBig) as many 256-row tiles as fill
// whole rounds of the chip with per_big workgroups each, the others (kPfTail) the rest in smaller tiles, unless that rest is more
// than tail_max row tiles (then the first take them too).  Both derive the split from the token counts.  The smaller tiles start
// as the compute units get free.  Whole calls and the copy that sets the lengths back, on one card, with the smaller tiles in a
// launch of their own behind the last of the whole ones and as here: 6 ragged prompts of up to 4001 tokens (D = 1024, r = 640)
// 74.5 and 71.7 us, 1 x 20000 74.5 and 72.4, 4097 tokens of D = 4096, r = 1024 102.1 and 99.0.
enum { kPfAll = 0, kPfBig = 1, kPfTail = 2 };
struct PfPart { int part, per_big, tail_max; };
template <int NBW, int NBT> struct pf_cfg {
    static constexpr int TN = 64 * NBW, TM = 128 * NBT;
    static constexpr int A_BYTES = TN * kLgStep, B_BYTES = TM * kLgStep, STAGE = A_BYTES + B_BYTES;
    static constexpr size_t LDS = 4 * (size_t)STAGE;
    static constexpr int PIECES = TN / 16;   // 1 KB pieces of the projector side per step
};
// (returns thread 0's arrival, see pf_arrive)
template <int NBW, int NBT>
__device__ __forceinline__ uint32_t prefill_tile(const PrefillArgs& a, int block, int n_col, const PfPart& p)
{
    typedef pf_cfg<NBW, NBT> C;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];  // [stage][projector rows | token rows]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;   // token group, latent group

    // ---- work list: (token tile, projection, latent tile), latent tile fastest; each XCD takes a run of it
    const int per_tile = 2 * n_col;
    int m0, m_end, proj, col;   // first row of the tile and end of its rows, in the run of B n_tok rows
    {
        const int unit = p.part == kPfAll ? C::TM : 256;   // rows the list counts in
        int n_tiles, t0v = 0, t1v = 0, c0 = 0, c1 = 0;
        if (a.n_new) {
            const int n0 = lane < a.B ? min(max(a.n_new[lane], 0), a.n_tok) : 0;
            const int n1 = lane + 64 < a.B ? min(max(a.n_new[lane + 64], 0), a.n_tok) : 0;
            t0v = (n0 + unit - 1) / unit; t1v = (n1 + unit - 1) / unit;
            c0 = (int)wave_incl_scan((uint32_t)t0v);
            c1 = (int)wave_incl_scan((uint32_t)t1v) + __builtin_amdgcn_readlane(c0, 63);
            n_tiles = __builtin_amdgcn_readlane(c1, 63);
        } else {
            n_tiles = (a.B * a.n_tok + unit - 1) / unit;
        }
        // the first launch of two takes whole rounds of the chip, the second one what is left, in its smaller tiles
        constexpr int SUB = 256 / C::TM;
        int first = 0, count = n_tiles;
        if (p.part != kPfAll) {
            int whole = n_tiles * p.per_big / 256 * 256 / p.per_big;
            if (n_tiles - whole > p.tail_max) whole = n_tiles;
            first = p.part == kPfTail ? whole : 0;
            count = p.part == kPfTail ? (n_tiles - whole) * SUB : whole;
        }
        const int total = count * per_tile;
        if (block >= total) return pf_arrive(a);  // uniform
        const int w = xcd_item(block, total);
        int tile = idiv(w, per_tile);
        const int rest = w - tile * per_tile;
        proj = idiv(rest, n_col); col = rest - proj * n_col;
        int sub = 0;
        if (p.part == kPfTail) { sub = (tile % SUB) * C::TM; tile = first + tile / SUB; }
        if (a.n_new) {  // the sequence whose tiles include this one
            const int b = __popcll(__ballot(lane < a.B && c0 <= tile)) + __popcll(__ballot(lane + 64 < a.B && c1 <= tile));
            const int l = b & 63;
            const int end = b < 64 ? __builtin_amdgcn_readlane(c0, l) : __builtin_amdgcn_readlane(c1, l);
            const int mine = b < 64 ? __builtin_amdgcn_readlane(t0v, l) : __builtin_amdgcn_readlane(t1v, l);
            const int n_b = min(max(a.n_new[b], 0), a.n_tok);
            m0 = b * a.n_tok + (tile - (end - mine)) * unit + sub;
            m_end = b * a.n_tok + n_b;
        } else {
            m0 = tile * unit + sub;
            m_end = a.B * a.n_tok;
        }
        if (m0 >= m_end) return pf_arrive(a);  // uniform: an empty part of a sequence's last tile
    }
    const int lat0 = col * C::TN;
    const size_t row_bytes = (size_t)a.D * 2;
    const unsigned char* X = static_cast<const unsigned char*>(a.X[proj]) + (size_t)m0 * row_bytes;
    const unsigned char* U = static_cast<const unsigned char*>(a.UT[proj]) + (size_t)lat0 * row_bytes;

    // this wave's 1 KB pieces (16 rows of 64 bytes) of a step: projector side wave, wave + 8, wave + 16, token side wave,
    // wave + 8.  Lane -> row lane / 4, position lane % 4; rows past the end re-read the last one and are never stored
    const uint32_t lds0 = lds_offset(lds);
    const int prow = lane >> 2, ppos = lane & 3;
    constexpr int NU = (C::PIECES + 7) / 8, NL = NU + NBT;   // loads of a wave per step
    uint32_t u_off[NU], x_off[NBT];
#pragma unroll
    for (int i = 0; i < NU; ++i) {
        const int row = (wave + 8 * i) * 16 + prow;
        u_off[i] = (uint32_t)min(row, a.r - 1 - lat0) * (uint32_t)row_bytes + (uint32_t)((ppos ^ ((row >> 2) & 3)) << 4);
    }
#pragma unroll
    for (int i = 0; i < NBT; ++i) {
        const int row = (wave + 8 * i) * 16 + prow;
        x_off[i] = (uint32_t)min(row, m_end - 1 - m0) * (uint32_t)row_bytes + (uint32_t)((ppos ^ ((row >> 2) & 3)) << 4);
    }
    const bool last_u = wave + 8 * (NU - 1) < C::PIECES;   // (uniform) this wave has the last of its projector pieces
    const int n_steps = a.D / 32;
    // load i of a step: token pieces, then projector pieces
    auto load_piece = [&](int i, int step, int stage) {
        const size_t at = (size_t)min(step, n_steps - 1) * kLgStep;  // (past the end: a step that nothing reads any more)
        const uint32_t st = lds0 + (uint32_t)stage * C::STAGE;
        if (i < NBT) load_lds16(X + at, x_off[i], st + C::A_BYTES + (wave + 8 * i) * 1024);
        else if (i + 1 < NL || last_u) load_lds16(U + at, u_off[i - NBT], st + (wave + 8 * (i - NBT)) * 1024);
    };
    auto load_step = [&](int step, int stage) {
#pragma unroll
        for (int i = 0; i < NL; ++i) load_piece(i, step, stage);
    };
    // waits until all but the newest K steps of this wave's loads have landed
    auto wait_but = [&](auto k) {
        constexpr int K = decltype(k)::value;
        if (last_u) vm_wait<K * NL>(); else vm_wait<K * (NL - 1)>();
    };

    f32x16 acc[NBW][NBT];
#pragma unroll
    for (int mb = 0; mb < NBW; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBT; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;
    // fragment addresses: row l32 of a 32-row block, 16-byte piece 2 ks + hi (the row bits of the XOR do not depend on the
    // block, whose rows start at a multiple of 32)
    const uint32_t at[2] = {(uint32_t)swz64(l32, hi), (uint32_t)swz64(l32, 2 + hi)};
    struct Frags { u32x4 a[NBW], b[NBT]; };
    const unsigned char* pa = lds + wn * NBW * 32 * kLgStep;
    const unsigned char* pb = lds + C::A_BYTES + wm * NBT * 32 * kLgStep;
    auto read_frag = [&](Frags& F, int i, int stage, int ks) {
        if (i < NBT) F.b[i] = *reinterpret_cast<const u32x4*>(pb + at[ks] + stage * C::STAGE + i * 32 * kLgStep);
        else F.a[i - NBT] = *reinterpret_cast<const u32x4*>(pa + at[ks] + stage * C::STAGE + (i - NBT) * 32 * kLgStep);
    };
    // One half step, in this order: the MFMAs of `F`, between them the reads of the next half step's fragments into `N` and
    // half of this wave's share of a later step's loads.  A load is held at issue while the path from the L2 is busy, so
    // loads issued together in front of the MFMAs would keep the matrix cores waiting (10 % at D = 4096).
    auto half_step = [&](const Frags& F, Frags& N, int n_stage, int n_ks, int step, int stage, auto half) {
        constexpr int NM = NBT * NBW, NR = NBW + NBT, H = decltype(half)::value, L0 = H ? (NL + 1) / 2 : 0, L1 = H ? NL : (NL + 1) / 2;
#pragma unroll
        for (int j = 0; j < NM; ++j) {
            mma_op<bf16_t>::run(F.a[j / NBT], F.b[j % NBT], acc[j / NBT][j % NBT]);
#pragma unroll
            for (int i = j * NR / NM; i < (j + 1) * NR / NM; ++i) read_frag(N, i, n_stage, n_ks);
#pragma unroll
            for (int i = L0 + j * (L1 - L0) / NM; i < L0 + (j + 1) * (L1 - L0) / NM; ++i) load_piece(i, step, stage);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    load_step(0, 0); load_step(1, 1); load_step(2, 2);
    // cache rows of this lane's tokens (null: not stored), found while the first loads are in flight
    unsigned char* dst[NBT];
#pragma unroll
    for (int nb = 0; nb < NBT; ++nb) {
        const int m = m0 + (wm * NBT + nb) * 32 + l32;
        const int mc = min(m, m_end - 1), b = (unsigned)mc / (unsigned)a.n_tok, t = mc - b * a.n_tok;
        const int row0 = a.seq_len[b];
        const long long row = (long long)row0 + t;
        const bool ok = m < m_end && row0 >= 0 && row < a.S_max;
        dst[nb] = ok ? static_cast<unsigned char*>(a.cache[proj]) + ((size_t)b * a.S_max + (size_t)row) * a.r * 2 : nullptr;
    }
    wait_but(std::integral_constant<int, 2>{});
    wg_barrier();
    Frags F0, F1;
#pragma unroll
    for (int i = 0; i < NBW + NBT; ++i) read_frag(F0, i, 0, 0);
    // In the smallest tiles a step is so short that it is felt where the loop lies in the lines of the instruction cache (64 tokens,
    // D = 4096, r = 1024: 20.5 us a call at the start of a line, 21.1 elsewhere; 200 tokens, r = 512: 21.1 and 21.6).  Aligned here,
    // with room for the instructions that the compiler puts in front of the loop (24 bytes and whole lines): a loop alignment given
    // to the compiler is not observed, so a test looks where the loop of the built library lies.
    if constexpr (NBW == 1 && NBT == 1)
        asm volatile(".p2align 6\n s_nop 0\n s_nop 0\n s_nop 0\n s_nop 0\n s_nop 0\n s_nop 0\n s_nop 0\n s_nop 0\n s_nop 0\n s_nop 0");
    for (int s0 = 0; s0 < n_steps; s0 += 4) {  // (n_steps is a multiple of 4)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // steps up to s + 1 have landed, everywhere; every wave is done with step s - 1
            wait_but(std::integral_constant<int, 1>{});
            wg_barrier();
            half_step(F0, F1, u, 1, s0 + u + 3, (u + 3) & 3, std::integral_constant<int, 0>{});
            half_step(F1, F0, (u + 1) & 3, 0, s0 + u + 3, (u + 3) & 3, std::integral_constant<int, 1>{});
        }
    }
    vm_wait<0>();  // (no load may land in LDS that another workgroup has been given, nor in the rows below)
    wg_barrier();
    const uint32_t order = pf_arrive(a);

    // acc[mb][nb][4a+c]: latent coordinate wn 32 NBW + mb 32 + 8a + 4hi + c, token wm 32 NBT + nb 32 + l32.  A wave turns 32 tokens at
    // a time in rows of its own in LDS (its coordinates of a token, the token's cache row behind them), so that consecutive lanes
    // store consecutive 16-byte pieces of a cache row.  Stored as they lie, 8 bytes a lane, every store reached 32 rows: whole calls
    // and the copy that sets the lengths back, before and now, 6 ragged prompts of up to 4001 tokens (D = 1024, r = 640) 68.6 and 61.6
    // us, 1 x 20000 70.7 and 62.8, 1 x 6000 (D = 4096, r = 1024) 98.0 and 96.0, 64 tokens 20.6 and 20.5.  The stores are whole lines that
    // nothing reads soon, so the caches are told not to keep them: inputs that change from call to call 67.3 -> 62.8, 1 x 6000 96.0 ->
    // 92.9 (8-byte stores with that hint: twice the time).
    constexpr int ROW = NBW * 64 + 16, PPR = NBW * 4;   // bytes and pieces of a row
    static_assert(8 * 32 * ROW <= (int)C::LDS, "rows of eight waves");
    unsigned char* rows = lds + wave * (32 * ROW);
    const int lat_w = lat0 + wn * NBW * 32;
#pragma unroll
    for (int nb = 0; nb < NBT; ++nb) {
#pragma unroll
        for (int mb = 0; mb < NBW; ++mb)
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                uint2 w;
                w.x = (uint32_t)f32_to_bf16(acc[mb][nb][v]) | ((uint32_t)f32_to_bf16(acc[mb][nb][v + 1]) << 16);
                w.y = (uint32_t)f32_to_bf16(acc[mb][nb][v + 2]) | ((uint32_t)f32_to_bf16(acc[mb][nb][v + 3]) << 16);
                *reinterpret_cast<uint2*>(rows + l32 * ROW + (mb * 32 + 2 * v + hi * 4) * 2) = w;
            }
        if (hi == 0) *reinterpret_cast<unsigned char**>(rows + l32 * ROW + NBW * 64) = dst[nb];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < PPR / 2; ++i) {
            const int q = i * 64 + lane, t = (unsigned)q / PPR, pc = q - t * PPR;
            unsigned char* const to = *reinterpret_cast<unsigned char* const*>(rows + t * ROW + NBW * 64);
            const u32x4 w = *reinterpret_cast<const u32x4*>(rows + t * ROW + pc * 16);
            // (r is a multiple of 64, so of the pieces' coordinates)
            if (to && lat_w + pc * 8 < a.r) __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(to + (size_t)(lat_w + pc * 8) * 2));
        }
        __builtin_amdgcn_wave_barrier();
    }
    return order;
}

template <int NBW, int NBT>
__global__ __launch_bounds__(kPfThreads, 2) void prefill_tile_kernel(PrefillArgs a, int n_col)
{
    pf_leave(a, prefill_tile<NBW, NBT>(a, (int)blockIdx.x, n_col, PfPart{kPfAll, 0, 0}));
}
// n_big workgroups for the whole rounds of tiles of 256 rows, the others for the rest in tiles of 128 rows x 64 UBW coordinates
template <int NBW, int UBW>
__global__ __launch_bounds__(kPfThreads, 2) void prefill_split_kernel(PrefillArgs a, int n_col, int n_big, int n_col_rest, int tail_max)
{
    const int per_big = 2 * n_col;
    uint32_t order;
    if ((int)blockIdx.x < n_big) order = prefill_tile<NBW, 2>(a, (int)blockIdx.x, n_col, PfPart{kPfBig, per_big, tail_max});
    else order = prefill_tile<UBW, 1>(a, (int)blockIdx.x - n_big, n_col_rest, PfPart{kPfTail, per_big, tail_max});
    pf_leave(a, order);
}

// after the prompt of a context without a count of arrivals (see arrival_count): advance the lengths
__global__ void advance_seq_len_kernel(int32_t* __restrict__ seq_len, const int32_t* __restrict__ n_new, int n_tok, int B,
                                       int S_max)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) pf_advance(seq_len, n_new, n_tok, b, S_max);
}

}  // namespace sals
