// C ABI of the SALS decode-step attention library: descriptor validation, workspace
// carving and kernel launches.  Every entry point only enqueues work on the caller's
// stream; nothing here allocates device memory or synchronises.
#include "../../include/sals.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "common.hpp"
#include "k_attend.hpp"
#include "k_calib.hpp"
#include "k_calib_all.hpp"
#include "k_dense.hpp"
#include "k_logits.hpp"
#include "k_logits_small.hpp"
#include "k_overlap.hpp"
#include "k_prefill.hpp"
#include "k_project.hpp"
#include "k_scores.hpp"
#include "k_topk.hpp"
#include "k_topk_multi.hpp"
#include "k_qvalue.hpp"
#include "k_value.hpp"
#include "k_window.hpp"
#include "host_block.hpp"
#include "polar_plan.hpp"

using namespace sals;

// Scratch of sals_latent_scores_noalloc: part of the device image, one copy per GPU.  In host code the
// name is only a handle for hipGetSymbolAddress; kernels are given the address looked up there.
static __device__ __align__(256) unsigned char scratch[SALS_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

struct Layout {  // byte offsets into the workspace
    size_t qt, ap_part, scores, idx, n_sel, n_lo, logits, plogits, stats, rope, tpart, qv_part, dn_part, tm_part, tm_hist, tm_meta, tm_cand, tm_srange, total;
    size_t arrived;              // 0: no room
    int lk;                      // logits row stride (floats)
    int max_parts;               // token tiles per head of the logits kernel, at most
    int pv_tok_per_wg, pv_ntr, pv_waves;  // value-sum token ranges, waves per workgroup (4 | 8)
    int qv_tok_per_wg, qv_ntr;   // quantised-value attention: token ranges
    int dn_chunks, dn_tok;       // dense baseline: token chunks per sequence (overlap score: tokens per chunk)
    int proj_np;                 // D-axis slices of the query projection
    int tm_chunks;               // chunks of the multi-workgroup selection (0: one workgroup per sequence)
    size_t w_section;            // elements per section of the packed weights
};


}  // namespace

struct ProfRecord { int kernel; hipEvent_t start, stop; };

// which logits kernel a context's shape gets: 1 = 2 heads x 256 tokens, 2 = 1 head x 128 tokens, 3 = 1 head x 64
// tokens (then: slices of the latent axis per tile, 128-byte steps loaded ahead); n_parts = token tiles per head
struct LogitsPlan { int pick, n_parts, ksplit, nst, forced = 0; };   // forced: slices that the tuning aid asks for

struct sals_ctx {
    sals_desc d;
    Layout L;
    unsigned char* ws;
    size_t ws_bytes;
    InvFreq inv;
    // launch shapes, fixed when the context is made (sals_create): nothing on the launch path reads the
    // environment, plans or sets kernel attributes
    LogitsPlan plan{3, 0, 1, 1};
    int score_rows = 16;         // cache rows per workgroup of the score kernel
    int score_stream = -1;       // read-once hint on the score kernel's cache loads: -1 by size, 0 / 1 forced (tuning aid)
    bool fuse_select = true;     // decode steps may select inside the logits kernel (tuning aid SALS_TUNE_FUSE_SELECT=0)
    // cos/sin table over the positions 0 .. S_max (in the workspace): 0 = not filled, 1 = fill enqueued on
    // rope_stream and marked by rope_ev, 2 = known to be complete
    int rope_state = 0;
    hipStream_t rope_stream = nullptr;
    hipEvent_t rope_ev = nullptr;
    bool lds_allowed = false;    // the logits kernels' dynamic-LDS attribute has been raised
    bool profiling = false;
    std::vector<ProfRecord> prof;
};

namespace {

const char* const kKernelNames[SALS_N_KERNELS] = {
    "project", "scores", "topk", "attend_logits", "attend_pv", "attend_out", "attend_qv", "dense_attend", "prefill"};

// Brackets one kernel launch with a pair of events while profiling is on.
struct ProfScope {
    sals_ctx* c;
    hipStream_t st;
    ProfRecord rec{};
    bool on;
    ProfScope(const sals_ctx* ctx, int kernel, hipStream_t s) : c(const_cast<sals_ctx*>(ctx)), st(s), on(ctx->profiling)
    {
        if (!on) return;
        rec.kernel = kernel;
        on = hipEventCreate(&rec.start) == hipSuccess;
        if (on && hipEventCreate(&rec.stop) != hipSuccess) { (void)hipEventDestroy(rec.start); on = false; }
        if (!on) return;
        try {
            c->prof.push_back(rec);
        } catch (const std::bad_alloc&) {  // (this launch is not timed)
            (void)hipEventDestroy(rec.start);
            (void)hipEventDestroy(rec.stop);
            on = false;
            return;
        }
        (void)hipEventRecord(rec.start, st);
    }
    ~ProfScope()
    {
        if (on) (void)hipEventRecord(rec.stop, st);
    }
};

sals_status validate(const sals_desc* d)
{
    if (!d) return SALS_ERR_INVALID_ARG;
    if (d->dtype != SALS_F32 && d->dtype != SALS_BF16) return SALS_ERR_INVALID_ARG;
    if (d->rope_style != SALS_ROPE_HALF && d->rope_style != SALS_ROPE_INTERLEAVED) return SALS_ERR_INVALID_ARG;
    if (d->B < 1 || d->S_max < 1 || d->H_q < 1 || d->H_kv < 1 || d->d < 2 || (d->d & 1)) return SALS_ERR_INVALID_ARG;
    if (d->H_q % d->H_kv != 0) return SALS_ERR_INVALID_ARG;
    if (d->r < 1 || d->r_score < 1 || d->r_score > d->r) return SALS_ERR_INVALID_ARG;
    if (d->top_k < 1 || d->n_recent < 0 || d->n_sink < 0) return SALS_ERR_INVALID_ARG;
    if (!(d->rope_theta > 0.f) || !std::isfinite(d->rope_theta)) return SALS_ERR_INVALID_ARG;
    // what the kernels cover
    if (d->d != kHeadDim) return SALS_ERR_UNSUPPORTED;
    if (d->r % 64 != 0 || d->r > 2048) return SALS_ERR_UNSUPPORTED;
    if (d->r_score % 8 != 0 || d->r_score > kScoreMaxR) return SALS_ERR_UNSUPPORTED;
    if (d->H_q / d->H_kv > kMaxGroup || d->H_q > kPvMaxHeads) return SALS_ERR_UNSUPPORTED;
    if (d->S_max > (1 << 20)) return SALS_ERR_UNSUPPORTED;  // the RoPE table takes 512 B per position
    if ((long long)d->B * (d->H_q / d->H_kv) > kProjMaxCols) return SALS_ERR_UNSUPPORTED;
    if ((long long)d->top_k + d->n_recent + d->n_sink > 65536) return SALS_ERR_UNSUPPORTED;
    return SALS_OK;
}

// KV heads per workgroup of the dense baseline: two where that makes 512-byte pieces (four were no better) and the stream is
// the bound.  fp32 rows of one head are 512 bytes already, and with four query heads per KV head the arithmetic wants the
// waves apart (batch 1, 65536 tokens, 8 KV heads: 54.9 us with one head, 60.0 with two).
inline int dense_heads(const sals_desc& d)
{
    return d.dtype == SALS_BF16 && d.H_q / d.H_kv < 4 && d.H_kv % 2 == 0 ? 2 : 1;
}

// Rows of an output projection workgroup: the (sequence, query head) pairs of a KV head, 1, 2, 4, 8 or 16 of them.
constexpr int kOutRows = 16;
int out_tile_rows(const sals_desc& d)
{
    int R = 1;
    while (R < kOutRows && R < d.B * (d.H_q / d.H_kv)) R *= 2;
    return R;
}

// `short_ranges`: fp32 value sums in ranges of one step of 64 tokens (otherwise of two), whose partial sums take more workspace.
Layout make_layout(const sals_desc& d, bool short_ranges = true)
{
    Layout L{};
    const int D = d.H_kv * d.d;
    const int k_tot = d.top_k + d.n_sink + d.n_recent;
    L.lk = ceil_div(k_tot, 128) * 128;  // whole steps of the value kernel (its last step may read up to the row end)
    L.w_section = (size_t)D * d.r;
    {   // query projection: slice the D axis until at least 160 workgroups stream U_k^T (measured: at r = 640 four
        // slices = 160 workgroups project as fast as eight, and the score kernel then adds four partial sums, not eight)
        int nks = D / (d.dtype == SALS_BF16 ? 32 : 16);
        int np = 1;
        while (np < kScoreMaxParts && (d.r / 16) * np < 160 && nks % (np * 2) == 0 && nks / (np * 2) >= 4) np *= 2;
        if (const char* e = std::getenv("SALS_TUNE_PROJ_NP")) { const int v = std::atoi(e); if (v >= 1 && v <= kScoreMaxParts && nks % v == 0) np = v; }  // tuning aid
        L.proj_np = np;
    }
    // value sum: split the selected tokens into ranges of whole 64-token steps (at least two steps, at most kPvMaxTok tokens) as
    // long as every workgroup still gets a CU of its own (measured: a few CUs with two workgroups set the kernel's duration)
    {
        int blocks = d.r / kPvCols;
        int want = std::min(std::max(1, 256 / (blocks * d.B)), kMaxRanges);
        int n_tr = std::max(1, std::min(want, ceil_div(k_tot, 2 * kPvTJ)));
        // fp32, if the workspace has room for it: ranges of one step, as far as the output projection still takes all ranges' sums
        // with one load (kOutRows lanes hold its rows, and further ranges of them).  128 tokens, r = 512, one sequence of 32 KV heads: 32.7
        // us a step with one range and 31.7 with two; past that line two loads cost more than the value sum gains: 4 sequences of 32
        // query and 8 KV heads, 256 tokens, r = 640 45.6 us with two ranges and 48.3 with four, 3 with 512 tokens 57.3 and 61.7.
        if (d.dtype == SALS_F32 && short_ranges)
            n_tr = std::max(n_tr, std::min(std::min(want, ceil_div(k_tot, kPvTJ)), kOutRows / out_tile_rows(d)));
        if (const char* e = std::getenv("SALS_TUNE_PV_RANGES")) n_tr = std::max(1, std::min(64, std::atoi(e)));  // tuning aid
        n_tr = std::max(n_tr, ceil_div(k_tot, kPvMaxTok));
        int tok = ceil_div(ceil_div(k_tot, n_tr), kPvTJ) * kPvTJ;
        // eight waves once each of them has two groups, in bf16 of 16 tokens (measured: 128 tokens are 0.5 us faster with four), in
        // fp32 of 8 (r = 640, one sequence: 192 tokens 6.5 us with eight and 7.2 with four, 64 tokens 4.8 and 4.6)
        L.pv_waves = tok >= (d.dtype == SALS_BF16 ? 4 : 2) * kPvTJ ? 8 : 4;
        if (const char* e = std::getenv("SALS_TUNE_PV_WAVES")) L.pv_waves = std::atoi(e) == 4 ? 4 : 8;  // tuning aid
        L.pv_tok_per_wg = tok;
        L.pv_ntr = ceil_div(k_tot, tok);
    }
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
    L.qt = take((size_t)L.proj_np * d.B * d.r * 4);
    L.ap_part = take((size_t)2 * kScoreMaxParts * d.B * d.r * 4);
    L.scores = take((size_t)d.B * d.S_max * 4);
    L.idx = take((size_t)d.B * k_tot * 4);
    L.n_sel = take((size_t)d.B * 4);
    L.n_lo = take((size_t)d.B * 4);                          // recent-window attention: tokens of the low-rank pass
    L.arrived = (size_t)d.B * 4 % kAlign ? L.n_lo + (size_t)d.B * 4 : 0;  // (in the padding, if there is any: see arrival_count)
    L.logits = take((size_t)d.B * d.H_q * L.lk * 4);
    // partial logits of the latent slices, for shapes with so few 64-token tiles that the latent axis is split too
    // (also for batches of short selections, whose multi-sequence tiles may split the latent axis)
    L.plogits = take((ceil_div(k_tot, kLsTok) * d.H_kv * d.B <= 128 || k_tot <= 64)
                         ? (size_t)kLsMaxSplit * d.B * d.H_q * L.lk * 4 : 0);
    L.max_parts = ceil_div(k_tot, 32) + 2;  // (room for the tiles of a recent-window pass beside the context's own)
    L.stats = take((size_t)d.B * d.H_q * L.max_parts * 8);
    L.rope = take((size_t)(d.S_max + 1) * kPairs * 8);  // positions 0 .. S_max (the query after a full cache)
    L.tpart = take((size_t)L.pv_ntr * d.B * d.H_q * d.r * 4);
    {   // quantised-value attention: one workgroup per (sequence, token range, KV head), 32 tokens side
        // by side; a second range (and with it the merge launch) only pays above ~32 tokens per slot
        int n_tr = k_tot <= 32 * kQvSlots ? 1 : std::min(kQvMaxRanges, ceil_div(k_tot, 16 * kQvSlots));
        if (const char* e = std::getenv("SALS_TUNE_QV_RANGES")) n_tr = std::max(1, std::min(kQvMaxRanges, std::atoi(e)));  // tuning aid
        n_tr = std::max(n_tr, ceil_div(k_tot, kQvMaxTok));
        L.qv_tok_per_wg = ceil_div(k_tot, n_tr);
        L.qv_ntr = ceil_div(k_tot, L.qv_tok_per_wg);
        L.qv_part = take((size_t)L.qv_ntr * d.B * d.H_q * kHeadDim * 4);
    }
    {   // dense baseline: token chunks (64 tokens at least) that make whole rounds of one workgroup per compute unit, or of two
        // where a key is shared by four query heads and more (then the arithmetic wants more waves) and in fp32 (a token at a
        // time per lane group), as few as do it well
        const int per = d.B * d.H_kv / dense_heads(d), target = d.dtype != SALS_BF16 || d.H_q / d.H_kv >= 4 ? 512 : 256;
        int n = 1;
        double best = 1e30;
        for (int k = 1; k <= std::min(kDnMaxChunks, std::max(1, d.S_max / 64)); ++k) {
            const double rounds = (double)k * per / target, cost = std::ceil(rounds) / rounds + 0.01 * k;
            if (cost < best) { best = cost; n = k; }
        }
        L.dn_tok = ceil_div(ceil_div(d.S_max, n), 16) * 16;
        L.dn_chunks = ceil_div(d.S_max, L.dn_tok);
        L.dn_part = take((size_t)d.B * d.H_q * L.dn_chunks * kDnRec * 4);
    }
    // Long sequences: selection spread over 8192-score chunks, from 32769 scores on, where topk_kernel's keys no longer fit in
    // registers: on its own the one launch takes 13.4 us at 32768 scores and 7.9 at 16384, the chain of four launches 17.9 and, at
    // 131072, 18.4.  In a decode step the chain has two launches (the score kernel leaves the ranges, the logits kernel ranks the
    // threshold bin), which beat the one launch from 16385 scores on (whole steps of 1 x (1024 of 32768), H_kv 32, r 1024 59.7
    // against 61.4 us), but order the list in another way; a step leaves the list that the selection call leaves, so both take the
    // same line.
    L.tm_chunks = d.S_max > 32768 ? ceil_div(d.S_max, kTmChunk) : 0;
    if (const int n = L.tm_chunks) {
        L.tm_part = take((size_t)d.B * n * sizeof(uint2));
        L.tm_hist = take((size_t)d.B * n * kTmRow * 4);
        L.tm_meta = take((size_t)d.B * sizeof(TopkMeta));
        L.tm_cand = take((size_t)d.B * kTmCand * sizeof(uint2));
        // key ranges the score kernel leaves per workgroup inside a decode step (at least 16 rows per workgroup)
        L.tm_srange = take((size_t)d.B * ceil_div(d.S_max, kScoreRowsPerIter) * sizeof(uint2));
    }
    L.total = o;
    return L;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool bad(const void* p) { return p == nullptr || !aligned16(p); }

inline sals_status launch_status()
{
    return hipGetLastError() == hipSuccess ? SALS_OK : SALS_ERR_HIP;
}

template <typename T> inline const T* w_section(const sals_ctx* c, const void* W, int sec)
{
    return static_cast<const T*>(W) + (size_t)sec * c->L.w_section;
}

// The count of arrivals of appends and prompt compressions, for a launch whose last workgroup advances the lengths in place of a
// second launch: calls of a context are ordered, so one is enough.  Cleared with the cos/sin table, so null until that is known to be
// filled (sals_prepare).  It lies in padding, of which batches of 64 and 128 sequences have none.
inline uint32_t* arrival_count(const sals_ctx* c) { return c->L.arrived ? reinterpret_cast<uint32_t*>(c->ws + c->L.arrived) : nullptr; }
inline uint32_t* arrivals(const sals_ctx* c) { return c->rope_state == 2 ? arrival_count(c) : nullptr; }

// q~ = U_k^T (summed query heads), as partial sums over slices of the D axis
template <typename T> sals_status launch_project(const sals_ctx* c, const void* W, const void* q, hipStream_t st)
{
    const sals_desc& d = c->d;
    ProjArgs a{};
    a.UT[0] = w_section<T>(c, W, 0);
    a.X[0] = q;
    a.out_f32 = reinterpret_cast<float*>(c->ws + c->L.qt);
    a.B = d.B; a.D = d.H_kv * d.d; a.r = d.r; a.H = d.H_q; a.H_kv = d.H_kv; a.d = d.d;
    a.S_max = d.S_max; a.nproj = 1; a.np = c->L.proj_np;
    ProfScope ps(c, SALS_K_PROJECT, st);
    const dim3 grid(d.r / 16, a.np), wg(kProjThreads);
    const int blocks = ceil_div(d.B * (d.H_q / d.H_kv), 16);
    if (blocks <= 1) hipLaunchKernelGGL((project_kernel<T, 1>), grid, wg, 0, st, a);
    else if (blocks <= 2) hipLaunchKernelGGL((project_kernel<T, 2>), grid, wg, 0, st, a);
    else if (blocks <= 4) hipLaunchKernelGGL((project_kernel<T, 4>), grid, wg, 0, st, a);
    else hipLaunchKernelGGL((project_kernel<T, 8>), grid, wg, 0, st, a);
    return launch_status();
}

// One token per sequence: k_new (and v_new, unless null) projected into cache0 (cache1), qa.bits > 0: its value quantised.
// `bump` advances the sequence lengths; ring > 0: the caches are rings of that many rows.
template <typename T>
sals_status launch_append(const sals_ctx* c, const void* W, const void* k_new, const void* v_new, void* cache0, void* cache1,
                          const QuantArgs& qa, int32_t* seq_len, hipStream_t st, bool bump, int ring = 0)
{
    const sals_desc& d = c->d;
    ProjArgs a{};
    a.UT[0] = w_section<T>(c, W, 0);
    a.UT[1] = w_section<T>(c, W, 1);
    a.X[0] = k_new; a.X[1] = v_new;
    a.cache[0] = cache0; a.cache[1] = cache1;
    a.seq_len = seq_len;
    a.B = d.B; a.D = d.H_kv * d.d; a.r = d.r; a.H = d.H_q; a.H_kv = d.H_kv; a.d = d.d;
    a.S_max = d.S_max; a.nproj = v_new ? 2 : 1;
    a.ring = ring;
    // An append that advances the lengths has a second launch anyway: it adds up slices of the D axis, as many (at most 8, of
    // 32 MFMA steps and more: shorter ones gain less than adding them up costs) as give the projection 128 workgroups.
    a.np = 1;
    a.out_f32 = reinterpret_cast<float*>(c->ws + c->L.ap_part);
    const int nks = a.D / (4 * elem<T>::vec);
    if (bump)
        while (a.np < kScoreMaxParts && d.r / 16 * a.nproj * a.np < 128 && nks % (2 * a.np) == 0 && nks / (2 * a.np) >= 32) a.np *= 2;
    const bool wide = nks / a.np > kProjWaves * kProjBatch;  // more MFMA steps than four waves request at once
    const int nw = wide ? kAppendWaves : kProjWaves;
    const dim3 grid(qa.bits ? std::max(d.r / 16, ceil_div(d.B * (a.D / kQvGroup), 2 * nw * a.np)) : d.r / 16, a.np, qa.bits ? 2 : a.nproj);
    a.arrived = bump && a.np == 1 ? arrivals(c) : nullptr;
    a.n_wg = grid.x * grid.y * grid.z;
    {
        ProfScope ps(c, SALS_K_PROJECT, st);
#define SALS_APPEND_H(NW, QUANT, HB) hipLaunchKernelGGL((append_kernel<T, NW, QUANT, HB>), grid, dim3(64 * NW), 0, st, a, qa)
#define SALS_APPEND(NW, QUANT)                                                                                           \
    do { if (d.B <= 16) SALS_APPEND_H(NW, QUANT, 1); else if (d.B <= 32) SALS_APPEND_H(NW, QUANT, 2);                    \
         else if (d.B <= 64 && NW == kProjWaves) SALS_APPEND_H(kProjWaves, QUANT, 4); else SALS_APPEND_H(NW, QUANT, 8); } while (0)
        if (qa.bits) { if (wide) SALS_APPEND(kAppendWaves, true); else SALS_APPEND(kProjWaves, true); }
        else { if (wide) SALS_APPEND(kAppendWaves, false); else SALS_APPEND(kProjWaves, false); }
#undef SALS_APPEND_H
#undef SALS_APPEND
    }
    if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    if (a.np > 1)
        hipLaunchKernelGGL((append_finish_kernel<T>), dim3(d.B), dim3(256), 0, st, a);
    else if (bump && !a.arrived)
        hipLaunchKernelGGL(bump_seq_len_kernel, dim3(ceil_div(d.B, 128)), dim3(128), 0, st, seq_len, d.B, d.S_max);
    return launch_status();
}

template <typename T>
// wg_range: where every workgroup leaves the key range of its scores (for the long-sequence selection of the same
// step), or nullptr
sals_status launch_scores(const sals_ctx* c, const void* Kc, const int32_t* seq_len, float* scores,
                          hipStream_t st, uint2* wg_range = nullptr)
{
    const sals_desc& d = c->d;
    constexpr int VEC = elem<T>::vec;
    const int nch = ceil_div(d.r_score / VEC, 16);
    const int rows = c->score_rows;
    dim3 grid(ceil_div(d.S_max, rows), d.B);
    const float* qt = reinterpret_cast<const float*>(c->ws + c->L.qt);
    const T* K = static_cast<const T*>(Kc);
    // a cache prefix of 32 MB and more is read as a stream the caches need not keep; a smaller one with plain loads (it
    // may still be cached from the previous step)
    bool stream = (size_t)d.B * d.S_max * d.r_score * sizeof(T) >= ((size_t)32 << 20);
    if (c->score_stream >= 0) stream = c->score_stream != 0;
    ProfScope ps(c, SALS_K_SCORES, st);
#define SALS_SCORES_CASE(N)                                                                         \
    case N:                                                                                         \
        if (stream)                                                                                  \
            hipLaunchKernelGGL((scores_kernel<T, N, true>), grid, dim3(kScoreThreads), 0, st, K, qt,    \
                               c->L.proj_np, seq_len, scores, d.B, d.S_max, d.r, d.r_score, rows,       \
                               wg_range, d.n_sink, d.n_recent);                                                         \
        else                                                                                         \
            hipLaunchKernelGGL((scores_kernel<T, N, false>), grid, dim3(kScoreThreads), 0, st, K, qt,   \
                               c->L.proj_np, seq_len, scores, d.B, d.S_max, d.r, d.r_score, rows,       \
                               wg_range, d.n_sink, d.n_recent);                                                         \
        break;
    switch (nch) {
        SALS_SCORES_CASE(1) SALS_SCORES_CASE(2) SALS_SCORES_CASE(3) SALS_SCORES_CASE(4)
        SALS_SCORES_CASE(5) SALS_SCORES_CASE(6) SALS_SCORES_CASE(7) SALS_SCORES_CASE(8)
        SALS_SCORES_CASE(9) SALS_SCORES_CASE(10) SALS_SCORES_CASE(11) SALS_SCORES_CASE(12)
        SALS_SCORES_CASE(13) SALS_SCORES_CASE(14) SALS_SCORES_CASE(15) SALS_SCORES_CASE(16)
        default: return SALS_ERR_UNSUPPORTED;
    }
#undef SALS_SCORES_CASE
    return launch_status();
}

// whether a decode step ranks the threshold bin in its logits kernel (the shapes with tiles of 128 and 256 tokens)
bool step_resolves(const sals_ctx* c) { return c->L.tm_chunks > 0 && (c->plan.pick == 1 || c->plan.pick == 2) && c->fuse_select; }
TopkResolve topk_resolve(const sals_ctx* c, int32_t* idx)
{
    return TopkResolve{reinterpret_cast<const TopkMeta*>(c->ws + c->L.tm_meta), reinterpret_cast<const uint2*>(c->ws + c->L.tm_cand), idx,
                       c->d.n_sink, c->d.top_k};
}

// wl: also leave the recent-window lists (see WindowLists); by default none
// in_step: the scores were written by this context's score kernel in the same step, which left its workgroups'
// key ranges in the workspace (the chain then needs no range pass of its own); with step_resolves() the threshold bin is left to the
// logits kernel
sals_status launch_topk(const sals_ctx* c, const float* scores, const int32_t* seq_len, int32_t* idx,
                        int32_t* n_sel, hipStream_t st, WindowLists wl = WindowLists{nullptr, nullptr, nullptr, 0},
                        bool in_step = false)
{
    const sals_desc& d = c->d;
    dim3 grid(d.B), block(kTopkThreads);
    ProfScope ps(c, SALS_K_TOPK, st);
#define SALS_TOPK(F4)                                                                                \
    hipLaunchKernelGGL((topk_kernel<F4>), grid, block, 0, st, scores, seq_len, idx, n_sel, d.S_max, \
                       d.top_k, d.n_sink, d.n_recent)
    if (c->L.tm_chunks > 0) {
        const Layout& L = c->L;
        const int nc = L.tm_chunks;
        TopkMultiWs ws{};
        ws.part = reinterpret_cast<uint2*>(c->ws + L.tm_part); ws.hist = reinterpret_cast<uint32_t*>(c->ws + L.tm_hist);
        ws.meta = reinterpret_cast<TopkMeta*>(c->ws + L.tm_meta); ws.cand = reinterpret_cast<uint2*>(c->ws + L.tm_cand);
        ws.range = ws.part; ws.n_range = nc;
        dim3 cgrid(nc, d.B);
        if (in_step) {
            ws.range = reinterpret_cast<const uint2*>(c->ws + L.tm_srange);
            ws.n_range = ceil_div(d.S_max, c->score_rows);
        } else {
            hipLaunchKernelGGL(topk_range_kernel, cgrid, block, 0, st, scores, seq_len, d.S_max, nc, d.n_sink, d.n_recent, ws.part);
        }
        hipLaunchKernelGGL(topk_hist_kernel, cgrid, block, 0, st, scores, seq_len, ws.range, ws.n_range, d.S_max, nc, d.n_sink,
                           d.n_recent, ws.hist);
#define SALS_PLACE(LAST)                                                                                          \
    hipLaunchKernelGGL((topk_place_kernel<LAST>), cgrid, block, 0, st, scores, seq_len, ws.range, ws.hist, ws.n_range, d.S_max, nc, \
                       d.top_k, d.n_sink, d.n_recent, idx, ws.meta, ws.cand, n_sel, wl)
        if (in_step && step_resolves(c)) { SALS_PLACE(true); return launch_status(); }
        SALS_PLACE(false);
#undef SALS_PLACE
        hipLaunchKernelGGL(topk_finish_kernel, grid, block, 0, st, ws.cand, ws.meta, seq_len, d.S_max, d.top_k, d.n_sink,
                           d.n_recent, idx, n_sel, scores, wl);
        return launch_status();
    }
#define SALS_TOPK_W(F4)                                                                                    \
    hipLaunchKernelGGL((topk_window_kernel<F4>), grid, block, 0, st, scores, seq_len, idx, n_sel, d.S_max, \
                       d.top_k, d.n_sink, d.n_recent, wl)
    if (wl.idx_hi != nullptr) {
        if (d.S_max <= 4096) SALS_TOPK_W(1);
        else if (d.S_max <= 8192) SALS_TOPK_W(2);
        else if (d.S_max <= 16384) SALS_TOPK_W(4);
        else SALS_TOPK_W(8);
        return launch_status();
    }
#undef SALS_TOPK_W
    if (d.S_max <= 4096) SALS_TOPK(1);
    else if (d.S_max <= 8192) SALS_TOPK(2);
    else if (d.S_max <= 16384) SALS_TOPK(4);
    else SALS_TOPK(8);
#undef SALS_TOPK
    return launch_status();
}

// rows per workgroup of the score kernel: a multiple of 16 giving roughly 1024 workgroups, 16..64 rows
// (measured optimum; the first 16 rows of a workgroup are requested before the sequence length is known, so
// shorter ranges would pay more for the empty part of a cache)
int plan_score_rows(const sals_desc& d)
{
    long long total_rows = (long long)d.B * d.S_max;
    int rows = (int)std::min<long long>(64, std::max<long long>(16, total_rows / 1024));
    if (const char* e = std::getenv("SALS_TUNE_SCORE_ROWS")) rows = std::max(16, std::min(1 << 16, std::atoi(e)));  // tuning aid
    return ceil_div(rows, kScoreRowsPerIter) * kScoreRowsPerIter;
}

// Enqueues the fill of the context's cos/sin table on `st` and marks it with an event.
sals_status enqueue_rope_table(sals_ctx* c, hipStream_t st)
{
    const size_t n = (size_t)(c->d.S_max + 1) * kPairs;
    hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<float2*>(c->ws + c->L.rope), c->inv, c->d.S_max + 1, arrival_count(c));
    if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    if (!c->rope_ev && hipEventCreateWithFlags(&c->rope_ev, hipEventDisableTiming) != hipSuccess) return SALS_ERR_HIP;
    if (hipEventRecord(c->rope_ev, st) != hipSuccess) return SALS_ERR_HIP;
    c->rope_stream = st;
    c->rope_state = 1;
    return SALS_OK;
}

// Before a kernel that reads the cos/sin table is enqueued on `st`.  A prepared context (sals_prepare) costs one
// comparison.  Otherwise the fill is enqueued on first use and later calls are ordered behind it: same stream by
// stream order, another stream by waiting for the event.  A stream under graph capture needs a prepared context
// (a captured fill would not run before eager work, and events of other streams cannot be consulted there).
sals_status ensure_rope_table(const sals_ctx* cc, hipStream_t st)
{
    sals_ctx* c = const_cast<sals_ctx*>(cc);
    if (c->rope_state == 2) return SALS_OK;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cap) != hipSuccess) return SALS_ERR_HIP;
    if (cap != hipStreamCaptureStatusNone) return SALS_ERR_INVALID_ARG;
    if (c->rope_state == 0) return enqueue_rope_table(c, st);
    if (hipEventQuery(c->rope_ev) == hipSuccess) { c->rope_state = 2; return SALS_OK; }
    (void)hipGetLastError();  // (hipErrorNotReady is not an error here)
    if (st == c->rope_stream) return SALS_OK;
    return hipStreamWaitEvent(st, c->rope_ev, 0) == hipSuccess ? SALS_OK : SALS_ERR_HIP;
}

// the logits kernels use more than the default 48 KB of dynamic LDS: raised once per context, on first use
template <typename T> sals_status allow_logits_lds(const sals_ctx* c);
template <typename T> sals_status ensure_lds_attr(const sals_ctx* cc)
{
    sals_ctx* c = const_cast<sals_ctx*>(cc);
    if (c->lds_allowed) return SALS_OK;
    if (allow_logits_lds<T>(c) != SALS_OK) return SALS_ERR_HIP;
    c->lds_allowed = true;
    return SALS_OK;
}

template <typename T>
sals_status launch_dense(const sals_ctx* c, const void* q, const int32_t* q_pos, const void* K, const void* V,
                         const int32_t* seq_len, void* out, hipStream_t st)
{
    const sals_desc& d = c->d;
    const Layout& L = c->L;
    if (ensure_rope_table(c, st) != SALS_OK) return SALS_ERR_HIP;
    float* part = reinterpret_cast<float*>(c->ws + L.dn_part);
    const float2* rope = reinterpret_cast<const float2*>(c->ws + L.rope);
    const int G = d.H_q / d.H_kv;
    const int hb = dense_heads(d);
    const dim3 grid(L.dn_chunks, d.H_kv / hb, d.B);
    ProfScope ps(c, SALS_K_DENSE, st);
#define SALS_DENSE(GMAX, HB)                                                                               \
    hipLaunchKernelGGL((dense_attend_kernel<T, GMAX, HB>), grid, dim3(256), 0, st, static_cast<const T*>(q), q_pos, \
                       static_cast<const T*>(K), static_cast<const T*>(V), seq_len, d.S_max, d.H_q, d.H_kv, L.dn_chunks, \
                       rope, c->inv, part, d.rope_style, 1.0f / std::sqrt((float)d.d))
    if constexpr (sizeof(T) == 2) {
        if (hb == 2) { if (G <= 1) SALS_DENSE(1, 2); else if (G <= 2) SALS_DENSE(2, 2); else SALS_DENSE(4, 2); }
    }
    if (hb == 1) {
        if (G <= 1) SALS_DENSE(1, 1); else if (G <= 2) SALS_DENSE(2, 1);
        else if (G <= 4) SALS_DENSE(4, 1); else SALS_DENSE(8, 1);
    }
#undef SALS_DENSE
    if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    hipLaunchKernelGGL((dense_merge_kernel<T>), dim3(d.B * d.H_q), dim3(128), 0, st, part, static_cast<T*>(out),
                       L.dn_chunks);
    return launch_status();
}

// quantised full-rank value cache; codes_w != nullptr: plus the recent window's ring of 8-bit rows (the last
// n_sel - n_lo[b] selected tokens), whose logits a second logits pass left in logits_w [B, H, lk_w]
struct QvCache {
    const void* codes; const void* meta; int bits;
    const void* codes_w = nullptr; const void* meta_w = nullptr; const float* logits_w = nullptr;
    const int32_t* n_lo = nullptr; int lk_w = 0, ring = 0;
};

// qv == nullptr: latent value cache Vc, value sum in latent space and output projection through U_v.
// Otherwise: values are the de-quantised rows of the quantised cache (Vc unused).
// ring > 0: Kc, Vc are rings of that many rows per sequence (token t in row t mod ring).
// res: the selection's threshold bin is still to be ranked (see step_resolves).
// other: another pass's split logits, added up by this pass's logits kernel on the side (not by the tiles of several sequences).
// phases: which of the three launches to enqueue (all of them by default).  link: where the logits kernel leaves
// its tile statistics and where the value kernel finds the statistics of the whole softmax, when two passes over
// different caches share one softmax (recent window); by default the context's own array.
enum { kPhaseLogits = 1, kPhaseValue = 2, kPhaseOut = 4, kPhaseAll = 7 };
struct StatsLink { float2* stats; int stride; int part0; };  // [B*H][stride] records, this pass's tiles from part0 on

// 128-byte steps that the 64-token logits kernel loads ahead: the largest divisor of a slice's step count
template <typename T> int steps_ahead(const sals_desc& d, int ksplit)
{
    const int nkc = d.r * (int)sizeof(T) / kLgChunk / ksplit;
    int n = kLsMaxChunk;
    while (nkc % n != 0) --n;
    return n;
}

template <typename T> LogitsPlan plan_logits(const sals_desc& d)
{
    const int k_tot = d.top_k + d.n_sink + d.n_recent;
    auto n_wg = [&](int heads, int tok) { return (long long)ceil_div(k_tot, tok) * (d.H_kv / heads) * d.B; };
    LogitsPlan P{3, 0, 1, 1};
    // the 64-token kernel's split of the latent axis: with fewer workgroups than half the chip, as far as every slice
    // keeps at least two steps and the workgroups still fit the chip in one round
    const int nkc128 = d.r * (int)sizeof(T) / kLgChunk;
    const long long n_wg1 = n_wg(1, kLsTok);
    const bool allow_split = [] { const char* e = std::getenv("SALS_TUNE_LOGITS_KSPLIT"); return !e || std::atoi(e) != 0; }();  // tuning aid
    if (allow_split && n_wg1 <= 128)
        for (int ks = kLsMaxSplit; ks >= 2; ks /= 2)
            if (n_wg1 * ks <= 256 && nkc128 % ks == 0 && nkc128 / ks >= 2) { P.ksplit = ks; break; }
    // Estimated duration of each kernel for this shape: microseconds per 64-byte step of the latent axis and around the
    // loop, and G = query heads per KV head in the epilogue, fitted to 70 measured shapes (of 53 in bf16 and 17 in fp32 one
    // got a kernel that was not its fastest, by 4 %).  Workgroups beyond one per compute unit queue up or share it, which
    // takes as long.  fp32 is bound by its matrix instructions.
    constexpr bool bf = sizeof(T) == 2;
    const double steps = (double)d.r * sizeof(T) / kLgStep, G = (double)(d.H_q / d.H_kv);
    auto rounds = [](long long n) { return (double)((n + 255) / 256); };
    auto t_big = [&](long long n) { return rounds(n) * steps * (bf ? 0.65 : 3.5) + 2.1 + 0.7 * G; };  // 2 heads x 256 tokens
    auto t_mid = [&](long long n, int ks) {  // 1 head x 128 tokens
        return rounds(n * ks) * steps / ks * (bf ? 0.26 : 0.93) + 3.3 + 0.35 * G + (ks > 1 ? 2.4 : 0.0);
    };
    auto t_small = [&](long long n, int ks) {  // 1 head x 64 tokens
        return rounds(n * ks) * (steps / ks * (bf ? 0.29 : 0.59) + 1.3 + 0.33 * G) + (ks > 1 ? 2.4 : 0.0);
    };
    {
        const double t1 = d.H_kv % 2 == 0 ? t_big(n_wg(2, 256)) : 1e30, t2 = t_mid(n_wg(1, 128), 1), t3 = t_small(n_wg1, P.ksplit);
        P.pick = t1 <= t2 && t1 <= t3 ? 1 : (t2 <= t3 ? 2 : 3);
    }
    if (const char* e = std::getenv("SALS_TUNE_LOGITS")) {  // tuning aid: 1 | 2 | 3
        const int v = std::atoi(e);
        if (v == 1 && d.H_kv % 2 == 0) P.pick = 1;
        if (v == 2 || v == 3) P.pick = v;
    }
    // A selection of at most 64 tokens per sequence (a recent window) in a batch: tiles of two sequences' selections,
    // 128 tokens against one pass over the head's projector, the latent axis cut until the launch fills the chip.
    const char* const force = std::getenv("SALS_TUNE_LOGITS");  // tuning aid: "4" asks for these tiles at any batch
    const bool forced4 = force && std::atoi(force) == 4;
    if (k_tot <= 64 && (d.B >= 8 || forced4)) {
        const int n_steps = d.r * (int)sizeof(T) / kLgStep;
        const long long tiles = (long long)ceil_div(d.B, 2) * d.H_kv;
        int ks = 1;
        // (one workgroup per compute unit, or two where that leaves long slices.  A step of 16 sequences, 32 heads, r_hi = 2048
        // with one / two / four slices: 109.3 / 109.2 / 113.5 us; of 8 sequences 82.6 / 79.0 / 76.9)
        while (ks < kLsMaxSplit && tiles * ks < 512 && n_steps % (2 * ks) == 0 && n_steps / (2 * ks) >= (tiles * ks < 256 ? 8 : 24)) ks *= 2;
        if (const char* e = std::getenv("SALS_TUNE_MULTI_KSPLIT")) {  // tuning aid: any divisor of the step count up to 8
            const int v = std::atoi(e);
            if (v >= 1 && v <= kLsMaxSplit && n_steps % v == 0) ks = P.forced = v;
        }
        if (forced4 || t_mid(tiles, ks) < t_small(n_wg1, P.ksplit)) {
            P.pick = 4; P.n_parts = 1; P.ksplit = ks;
            return P;
        }
    }
    if (P.pick != 3) {
        P.n_parts = ceil_div(k_tot, P.pick == 2 ? 128 : 256);
        P.ksplit = 1;
        return P;
    }
    P.n_parts = ceil_div(k_tot, kLsTok);
    P.nst = steps_ahead<T>(d, P.ksplit);
    return P;
}

// the 64-token logits kernel for a number of steps loaded ahead, with or without the selection inside
template <typename T> struct SmallLogits {
    typedef void (*Fn)(const int32_t*, const int32_t*, const T*, int, int, int, int, int, int, int, int, const T*, const T*,
                       const int32_t*, const float2*, InvFreq, float*, float2*, int, int, int, float, int, float*, int,
                       FusedSelect);
    typedef void (*SideFn)(const int32_t*, const int32_t*, const T*, int, int, int, int, int, int, int, int, const T*, const T*,
                           const int32_t*, const float2*, InvFreq, float*, float2*, int, int, int, float, int, float*, int,
                           SplitLogits);
    static SideFn side(int nst)
    {
#define SALS_LS(N) case N: return attend_logits_small_side_kernel<T, N>;
        switch (nst) {
            SALS_LS(1) SALS_LS(2) SALS_LS(3) SALS_LS(4) SALS_LS(5) SALS_LS(6) SALS_LS(7) SALS_LS(8) SALS_LS(9)
            default: return attend_logits_small_side_kernel<T, 10>;
        }
#undef SALS_LS
    }
    static Fn get(int nst, bool fused)
    {
#define SALS_LS(N) case N: return fused ? (Fn)attend_logits_small_kernel<T, N, true> : (Fn)attend_logits_small_kernel<T, N, false>;
        switch (nst) {
            SALS_LS(1) SALS_LS(2) SALS_LS(3) SALS_LS(4) SALS_LS(5) SALS_LS(6) SALS_LS(7) SALS_LS(8) SALS_LS(9)
            default: return fused ? (Fn)attend_logits_small_kernel<T, 10, true> : (Fn)attend_logits_small_kernel<T, 10, false>;
        }
#undef SALS_LS
    }
};

// the window's logits and the step's selection in one launch, for one sequence (64-token form) and for a batch
template <typename T> struct WindowSelectSmall {
    typedef void (*Fn)(StepSelect, const T*, int, int, int, int, int, int, int, int, const T*, const T*, const int32_t*, const float2*,
                       InvFreq, float*, float2*, int, int, int, float, float*, int);
    static Fn get(int nst)
    {
#define SALS_WS(N) case N: return window_select_small_kernel<T, N>;
        switch (nst) {
            SALS_WS(1) SALS_WS(2) SALS_WS(3) SALS_WS(4) SALS_WS(5) SALS_WS(6) SALS_WS(7) SALS_WS(8) SALS_WS(9)
            default: return window_select_small_kernel<T, 10>;
        }
#undef SALS_WS
    }
};
template <typename T> auto window_select_for(int group, bool wide)
{
    if constexpr (sizeof(T) == 2) {
        if (wide) return window_select_kernel<T, 1, 1, true>;
    }
    if (group == 1) return window_select_kernel<T, 1, 1, false>;
    if (group == 4) return window_select_kernel<T, 4, 4, false>;
    if (group % 4 == 0) return window_select_kernel<T, 4, 0, false>;
    return window_select_kernel<T, 1, 0, false>;
}
int select_blocks(const sals_desc& d) { return ceil_div(d.B, kXcds) * kXcds; }
// Slices of the window's latent axis where the launch that it shares with the selection has tiles of two heads and four sequences (0: it
// has not): as many as fit beside the selection, one workgroup per compute unit, at least two (two rounds of those are shorter than
// one of the whole axis), of two steps and more.  (One slice would leave its statistics itself, in another order than the tiles of a head
// and two sequences that the window's logits have in a launch of their own: a step and its stages agree bit for bit.)  Such a tile reads
// half as much per product as one of a head and two sequences, which is what binds those: a step with 2-bit values, 32 heads, r = 512,
// r_hi = 2048 in us with the latter's slices and with these: 8 sequences 73.2 and 70.6, 12 95.8 and 91.7, 16 109.3 and 104.2, 24 152.7
// and 142.4, 32 189.4 and 179.5; 16 with r_hi = 1024 88.2 and 85.2.  (fp32 is bound by its matrix instructions.  Four query heads per
// KV head: r_hi = 2048 as fast, 1024 3 % faster, not worth kernels of their own.)
int wide_window_slices(const sals_ctx* win)
{
    const sals_desc& d = win->d;
    const int steps = d.r * 2 / kLgStep, forced = win->plan.forced;
    if (win->plan.pick != 4 || d.dtype != SALS_BF16 || d.H_q != d.H_kv || d.H_kv % 2 != 0 || steps < 4 || forced == 1) return 0;
    if (forced) return forced;
    const int tiles = ceil_div(d.B, 4) * (d.H_kv / 2);
    return std::min({std::max(2, (256 - select_blocks(d)) / tiles), kLsMaxSplit, steps / 2});
}
// Slices in that launch, wide tiles or not: the window's own plan, halved while its workgroups fit the chip at once (one per compute unit
// in the 64-token form, two otherwise) and do not together with the selection's.  (A workgroup too many is a round too many: one sequence,
// eight slices would be 257 workgroups.)
int window_select_slices(const sals_ctx* win)
{
    if (const int ks = wide_window_slices(win)) return ks;
    const LogitsPlan& P = win->plan;
    const sals_desc& d = win->d;
    const int tiles = P.pick == 4 ? ceil_div(d.B, 2) * d.H_kv : P.n_parts * d.H_kv * d.B, slots = P.pick == 4 ? 512 : 256;
    int ks = P.ksplit;
    while (ks > 1 && tiles * ks <= slots && tiles * ks + d.B > slots) ks /= 2;
    return ks;
}
// Whether a decode step has the window's logits in its selection's launch.  Both small: sequences of at most kWsMaxS tokens,
// windows that fill tiles of one or two sequences; and what halved slices of the 64-token form take longer (a 64-byte step 0.29
// us, in fp32 0.59) is less than the launches save.  (One fp32 sequence of 1024 and of 8192 tokens, launches of their own and the
// shared one: r_hi 1280 59.0 and 56.5, 62.1 and 58.3 us a step, r_hi 1536 59.9 and 59.8, 63.0 and 61.1, r_hi 2048 62.9 and 65.0, 66.1
// and 66.7; four bf16 ones of 1024 tokens: r_hi 1536 47.0 and 46.5, r_hi 2048 49.1 and 50.3.)
bool window_in_select(const sals_ctx* win)
{
    const LogitsPlan& P = win->plan;
    if (win->d.S_max > kWsMaxS || !win->fuse_select || (P.pick != 3 && P.pick != 4)) return false;
    const bool bf = win->d.dtype == SALS_BF16;
    const int steps = win->d.r * (bf ? 2 : 4) / kLgStep;
    return P.pick == 4 || (steps / window_select_slices(win) - steps / P.ksplit) * (bf ? 0.29 : 0.59) < 8.0;
}
int window_slices(const sals_ctx* win) { return window_in_select(win) ? window_select_slices(win) : win->plan.ksplit; }

// Whether a whole decode step on this context lets the logits kernel select by itself (no selection launch): the
// 64-token kernel in one round of workgroups, a cache of at most 4096 rows whose score rows start 16-byte aligned, a selection that
// fits the kernel's list.  (Also where the latent axis is split, every slice selecting by itself: one sequence in fp32, 1024 tokens,
// 128 selected, four slices: 32.1 -> 30.9 us a step; 8 KV heads in bf16, 4096 tokens, 512 selected, two slices: 27.3 -> 26.2.  In two
// or three rounds, which fp32 has, the selection of each of them costs more than the launch; inside and as a launch: 5 sequences of
// 4096 tokens, 130 selected, H_kv 32, r 512 74.2 and 73.6 us, 6 sequences, 320 selected, r 256 83.1 and 76.3.)
bool fused_selection(const sals_ctx* c)
{
    const sals_desc& d = c->d;
    return c->plan.pick == 3 && (long long)c->plan.n_parts * d.H_kv * d.B * c->plan.ksplit <= 256 && d.S_max <= kLsFusedMaxS &&
           d.S_max % 4 == 0 && d.top_k + d.n_sink + d.n_recent <= kLsFusedMaxK && c->fuse_select;
}

// the instantiation of attend_logits_kernel (256- and 128-token tiles) for a group size (query heads per KV head)
template <typename T, int HEADS, int NTG, int NB, bool MULTI = false> auto logits_kernel_for(int group)
{
    if (group == 1) return attend_logits_kernel<T, HEADS, NTG, NB, 1, 1, MULTI>;
    if (group == 4) return attend_logits_kernel<T, HEADS, NTG, NB, 4, 4, MULTI>;
    if (group % 4 == 0) return attend_logits_kernel<T, HEADS, NTG, NB, 4, 0, MULTI>;
    return attend_logits_kernel<T, HEADS, NTG, NB, 1, 0, MULTI>;
}

// the same with another pass's split logits on the side
template <typename T, int HEADS, int NTG, int NB> auto logits_side_kernel_for(int group)
{
    if (group == 1) return attend_logits_side_kernel<T, HEADS, NTG, NB, 1, 1>;
    if (group == 4) return attend_logits_side_kernel<T, HEADS, NTG, NB, 4, 4>;
    if (group % 4 == 0) return attend_logits_side_kernel<T, HEADS, NTG, NB, 4, 0>;
    return attend_logits_side_kernel<T, HEADS, NTG, NB, 1, 0>;
}

// the same on a selection whose threshold bin is still to be ranked
template <typename T, int HEADS, int NTG, int NB> auto logits_resolve_kernel_for(int group)
{
    if (group == 1) return attend_logits_resolve_kernel<T, HEADS, NTG, NB, 1, 1>;
    if (group == 4) return attend_logits_resolve_kernel<T, HEADS, NTG, NB, 4, 4>;
    if (group % 4 == 0) return attend_logits_resolve_kernel<T, HEADS, NTG, NB, 4, 0>;
    return attend_logits_resolve_kernel<T, HEADS, NTG, NB, 1, 0>;
}

template <typename T> sals_status allow_logits_lds(const sals_ctx* c)
{
    const LogitsPlan& P = c->plan;
    const int group = c->d.H_q / c->d.H_kv;
    auto allow = [](const void* kern, size_t bytes) {
        return bytes <= 48 * 1024 ||
               hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
    };
    bool ok = true;
    if (P.pick == 1) ok = allow(reinterpret_cast<const void*>(logits_kernel_for<T, 2, 4, 2>(group)), logits_cfg<2, 4, 2>::LDS);
    else if (P.pick == 2) ok = allow(reinterpret_cast<const void*>(logits_kernel_for<T, 1, 4, 1>(group)), logits_cfg<1, 4, 1>::LDS);
    else if (P.pick == 4) ok = allow(reinterpret_cast<const void*>(logits_kernel_for<T, 1, 4, 1, true>(group)), logits_cfg<1, 4, 1>::LDS);
    else {
        ok = allow(reinterpret_cast<const void*>(SmallLogits<T>::get(P.nst, false)), kLsLds) &&
             allow(reinterpret_cast<const void*>(SmallLogits<T>::get(P.nst, true)), kLsLds);
    }
    if (ok && step_resolves(c)) {
        if (P.pick == 1) ok = allow(reinterpret_cast<const void*>(logits_resolve_kernel_for<T, 2, 4, 2>(group)), logits_cfg<2, 4, 2>::LDS);
        if (P.pick == 2) ok = allow(reinterpret_cast<const void*>(logits_resolve_kernel_for<T, 1, 4, 1>(group)), logits_cfg<1, 4, 1>::LDS);
    }
    // (a context with recent tokens may have a window beside it)
    if (ok && c->d.n_recent > 0) {
        if (P.pick == 1) ok = allow(reinterpret_cast<const void*>(logits_side_kernel_for<T, 2, 4, 2>(group)), logits_cfg<2, 4, 2>::LDS);
        if (P.pick == 2) ok = allow(reinterpret_cast<const void*>(logits_side_kernel_for<T, 1, 4, 1>(group)), logits_cfg<1, 4, 1>::LDS);
        if (P.pick == 3) ok = allow(reinterpret_cast<const void*>(SmallLogits<T>::side(P.nst)), kLsLds);
    }
    // (a context without sinks and recent tokens may be a window)
    if (ok && c->d.n_sink == 0 && c->d.n_recent == 0) {
        if (P.pick == 4) {
            const bool wide = wide_window_slices(c) > 0;
            ok = allow(reinterpret_cast<const void*>(window_select_for<T>(group, wide)), wide ? logits_cfg<2, 4, 2>::LDS : logits_cfg<1, 4, 1>::LDS);
        }
        if (P.pick == 3) {
            const int nst = steps_ahead<T>(c->d, window_slices(c));
            ok = allow(reinterpret_cast<const void*>(WindowSelectSmall<T>::get(nst)), kLsLds) &&
                 allow(reinterpret_cast<const void*>(SmallLogits<T>::get(nst, false)), kLsLds);
        }
    }
    return ok ? SALS_OK : SALS_ERR_HIP;
}

// a context's split logits (see SplitLogits)
SplitLogits split_logits(const sals_ctx* c, int ksplit, const int32_t* n_sel, float2* stats, int stats_stride)
{
    return SplitLogits{reinterpret_cast<const float*>(c->ws + c->L.plogits), n_sel, reinterpret_cast<float*>(c->ws + c->L.logits), stats,
                       ksplit, c->plan.n_parts, c->d.B * c->d.H_q, c->d.H_q, c->L.lk, stats_stride};
}

// Split logits that the value kernel adds up itself, in LDS: quantised values if their kernel has one range (a workgroup then reads
// its heads' partial sums and no others), latent ones as far as a workgroup may read a whole sequence's (see pv_block).  Whole steps
// with the launch that adds them up -> without, one sequence unless said: 32 KV heads, 128 tokens 25.6 -> 23.8 us, 2 x 128 26.9 ->
// 25.0, 3 x 128 of 8 KV heads 27.5 -> 25.9, fp32 256 tokens 41.7 -> 40.7; past the line, 8 KV heads, 512 tokens (256 KB) 26.8 -> 28.6.
// 4-bit values, 32 KV heads, 256 tokens 30.7 -> 29.2, 8 KV heads, 512 tokens 30.1 -> 28.7, 1000 tokens 40.3 -> 40.1.
bool value_adds_slices(const sals_ctx* c, int ksplit, bool quantised)
{
    const sals_desc& d = c->d;
    const size_t k_tot = (size_t)d.top_k + d.n_sink + d.n_recent;
    if (ksplit <= 1) return false;
    if (quantised) return c->L.qv_ntr == 1 && k_tot <= kQvSplitTok;
    return c->L.pv_tok_per_wg <= kPvSplitTok && d.H_q * k_tot * ksplit * 4 <= kPvSplitBytes;
}

// Value sum over the selected tokens of a cache, and of a second one under the same softmax (the recent window).
struct PvPass { const sals_ctx* c; const int32_t* idx; const int32_t* n_sel; const void* Vc; int ring; };
template <typename T>
void launch_pv(const sals_ctx* c, const float2* stats, int stats_stride, const PvPass& a, const PvPass* b, const T* Uv,
               hipStream_t st, int ksplit = 1)  // > 1: the logits of `a` (alone) are still that many partial sums
{
    const sals_desc& d = c->d;
    ProfScope ps(c, SALS_K_ATTEND_PV, st);
    auto of = [](const PvPass& p) {
        const sals_desc& e = p.c->d;
        const Layout& L = p.c->L;
        return PvSecond<T>{p.idx, p.n_sel, static_cast<const T*>(p.Vc), reinterpret_cast<const float*>(p.c->ws + L.logits),
                           reinterpret_cast<float*>(p.c->ws + L.tpart), e.r, L.pv_ntr, L.pv_tok_per_wg,
                           e.top_k + e.n_sink + e.n_recent, L.lk, e.S_max, p.ring};
    };
    const PvSecond<T> f = of(a), g = b ? of(*b) : PvSecond<T>{};
    const int n_items = f.r / kPvCols * f.n_tr * d.B;
    // idle compute units warm U_v, up to what the launch can read beside its own loads (measured: 5 MB cost it nothing
    // and save the next launch 0.8 us, 8 MB cost what they save)
    const size_t uv_bytes = (size_t)d.H_kv * kHeadDim * d.r * sizeof(T);
    const int n_more = b ? g.r / kPvCols * g.n_tr * d.B
                         : (n_items < 256 && uv_bytes <= (size_t)6 << 20 ? (256 - n_items) / kXcds * kXcds : 0);
    const bool w8 = a.c->L.pv_waves == 8 || (b && b->c->L.pv_waves == 8);
#define SALS_PV(NW, MB, TWO)                                                                                              \
    hipLaunchKernelGGL((attend_pv_kernel<T, NW, MB, TWO>), dim3(n_items + n_more), dim3(NW * 64), 0, st, f.idx,            \
                       f.n_sel, stats, d.B, f.r, f.n_tr, stats_stride, f.tok_per_wg, f.k_tot, d.H_q, f.lk, f.Vc, f.logits, \
                       f.Tpart, f.S_max, f.ring, Uv, d.H_kv, g)
#define SALS_PV_B(NW, MB) do { if (b) SALS_PV(NW, MB, true); else SALS_PV(NW, MB, false); } while (0)
#define SALS_PV_S(NW, MB)                                                                                                 \
    hipLaunchKernelGGL((attend_pv_split_kernel<T, NW, MB>), dim3(n_items + n_more), dim3(NW * 64), 0, st, f.idx, f.n_sel,  \
                       reinterpret_cast<const float*>(c->ws + c->L.plogits), d.B, f.r, f.n_tr, ksplit, f.tok_per_wg, f.k_tot, \
                       d.H_q, f.lk, f.Vc, f.Tpart, f.S_max, f.ring, Uv, d.H_kv)
    if (ksplit > 1) {
        if (d.H_q <= 32) { if (w8) SALS_PV_S(8, 1); else SALS_PV_S(4, 1); }
        else { if (w8) SALS_PV_S(8, 2); else SALS_PV_S(4, 2); }
    }
    else if (d.H_q <= 32) { if (w8) SALS_PV_B(8, 1); else SALS_PV_B(4, 1); }
    else { if (w8) SALS_PV_B(8, 2); else SALS_PV_B(4, 2); }
#undef SALS_PV_S
#undef SALS_PV_B
#undef SALS_PV
}

// Output projection.  The loads of a wave (BATCH latent steps x RPR groups of token ranges) follow what there is, so that the
// usual ranks need one memory round trip and few loads are repeated.  r2 > 0: a second cache of that rank beside the first.
template <typename T>
void launch_out(hipStream_t st, const sals_desc& d, int n_tr, const T* Uv, const float* tpart, int r2, int n_tr2, const T* Uv2,
                const float* tpart2, void* out)
{
    const int n_rows = d.B * (d.H_q / d.H_kv), R = out_tile_rows(d);
    const int spw = ceil_div(d.r / (4 * elem<T>::vec), kOutWaves), loads = ceil_div(n_tr, kOutRows / R);
    const dim3 grid(d.H_kv, kHeadDim / 16, ceil_div(n_rows, R));
#define SALS_OUT(BATCH, RPR, BATCH2)                                                                                      \
    hipLaunchKernelGGL((attend_out_kernel<T, BATCH, RPR, BATCH2>), grid, dim3(64 * kOutWaves), 0, st, Uv, tpart, d.B, d.r, \
                       d.H_q, d.H_kv, n_tr, R, r2, n_tr2, Uv2, tpart2, static_cast<T*>(out))
#define SALS_OUT_L(BATCH, BATCH2)                                                                                         \
    do { if (loads > 1) SALS_OUT(BATCH, 2, BATCH2); else SALS_OUT(BATCH, 1, BATCH2); } while (0)
    if (r2 > 0) SALS_OUT_L(3, 8);
    else if (spw <= 2) SALS_OUT_L(2, 0);
    else if (spw <= 3) SALS_OUT_L(3, 0);
    else SALS_OUT_L(4, 0);
#undef SALS_OUT_L
#undef SALS_OUT
}

template <typename T>
sals_status launch_attend(const sals_ctx* c, const void* q, const int32_t* q_pos, const void* Kc,
                          const void* Vc, const void* W, const int32_t* idx, const int32_t* n_sel, void* out,
                          hipStream_t st, const QvCache* qv = nullptr, int ring = 0, int phases = kPhaseAll,
                          const StatsLink* link = nullptr, const FusedSelect* fs = nullptr, const SplitLogits* other = nullptr,
                          const TopkResolve* res = nullptr)
{
    const sals_desc& d = c->d;
    const Layout& L = c->L;
    const int k_tot = d.top_k + d.n_sink + d.n_recent;
    float* logits = reinterpret_cast<float*>(c->ws + L.logits);
    LogitsPlan P = c->plan;
    if (ring > 0 && P.pick >= 3) {  // (as in a decode step)
        P.ksplit = window_slices(c);
        if (P.pick == 3) P.nst = steps_ahead<T>(d, P.ksplit);
    }
    const bool value_adds = phases == kPhaseAll && link == nullptr && (!qv || !qv->codes_w) && value_adds_slices(c, P.ksplit, qv != nullptr);
    // tile statistics: written by this pass's logits kernel from record `part0` on, read as a whole by the value kernel
    float2* const stats_all = link ? link->stats : reinterpret_cast<float2*>(c->ws + L.stats);
    float2* const stats = stats_all + (link ? link->part0 : 0);
    const int stats_stride = link ? link->stride : P.n_parts;
    const float2* rope = reinterpret_cast<const float2*>(c->ws + L.rope);
    float* tpart = reinterpret_cast<float*>(c->ws + L.tpart);
    const int n_parts = P.n_parts;
    if (phases & kPhaseLogits) {
        sals_status rs = ensure_rope_table(c, st);
        if (rs == SALS_OK) rs = ensure_lds_attr<T>(c);
        if (rs != SALS_OK) return rs;
        // replicate the smaller operand across the XCDs' L2s: all of U_k, or the gathered rows
        const size_t a_bytes = (size_t)d.H_kv * kHeadDim * d.r, b_bytes = (size_t)d.B * k_tot * d.r;
        const int heads_fastest = a_bytes <= b_bytes ? 1 : 0;
        ProfScope ps(c, SALS_K_ATTEND_LOGITS, st);
#define SALS_LOGITS_ARGS                                                                                          \
    static_cast<const T*>(Kc), w_section<T>(c, W, 2), idx, n_sel, static_cast<const T*>(q), q_pos, rope, c->inv,   \
        logits, stats, d.B, d.S_max, d.r, d.H_q, d.H_kv, k_tot, L.lk, n_parts, heads_fastest, d.rope_style,        \
        1.0f / std::sqrt((float)d.d), ring, stats_stride, static_cast<float*>(nullptr), 1
#define SALS_LOGITS(HEADS, NTG, NB)                                                                              \
    do {                                                                                                     \
        typedef logits_cfg<HEADS, NTG, NB> LC;                                                               \
        const dim3 grid(n_parts * (d.H_kv / HEADS) * d.B);                                                   \
        if (other) hipLaunchKernelGGL((logits_side_kernel_for<T, HEADS, NTG, NB>(d.H_q / d.H_kv)), grid, dim3(LC::NT), LC::LDS, st, \
                                      SALS_LOGITS_ARGS, *other);                                             \
        else if (res) hipLaunchKernelGGL((logits_resolve_kernel_for<T, HEADS, NTG, NB>(d.H_q / d.H_kv)), grid, dim3(LC::NT), LC::LDS, st, \
                                         SALS_LOGITS_ARGS, *res);                                            \
        else hipLaunchKernelGGL((logits_kernel_for<T, HEADS, NTG, NB>(d.H_q / d.H_kv)), grid, dim3(LC::NT), LC::LDS, st, \
                                SALS_LOGITS_ARGS);                                                           \
    } while (0)
        const int pick = P.pick;
        if (pick == 1) SALS_LOGITS(2, 4, 2);        // 2 heads x 256 tokens, 8 waves
        else if (pick == 2) SALS_LOGITS(1, 4, 1);   // 1 head  x 128 tokens
        else if (pick == 4) {  // two sequences' short selections per 128-token tile, latent axis in P.ksplit slices
            typedef logits_cfg<1, 4, 1> LC;
            auto kern = logits_kernel_for<T, 1, 4, 1, true>(d.H_q / d.H_kv);
            float* plogits = reinterpret_cast<float*>(c->ws + L.plogits);
            hipLaunchKernelGGL(kern, dim3(ceil_div(d.B, 2) * d.H_kv * P.ksplit), dim3(LC::NT), LC::LDS, st,
                               static_cast<const T*>(Kc), w_section<T>(c, W, 2), idx, n_sel, static_cast<const T*>(q), q_pos,
                               rope, c->inv, logits, stats, d.B, d.S_max, d.r, d.H_q, d.H_kv, k_tot, L.lk, 1, heads_fastest,
                               d.rope_style, 1.0f / std::sqrt((float)d.d), ring, stats_stride, plogits, P.ksplit);
        }
        else {  // few tiles: 1 head x 64 tokens with the whole latent axis loaded ahead
            const int ksplit = P.ksplit, nst = P.nst;
            float* plogits = reinterpret_cast<float*>(c->ws + L.plogits);
            const dim3 grid(n_parts * d.H_kv * d.B * ksplit);
#define SALS_LS_ARGS                                                                                                      \
    idx, n_sel, w_section<T>(c, W, 2), d.B, d.H_kv, n_parts, heads_fastest, ksplit, k_tot, d.r, d.H_q,                     \
        static_cast<const T*>(Kc), static_cast<const T*>(q), q_pos, rope, c->inv, logits, stats, d.S_max, L.lk,            \
        d.rope_style, 1.0f / std::sqrt((float)d.d), ring, plogits, stats_stride
            // fs: idx / n_sel are outputs of this launch (the kernel selects from fs->scores itself)
            if (other) {
                hipLaunchKernelGGL(SmallLogits<T>::side(nst), grid, dim3(kLsThreads), kLsLds, st, SALS_LS_ARGS, *other);
            } else {
                const FusedSelect fsel = fs ? *fs : FusedSelect{nullptr, nullptr, 0, 0, 0};
                hipLaunchKernelGGL(SmallLogits<T>::get(nst, fs != nullptr), grid, dim3(kLsThreads), kLsLds, st, SALS_LS_ARGS, fsel);
            }
#undef SALS_LS_ARGS
        }
        if (P.ksplit > 1 && !value_adds) {
            if (launch_status() != SALS_OK) return SALS_ERR_HIP;
            hipLaunchKernelGGL(logits_finish_kernel, dim3(n_parts, d.B * d.H_q), dim3(64), 0, st,
                               split_logits(c, P.ksplit, n_sel, stats, stats_stride));
        }
#undef SALS_LOGITS
#undef SALS_LOGITS_ARGS
        if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    }
    if (qv != nullptr) {
        ProfScope ps(c, SALS_K_ATTEND_QV, st);
        QvArgs a{};
        a.Vq = static_cast<const unsigned char*>(qv->codes); a.Vmeta = qv->meta; a.idx = idx; a.n_sel = n_sel;
        a.logits = logits; a.stats = stats_all; a.part = reinterpret_cast<float*>(c->ws + L.qv_part); a.out = out;
        a.n_parts = stats_stride; a.B = d.B; a.S_max = d.S_max; a.H = d.H_q; a.H_kv = d.H_kv; a.k_tot = k_tot; a.lk = L.lk;
        a.tok_per_wg = L.qv_tok_per_wg; a.n_tr = L.qv_ntr; a.part0 = 0; a.n_tr_all = L.qv_ntr;
        a.Vq_w = static_cast<const unsigned char*>(qv->codes_w); a.Vmeta_w = qv->meta_w; a.logits_w = qv->logits_w;
        a.n_lo = qv->n_lo; a.lk_w = qv->lk_w; a.ring = qv->ring; a.ksplit = P.ksplit;
        if (value_adds) a.logits = reinterpret_cast<const float*>(c->ws + L.plogits);
        const bool win = qv->codes_w != nullptr;
        const dim3 grid(L.qv_ntr * d.H_kv * d.B);
        const int G = d.H_q / d.H_kv;
#define SALS_QV(BITS, GMAX)                                                                             \
    do {                                                                                                \
        if (win) hipLaunchKernelGGL((attend_qv_kernel<T, BITS, GMAX, true>), grid, dim3(256), 0, st, a); \
        else if (value_adds) hipLaunchKernelGGL((attend_qv_kernel<T, BITS, GMAX, false, true>), grid, dim3(256), 0, st, a); \
        else hipLaunchKernelGGL((attend_qv_kernel<T, BITS, GMAX, false>), grid, dim3(256), 0, st, a);   \
    } while (0)
#define SALS_QV_G(BITS)                                                                                 \
    do {                                                                                                \
        if (G <= 1) SALS_QV(BITS, 1); else if (G <= 2) SALS_QV(BITS, 2);                                \
        else if (G <= 4) SALS_QV(BITS, 4); else SALS_QV(BITS, 8);                                       \
    } while (0)
        if (qv->bits == 4) SALS_QV_G(4); else SALS_QV_G(2);
#undef SALS_QV_G
#undef SALS_QV
        if (launch_status() != SALS_OK) return SALS_ERR_HIP;
        if (L.qv_ntr > 1) {
            const size_t n4 = (size_t)d.B * d.H_q * kHeadDim / 4;
            hipLaunchKernelGGL((qv_merge_kernel<T>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, a.part,
                               static_cast<T*>(out), L.qv_ntr, n4);
        }
        return launch_status();
    }
    if (phases & kPhaseValue)
        launch_pv<T>(c, stats_all, stats_stride, PvPass{c, idx, n_sel, Vc, ring}, nullptr, w_section<T>(c, W, 3), st,
                     value_adds ? P.ksplit : 1);
    if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    if (phases & kPhaseOut) {
        ProfScope ps(c, SALS_K_ATTEND_OUT, st);
        launch_out<T>(st, d, L.pv_ntr, w_section<T>(c, W, 3), tpart, 0, 0, nullptr, nullptr, out);
    }
    return launch_status();
}

}  // namespace

extern "C" {

const char* sals_status_string(sals_status s)
{
    switch (s) {
        case SALS_OK: return "SALS_OK";
        case SALS_ERR_INVALID_ARG: return "SALS_ERR_INVALID_ARG";
        case SALS_ERR_UNSUPPORTED: return "SALS_ERR_UNSUPPORTED";
        case SALS_ERR_WORKSPACE: return "SALS_ERR_WORKSPACE";
        case SALS_ERR_HIP: return "SALS_ERR_HIP";
    }
    return "SALS_ERR_UNKNOWN";
}

sals_status sals_workspace_bytes(const sals_desc* desc, size_t* bytes)
{
    if (!bytes) return SALS_ERR_INVALID_ARG;
    sals_status s = validate(desc);
    if (s != SALS_OK) return s;
    *bytes = make_layout(*desc).total;
    return SALS_OK;
}

sals_status sals_packed_weight_bytes(const sals_desc* desc, size_t* bytes)
{
    if (!bytes) return SALS_ERR_INVALID_ARG;
    sals_status s = validate(desc);
    if (s != SALS_OK) return s;
    *bytes = align_up(4 * make_layout(*desc).w_section * (desc->dtype == SALS_BF16 ? 2 : 4));
    return SALS_OK;
}

sals_status sals_create(const sals_desc* desc, void* d_workspace, size_t workspace_bytes, sals_ctx** out)
{
    if (!out) return SALS_ERR_INVALID_ARG;
    *out = nullptr;
    sals_status s = validate(desc);
    if (s != SALS_OK) return s;
    Layout L = make_layout(*desc);
    if (workspace_bytes < L.total) L = make_layout(*desc, false);
    if (!d_workspace || (reinterpret_cast<uintptr_t>(d_workspace) % kAlign) != 0 || workspace_bytes < L.total)
        return SALS_ERR_WORKSPACE;
    sals_ctx* c = new (std::nothrow) sals_ctx;
    if (!c) return SALS_ERR_INVALID_ARG;
    c->d = *desc;
    c->L = L;
    c->ws = static_cast<unsigned char*>(d_workspace);
    c->ws_bytes = workspace_bytes;
    for (int p = 0; p < kPairs; ++p)
        c->inv.f[p] = std::pow((double)desc->rope_theta, -2.0 * (double)p / (double)desc->d);
    const bool bf = desc->dtype == SALS_BF16;
    c->plan = bf ? plan_logits<bf16_t>(c->d) : plan_logits<float>(c->d);
    c->score_rows = plan_score_rows(c->d);
    if (const char* e = std::getenv("SALS_TUNE_SCORE_STREAM")) c->score_stream = std::atoi(e) != 0;  // tuning aid
    if (const char* e = std::getenv("SALS_TUNE_FUSE_SELECT")) c->fuse_select = std::atoi(e) != 0;  // tuning aid
    *out = c;
    return SALS_OK;
}

sals_status sals_prepare(sals_ctx* ctx, void* hip_stream)
{
    if (!ctx) return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (ctx->rope_state != 2) {
        if (ctx->rope_state == 0) {
            sals_status s = enqueue_rope_table(ctx, st);
            if (s != SALS_OK) return s;
        }
        if (hipEventSynchronize(ctx->rope_ev) != hipSuccess) return SALS_ERR_HIP;
        ctx->rope_state = 2;
    }
    return ctx->d.dtype == SALS_BF16 ? ensure_lds_attr<bf16_t>(ctx) : ensure_lds_attr<float>(ctx);
}

void sals_destroy(sals_ctx* ctx)
{
    if (!ctx) return;
    for (auto& r : ctx->prof) { (void)hipEventDestroy(r.start); (void)hipEventDestroy(r.stop); }
    if (ctx->rope_ev) (void)hipEventDestroy(ctx->rope_ev);
    delete ctx;
}

sals_status sals_pack_weights(sals_ctx* ctx, const void* Uk, const void* Uv, void* W, void* hip_stream)
{
    if (!ctx || bad(Uk) || bad(Uv) || !W || (reinterpret_cast<uintptr_t>(W) % kAlign) != 0)
        return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const sals_desc& d = ctx->d;
    const size_t n = ctx->L.w_section;
    dim3 grid((unsigned)std::min<size_t>(2048, (n + 255) / 256), 4);
    if (d.dtype == SALS_BF16)
        hipLaunchKernelGGL((pack_weights_kernel<bf16_t>), grid, dim3(256), 0, st, static_cast<const bf16_t*>(Uk),
                           static_cast<const bf16_t*>(Uv), static_cast<bf16_t*>(W), n, d.H_kv * d.d, d.r,
                           d.rope_style);
    else
        hipLaunchKernelGGL((pack_weights_kernel<float>), grid, dim3(256), 0, st, static_cast<const float*>(Uk),
                           static_cast<const float*>(Uv), static_cast<float*>(W), n, d.H_kv * d.d, d.r,
                           d.rope_style);
    return launch_status();
}

const char* sals_kernel_name(int kernel)
{
    return (kernel >= 0 && kernel < SALS_N_KERNELS) ? kKernelNames[kernel] : "unknown";
}

sals_status sals_profile_enable(sals_ctx* ctx, int on)
{
    if (!ctx) return SALS_ERR_INVALID_ARG;
    ctx->profiling = on != 0;
    return SALS_OK;
}

sals_status sals_profile_collect(sals_ctx* ctx, double* total_ms, int32_t* launches)
{
    if (!ctx || !total_ms || !launches) return SALS_ERR_INVALID_ARG;
    for (int k = 0; k < SALS_N_KERNELS; ++k) { total_ms[k] = 0.0; launches[k] = 0; }
    sals_status st = SALS_OK;
    for (auto& r : ctx->prof) {
        float ms = 0.f;
        if (hipEventSynchronize(r.stop) != hipSuccess || hipEventElapsedTime(&ms, r.start, r.stop) != hipSuccess)
            st = SALS_ERR_HIP;
        total_ms[r.kernel] += ms;
        launches[r.kernel] += 1;
        (void)hipEventDestroy(r.start);
        (void)hipEventDestroy(r.stop);
    }
    ctx->prof.clear();
    return st;
}

sals_status sals_compress_append(sals_ctx* ctx, const void* k_new, const void* v_new, const void* W, void* Kc,
                                 void* Vc, int32_t* seq_len, void* hip_stream)
{
    if (!ctx || bad(k_new) || bad(v_new) || bad(W) || bad(Kc) || bad(Vc) || !seq_len) return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    return ctx->d.dtype == SALS_BF16
               ? launch_append<bf16_t>(ctx, W, k_new, v_new, Kc, Vc, QuantArgs{}, seq_len, st, true)
               : launch_append<float>(ctx, W, k_new, v_new, Kc, Vc, QuantArgs{}, seq_len, st, true);
}

namespace {
// Tiles of the bf16 prompt compression: the choice with the smallest estimated duration in us, where a round of one workgroup
// per compute unit takes (64-byte steps of the D axis x measured time per step + start and store of a tile).  A step takes
// `full` with the whole chip at work (the matrix cores' clock follows the power drawn) and `idle` with few workgroups.
// The tiles that do not fill a round may become smaller ones (see PfPart).
struct PrefillTile { int nbw, nbt; double idle, full, over; };
constexpr PrefillTile kPrefillTiles[] = {
    {1, 1, 0.105, 0.20, 2.0}, {2, 1, 0.145, 0.286, 3.0}, {3, 1, 0.19, 0.38, 4.0},
    {2, 2, 0.27, 0.51, 7.5}, {4, 2, 0.475, 0.68, 10.0}, {5, 2, 0.58, 0.82, 10.0}};
// Where the sequences' token counts are known on the device only, and may be well below n_tok, large tiles that the whole of n_tok would
// fill may lie idle; the estimate is then more in favour of 256 x 128 tiles and smaller ones.  Whole calls with the estimates below and
// above in us: without counts 1 x 4097, D = 4096, r = 1024 96.3 and 77.4, 4 x 1391, r = 832 101.7 and 89.5, 2 x 11255, D = 1024, r = 256
// 37.7 and 32.1; with counts from a half of n_tok on, 6 x 830, D = 4096, r = 896 76.3 and 80.7, 6 x 1101, D = 1024, r = 576 26.6 and 28.1.
constexpr PrefillTile kPrefillTilesCounts[] = {
    {1, 1, 0.105, 0.20, 2.0}, {2, 1, 0.145, 0.286, 3.0}, {3, 1, 0.19, 0.38, 4.0},
    {2, 2, 0.255, 0.45, 6.0}, {4, 2, 0.475, 0.68, 12.0}, {5, 2, 0.58, 0.82, 13.0}};
struct PrefillPlan { PrefillTile main, tail; int tail_max; };  // tail_max == 0: all tiles alike
PrefillPlan plan_prefill(const sals_desc& d, int n_tok, bool counts)
{
    const auto& tiles_of = counts ? kPrefillTilesCounts : kPrefillTiles;
    PrefillPlan best{tiles_of[0], tiles_of[0], 0};
    double best_us = 1e30;
    const double steps = (double)(d.H_kv * d.d) / 32.0;
    auto rounds_us = [&](const PrefillTile& t, double tiles) {
        const double rounds = std::floor(tiles / 256.0), rest = tiles / 256.0 - rounds;
        return rounds * (steps * t.full + t.over) + (rest > 0.0 ? steps * (t.idle + (t.full - t.idle) * rest) + t.over : 0.0);
    };
    auto per_row_tile = [&](const PrefillTile& t) { return ceil_div(d.r, 64 * t.nbw) * 2; };
    for (const PrefillTile& t : tiles_of) {
        const long long row_tiles = ((long long)d.B * n_tok + 128 * t.nbt - 1) / (128 * t.nbt);
        const int per = per_row_tile(t);
        const double us = rounds_us(t, (double)row_tiles * per);
        if (us < best_us) { best_us = us; best = PrefillPlan{t, t, 0}; }
        if (t.nbt != 2) continue;
        const long long whole = row_tiles * per / 256 * 256 / per;
        if (whole == 0 || whole == row_tiles) continue;
        for (const PrefillTile& u : tiles_of) {
            if (u.nbt != 1) continue;
            const double us2 = rounds_us(t, (double)whole * per) + rounds_us(u, (double)(row_tiles - whole) * 2 * per_row_tile(u));
            // (the token counts may be smaller than n_tok: the tail is used for any rest up to this one or two thirds of a round)
            if (us2 < best_us) { best_us = us2; best = PrefillPlan{t, u, std::max((int)(row_tiles - whole), 171 / per)}; }
        }
    }
    return best;
}
}  // namespace

sals_status sals_compress_prefill(sals_ctx* ctx, const void* k_new, const void* v_new, const void* W, void* Kc,
                                  void* Vc, int32_t* seq_len, const int32_t* n_new, int32_t n_tok, void* hip_stream)
{
    if (!ctx || bad(k_new) || bad(v_new) || bad(W) || bad(Kc) || bad(Vc) || !seq_len) return SALS_ERR_INVALID_ARG;
    if (n_tok < 1 || n_tok > ctx->d.S_max) return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const sals_desc& d = ctx->d;
    const bool bf = d.dtype == SALS_BF16;
    PrefillArgs a{};
    a.X[0] = k_new; a.X[1] = v_new;
    a.cache[0] = Kc; a.cache[1] = Vc;
    a.seq_len = seq_len; a.n_new = n_new;
    a.n_tok = n_tok; a.D = d.H_kv * d.d; a.r = d.r; a.S_max = d.S_max; a.B = d.B; a.nproj = 2;
    for (int p = 0; p < 2; ++p)
        a.UT[p] = bf ? static_cast<const void*>(w_section<bf16_t>(ctx, W, p)) : static_cast<const void*>(w_section<float>(ctx, W, p));
    auto allow = [](const void* kern, size_t lds) {
        return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
    };
    a.arrived = arrivals(ctx);
    ProfScope ps(ctx, SALS_K_PREFILL, st);
    if (bf) {
        const PrefillPlan P = plan_prefill(d, n_tok, n_new != nullptr);
        const PrefillTile t = P.main;
        const int n_col = ceil_div(d.r, 64 * t.nbw), tm = 128 * t.nbt;
        // every token tile a batch of these sizes can have (workgroups past the tiles that hold tokens leave)
        const int n_tiles = n_new ? d.B * ceil_div(n_tok, tm) : (int)(((long long)d.B * n_tok + tm - 1) / tm);
        if (P.tail_max == 0) {
            a.n_wg = n_tiles * 2 * n_col;
#define SALS_PREFILL(N, T)                                                                                              \
            if (t.nbw == N && t.nbt == T) {                                                                             \
                auto kern = prefill_tile_kernel<N, T>;                                                                  \
                constexpr size_t lds = pf_cfg<N, T>::LDS;                                                               \
                if (!allow(reinterpret_cast<const void*>(kern), lds)) return SALS_ERR_HIP;                              \
                hipLaunchKernelGGL(kern, dim3(a.n_wg), dim3(kPfThreads), lds, st, a, n_col);                            \
            }
            SALS_PREFILL(1, 1) SALS_PREFILL(2, 1) SALS_PREFILL(3, 1) SALS_PREFILL(2, 2) SALS_PREFILL(4, 2) SALS_PREFILL(5, 2)
        } else {
            const int n_col_rest = ceil_div(d.r, 64 * P.tail.nbw), n_rest = std::min(n_tiles, P.tail_max) * 2 * 2 * n_col_rest;
            const int n_big = ceil_div(n_tiles * 2 * n_col, kXcds) * kXcds;  // (either kind is dealt to the XCDs from the first on)
            a.n_wg = n_big + n_rest;
#define SALS_PREFILL_SPLIT(N, U)                                                                                        \
            if (t.nbw == N && P.tail.nbw == U) {                                                                        \
                auto kern = prefill_split_kernel<N, U>;                                                                 \
                constexpr size_t lds = std::max(pf_cfg<N, 2>::LDS, pf_cfg<U, 1>::LDS);                                  \
                if (!allow(reinterpret_cast<const void*>(kern), lds)) return SALS_ERR_HIP;                              \
                hipLaunchKernelGGL(kern, dim3(a.n_wg), dim3(kPfThreads), lds, st, a, n_col, n_big, n_col_rest,   \
                                   P.tail_max);                                                                         \
            }
            SALS_PREFILL_SPLIT(2, 1) SALS_PREFILL_SPLIT(2, 2) SALS_PREFILL_SPLIT(2, 3) SALS_PREFILL_SPLIT(4, 1) SALS_PREFILL_SPLIT(4, 2)
            SALS_PREFILL_SPLIT(4, 3) SALS_PREFILL_SPLIT(5, 1) SALS_PREFILL_SPLIT(5, 2) SALS_PREFILL_SPLIT(5, 3)
        }
        if (launch_status() != SALS_OK) return SALS_ERR_HIP;
#undef SALS_PREFILL_SPLIT
#undef SALS_PREFILL
    } else {
        const int nl = d.r % 128 == 0 ? 128 : 64;
        // 256-token tiles unless they would fill less than three quarters of the chip's 512 workgroup slots
        const int tok = (nl == 128 && (long long)ceil_div(n_tok, 256) * (d.r / nl) * d.B * 2 < 384) ? 128 : 256;
        const dim3 grid(ceil_div(n_tok, tok), d.r / nl, d.B * 2);
        a.n_wg = grid.x * grid.y * grid.z;
        const size_t lds = prefill_lds_bytes(tok, nl);
        auto kern = nl == 64 ? prefill_compress_kernel<256, 64>
                             : (tok == 128 ? prefill_compress_kernel<128, 128> : prefill_compress_kernel<256, 128>);
        if (!allow(reinterpret_cast<const void*>(kern), lds)) return SALS_ERR_HIP;
        hipLaunchKernelGGL(kern, grid, dim3(kPfThreads), lds, st, a);
    }
    if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    if (a.arrived) return SALS_OK;
    hipLaunchKernelGGL(advance_seq_len_kernel, dim3(ceil_div(d.B, 128)), dim3(128), 0, st, seq_len, n_new, n_tok, d.B, d.S_max);
    return launch_status();
}

sals_status sals_latent_scores(sals_ctx* ctx, const void* q, const void* W, const void* Kc,
                               const int32_t* seq_len, float* scores, void* hip_stream)
{
    if (!ctx || bad(q) || bad(W) || bad(Kc) || !seq_len || bad(scores)) return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    sals_status s = ctx->d.dtype == SALS_BF16
                        ? launch_project<bf16_t>(ctx, W, q, st)
                        : launch_project<float>(ctx, W, q, st);
    if (s != SALS_OK) return s;
    return ctx->d.dtype == SALS_BF16 ? launch_scores<bf16_t>(ctx, Kc, seq_len, scores, st)
                                     : launch_scores<float>(ctx, Kc, seq_len, scores, st);
}

namespace {
// The score stage inside a decode step: as sals_latent_scores, and for sequences long enough for the selection
// chain the score kernel also leaves its workgroups' key ranges for it.
sals_status step_scores(sals_ctx* ctx, const void* q, const void* W, const void* Kc, const int32_t* seq_len,
                        float* scores, hipStream_t st)
{
    if (!ctx || bad(q) || bad(W) || bad(Kc) || !seq_len || bad(scores)) return SALS_ERR_INVALID_ARG;
    sals_status s = ctx->d.dtype == SALS_BF16
                        ? launch_project<bf16_t>(ctx, W, q, st)
                        : launch_project<float>(ctx, W, q, st);
    if (s != SALS_OK) return s;
    uint2* wg_range = ctx->L.tm_chunks > 0 ? reinterpret_cast<uint2*>(ctx->ws + ctx->L.tm_srange) : nullptr;
    return ctx->d.dtype == SALS_BF16 ? launch_scores<bf16_t>(ctx, Kc, seq_len, scores, st, wg_range)
                                     : launch_scores<float>(ctx, Kc, seq_len, scores, st, wg_range);
}
}  // namespace

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices];  // per device: address of `scratch` there (nullptr: not looked up yet)

// address of the current device's copy of `scratch`; looked up once per device, with that device current
sals_status scratch_on_current_device(unsigned char** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SALS_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return SALS_ERR_HIP;
        g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
    }
    *out = g_scratch_ptr[dev];
    return SALS_OK;
}
}  // namespace

sals_status sals_latent_scores_noalloc(const sals_desc* desc, const void* q, const void* W, const void* Kc,
                                       const int32_t* seq_len, float* scores, void* hip_stream)
{
    sals_status s = validate(desc);
    if (s != SALS_OK) return s;
    if (bad(q) || bad(W) || bad(Kc) || !seq_len || bad(scores)) return SALS_ERR_INVALID_ARG;
    // a context on the stack whose "workspace" is the static array: these two launches only use the slot of
    // the partial sums of q~, placed at offset 0
    sals_ctx tmp;
    tmp.d = *desc;
    tmp.L = make_layout(*desc);
    tmp.L.qt = 0;
    tmp.score_rows = plan_score_rows(*desc);
    const size_t need = (size_t)tmp.L.proj_np * desc->B * desc->r * 4;
    if (need > (size_t)SALS_NOALLOC_SCRATCH_BYTES) return SALS_ERR_WORKSPACE;
    s = scratch_on_current_device(&tmp.ws);
    if (s != SALS_OK) return s;
    tmp.ws_bytes = SALS_NOALLOC_SCRATCH_BYTES;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    s = desc->dtype == SALS_BF16 ? launch_project<bf16_t>(&tmp, W, q, st)
                                 : launch_project<float>(&tmp, W, q, st);
    if (s != SALS_OK) return s;
    return desc->dtype == SALS_BF16 ? launch_scores<bf16_t>(&tmp, Kc, seq_len, scores, st)
                                    : launch_scores<float>(&tmp, Kc, seq_len, scores, st);
}

sals_status sals_topk_select(sals_ctx* ctx, const float* scores, const int32_t* seq_len, int32_t* idx,
                             int32_t* n_sel, void* hip_stream)
{
    if (!ctx || bad(scores) || !seq_len || !idx || !n_sel) return SALS_ERR_INVALID_ARG;
    return launch_topk(ctx, scores, seq_len, idx, n_sel, static_cast<hipStream_t>(hip_stream));
}

sals_status sals_sparse_attend(sals_ctx* ctx, const void* q, const int32_t* q_pos, const void* Kc,
                               const void* Vc, const void* W, const int32_t* idx, const int32_t* n_sel,
                               void* out, void* hip_stream)
{
    if (!ctx || bad(q) || !q_pos || bad(Kc) || bad(Vc) || bad(W) || !idx || !n_sel || bad(out))
        return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    return ctx->d.dtype == SALS_BF16 ? launch_attend<bf16_t>(ctx, q, q_pos, Kc, Vc, W, idx, n_sel, out, st)
                                     : launch_attend<float>(ctx, q, q_pos, Kc, Vc, W, idx, n_sel, out, st);
}

sals_status sals_decode_step(sals_ctx* ctx, const void* q, const int32_t* q_pos, const void* Kc,
                             const void* Vc, const void* W, const int32_t* seq_len, void* out, float* scores,
                             int32_t* idx, int32_t* n_sel, void* hip_stream)
{
    if (!ctx || bad(q) || !q_pos || bad(Kc) || bad(Vc) || bad(W) || !seq_len || bad(out))
        return SALS_ERR_INVALID_ARG;
    if (scores && !aligned16(scores)) return SALS_ERR_INVALID_ARG;
    if (!scores) scores = reinterpret_cast<float*>(ctx->ws + ctx->L.scores);
    if (!idx) idx = reinterpret_cast<int32_t*>(ctx->ws + ctx->L.idx);
    if (!n_sel) n_sel = reinterpret_cast<int32_t*>(ctx->ws + ctx->L.n_sel);
    sals_status s = step_scores(ctx, q, W, Kc, seq_len, scores, static_cast<hipStream_t>(hip_stream));
    if (s != SALS_OK) return s;
    if (fused_selection(ctx)) {  // one launch fewer: the logits kernel selects and leaves idx / n_sel behind
        if (bad(Vc)) return SALS_ERR_INVALID_ARG;
        const FusedSelect fs{scores, seq_len, ctx->d.top_k, ctx->d.n_sink, ctx->d.n_recent};
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        return ctx->d.dtype == SALS_BF16
                   ? launch_attend<bf16_t>(ctx, q, q_pos, Kc, Vc, W, idx, n_sel, out, st, nullptr, 0, kPhaseAll, nullptr, &fs)
                   : launch_attend<float>(ctx, q, q_pos, Kc, Vc, W, idx, n_sel, out, st, nullptr, 0, kPhaseAll, nullptr, &fs);
    }
    s = launch_topk(ctx, scores, seq_len, idx, n_sel, static_cast<hipStream_t>(hip_stream),
                    WindowLists{nullptr, nullptr, nullptr, 0}, true);
    if (s != SALS_OK) return s;
    if (step_resolves(ctx)) {
        if (bad(Vc)) return SALS_ERR_INVALID_ARG;
        const TopkResolve res = topk_resolve(ctx, idx);
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        return ctx->d.dtype == SALS_BF16 ? launch_attend<bf16_t>(ctx, q, q_pos, Kc, Vc, W, idx, n_sel, out, st, nullptr, 0, kPhaseAll,
                                                                 nullptr, nullptr, nullptr, &res)
                                         : launch_attend<float>(ctx, q, q_pos, Kc, Vc, W, idx, n_sel, out, st, nullptr, 0, kPhaseAll,
                                                                nullptr, nullptr, nullptr, &res);
    }
    return sals_sparse_attend(ctx, q, q_pos, Kc, Vc, W, idx, n_sel, out, hip_stream);
}

sals_status sals_qv_row_bytes(const sals_desc* desc, int bits, size_t* code_bytes, size_t* meta_bytes)
{
    if (!code_bytes || !meta_bytes) return SALS_ERR_INVALID_ARG;
    sals_status s = validate(desc);
    if (s != SALS_OK) return s;
    if (bits != 2 && bits != 4) return SALS_ERR_UNSUPPORTED;
    const size_t D = (size_t)desc->H_kv * desc->d;
    *code_bytes = D * bits / 8;
    *meta_bytes = D / kQvGroup * 2 * (desc->dtype == SALS_BF16 ? 2 : 4);
    return SALS_OK;
}

sals_status sals_compress_append_qv(sals_ctx* ctx, const void* k_new, const void* v_new, const void* W, void* Kc,
                                    void* Vq, void* Vmeta, int bits, int32_t* seq_len, void* hip_stream)
{
    if (!ctx || bad(k_new) || bad(v_new) || bad(W) || bad(Kc) || bad(Vq) || bad(Vmeta) || !seq_len)
        return SALS_ERR_INVALID_ARG;
    if (bits != 2 && bits != 4) return SALS_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const QuantArgs qa{v_new, Vq, Vmeta, bits};
    return ctx->d.dtype == SALS_BF16 ? launch_append<bf16_t>(ctx, W, k_new, nullptr, Kc, nullptr, qa, seq_len, st, true)
                                     : launch_append<float>(ctx, W, k_new, nullptr, Kc, nullptr, qa, seq_len, st, true);
}

sals_status sals_sparse_attend_qv(sals_ctx* ctx, const void* q, const int32_t* q_pos, const void* Kc,
                                  const void* Vq, const void* Vmeta, int bits, const void* W, const int32_t* idx,
                                  const int32_t* n_sel, void* out, void* hip_stream)
{
    if (!ctx || bad(q) || !q_pos || bad(Kc) || bad(Vq) || bad(Vmeta) || bad(W) || !idx || !n_sel || bad(out))
        return SALS_ERR_INVALID_ARG;
    if (bits != 2 && bits != 4) return SALS_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const QvCache qv{Vq, Vmeta, bits};
    return ctx->d.dtype == SALS_BF16 ? launch_attend<bf16_t>(ctx, q, q_pos, Kc, nullptr, W, idx, n_sel, out, st, &qv)
                                     : launch_attend<float>(ctx, q, q_pos, Kc, nullptr, W, idx, n_sel, out, st, &qv);
}

sals_status sals_decode_step_qv(sals_ctx* ctx, const void* q, const int32_t* q_pos, const void* Kc,
                                const void* Vq, const void* Vmeta, int bits, const void* W, const int32_t* seq_len,
                                void* out, float* scores, int32_t* idx, int32_t* n_sel, void* hip_stream)
{
    if (!ctx || bad(q) || !q_pos || bad(Kc) || bad(Vq) || bad(Vmeta) || bad(W) || !seq_len || bad(out))
        return SALS_ERR_INVALID_ARG;
    if (bits != 2 && bits != 4) return SALS_ERR_UNSUPPORTED;
    if (scores && !aligned16(scores)) return SALS_ERR_INVALID_ARG;
    if (!scores) scores = reinterpret_cast<float*>(ctx->ws + ctx->L.scores);
    if (!idx) idx = reinterpret_cast<int32_t*>(ctx->ws + ctx->L.idx);
    if (!n_sel) n_sel = reinterpret_cast<int32_t*>(ctx->ws + ctx->L.n_sel);
    sals_status s = step_scores(ctx, q, W, Kc, seq_len, scores, static_cast<hipStream_t>(hip_stream));
    if (s != SALS_OK) return s;
    if (fused_selection(ctx)) {  // one launch fewer: the logits kernel selects and leaves idx / n_sel behind
        const FusedSelect fs{scores, seq_len, ctx->d.top_k, ctx->d.n_sink, ctx->d.n_recent};
        const QvCache qv{Vq, Vmeta, bits};
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        return ctx->d.dtype == SALS_BF16
                   ? launch_attend<bf16_t>(ctx, q, q_pos, Kc, nullptr, W, idx, n_sel, out, st, &qv, 0, kPhaseAll, nullptr, &fs)
                   : launch_attend<float>(ctx, q, q_pos, Kc, nullptr, W, idx, n_sel, out, st, &qv, 0, kPhaseAll, nullptr, &fs);
    }
    s = launch_topk(ctx, scores, seq_len, idx, n_sel, static_cast<hipStream_t>(hip_stream),
                    WindowLists{nullptr, nullptr, nullptr, 0}, true);
    if (s != SALS_OK) return s;
    if (step_resolves(ctx)) {
        const QvCache qv{Vq, Vmeta, bits};
        const TopkResolve res = topk_resolve(ctx, idx);
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        return ctx->d.dtype == SALS_BF16 ? launch_attend<bf16_t>(ctx, q, q_pos, Kc, nullptr, W, idx, n_sel, out, st, &qv, 0, kPhaseAll,
                                                                 nullptr, nullptr, nullptr, &res)
                                         : launch_attend<float>(ctx, q, q_pos, Kc, nullptr, W, idx, n_sel, out, st, &qv, 0, kPhaseAll,
                                                                nullptr, nullptr, nullptr, &res);
    }
    return sals_sparse_attend_qv(ctx, q, q_pos, Kc, Vq, Vmeta, bits, W, idx, n_sel, out, hip_stream);
}

sals_status sals_dense_attend(sals_ctx* ctx, const void* q, const int32_t* q_pos, const void* K, const void* V,
                              const int32_t* seq_len, void* out, void* hip_stream)
{
    if (!ctx || bad(q) || !q_pos || bad(K) || bad(V) || !seq_len || bad(out)) return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    return ctx->d.dtype == SALS_BF16 ? launch_dense<bf16_t>(ctx, q, q_pos, K, V, seq_len, out, st)
                                     : launch_dense<float>(ctx, q, q_pos, K, V, seq_len, out, st);
}

// ---- recent window (second, higher-rank ring cache) ------------------------------------------------

namespace {
// `win` must describe the same model and batch as `ctx`, at another rank, and select exactly the recent tokens
sals_status window_pair_ok(const sals_ctx* ctx, const sals_ctx* win)
{
    if (!ctx || !win || ctx == win) return SALS_ERR_INVALID_ARG;
    const sals_desc &a = ctx->d, &b = win->d;
    if (a.B != b.B || a.S_max != b.S_max || a.H_q != b.H_q || a.H_kv != b.H_kv || a.d != b.d ||
        a.rope_theta != b.rope_theta || a.rope_style != b.rope_style || a.dtype != b.dtype)
        return SALS_ERR_INVALID_ARG;
    if (b.n_sink != 0 || b.n_recent != 0 || a.n_recent < 1 || b.top_k != a.n_recent) return SALS_ERR_INVALID_ARG;
    return SALS_OK;
}
}  // namespace

sals_status sals_window_append(sals_ctx* win, const void* k_new, const void* v_new, const void* W_hi, void* Kw,
                               void* Vw, const int32_t* seq_len, void* hip_stream)
{
    if (!win || bad(k_new) || bad(v_new) || bad(W_hi) || bad(Kw) || bad(Vw) || !seq_len) return SALS_ERR_INVALID_ARG;
    if (win->d.n_sink != 0 || win->d.n_recent != 0) return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int32_t* sl = const_cast<int32_t*>(seq_len);  // read only: no length is advanced here
    const int ring = win->d.top_k;
    return win->d.dtype == SALS_BF16
               ? launch_append<bf16_t>(win, W_hi, k_new, v_new, Kw, Vw, QuantArgs{}, sl, st, false, ring)
               : launch_append<float>(win, W_hi, k_new, v_new, Kw, Vw, QuantArgs{}, sl, st, false, ring);
}

}  // extern "C"

namespace {
// where the two passes' token lists live: the window's list and count in the window context's workspace, the
// low-rank pass's count in the main context's
WindowLists window_lists(sals_ctx* ctx, sals_ctx* win)
{
    return WindowLists{reinterpret_cast<int32_t*>(win->ws + win->L.idx), reinterpret_cast<int32_t*>(ctx->ws + ctx->L.n_lo),
                       reinterpret_cast<int32_t*>(win->ws + win->L.n_sel), win->d.top_k};
}

// where the two passes leave their tile statistics: side by side in the main context's array
StatsLink window_stats(sals_ctx* ctx, sals_ctx* win, bool hi)
{
    return StatsLink{reinterpret_cast<float2*>(ctx->ws + ctx->L.stats), ctx->plan.n_parts + win->plan.n_parts, hi ? ctx->plan.n_parts : 0};
}

// A step's selection together with the window's logits.
bool window_select_fits(const sals_ctx* ctx, const sals_ctx* win)
{
    return window_in_select(win) && ctx->plan.n_parts + win->plan.n_parts <= ctx->L.max_parts;
}
template <typename T>
sals_status launch_window_select(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos, const void* Kw, const void* W_hi,
                                 const float* scores, const int32_t* seq_len, int32_t* idx, int32_t* n_sel, hipStream_t st)
{
    const sals_desc &d = ctx->d, &e = win->d;
    const Layout& L = win->L;
    sals_status s = ensure_rope_table(win, st);
    if (s == SALS_OK) s = ensure_lds_attr<T>(win);
    if (s != SALS_OK) return s;
    const StatsLink link = window_stats(ctx, win, true);
    const StepSelect sel{scores, seq_len, idx, n_sel, select_blocks(d), d.B, d.S_max, d.top_k, d.n_sink, d.n_recent, window_lists(ctx, win)};
    const float2* rope = reinterpret_cast<const float2*>(win->ws + L.rope);
    float* logits = reinterpret_cast<float*>(win->ws + L.logits);
    float* plogits = reinterpret_cast<float*>(win->ws + L.plogits);
    const float scale = 1.0f / std::sqrt((float)e.d);
    const int w = e.top_k, ks = window_slices(win);
    float2* stats = link.stats + link.part0;
    ProfScope ps(ctx, SALS_K_TOPK, st);
    if (win->plan.pick == 4) {
        typedef logits_cfg<1, 4, 1> LC;
        typedef logits_cfg<2, 4, 2> WC;   // wide tiles
        const bool wide = wide_window_slices(win) > 0;
        auto kern = window_select_for<T>(e.H_q / e.H_kv, wide);
        static_assert(LC::NT == 256 && WC::NT == 512 && LC::LDS >= sizeof(TopkShared), "the selection runs in the logits kernel's workgroup");
        const int tiles = wide ? ceil_div(e.B, 4) * (e.H_kv / 2) : ceil_div(e.B, 2) * e.H_kv;
        hipLaunchKernelGGL(kern, dim3(sel.n_blocks + tiles * ks), dim3(wide ? WC::NT : LC::NT), wide ? WC::LDS : LC::LDS, st, sel,
                           static_cast<const T*>(Kw), w_section<T>(win, W_hi, 2), static_cast<const T*>(q), q_pos, rope, win->inv, logits,
                           stats, e.B, e.S_max, e.r, e.H_q, e.H_kv, w, L.lk, e.rope_style, scale, link.stride, plogits, ks);
    } else {
        const size_t a_bytes = (size_t)e.H_kv * kHeadDim * e.r, b_bytes = (size_t)e.B * w * e.r;
        auto kern = WindowSelectSmall<T>::get(steps_ahead<T>(e, ks));
        hipLaunchKernelGGL(kern, dim3(sel.n_blocks + win->plan.n_parts * e.H_kv * e.B * ks), dim3(kLsThreads), kLsLds, st, sel,
                           w_section<T>(win, W_hi, 2), e.B, e.H_kv, win->plan.n_parts, a_bytes <= b_bytes ? 1 : 0, ks, w, e.r, e.H_q,
                           static_cast<const T*>(Kw), static_cast<const T*>(q), q_pos, rope, win->inv, logits, stats, e.S_max, L.lk,
                           e.rope_style, scale, plogits, link.stride);
    }
    return launch_status();
}

// The two logits passes.  have: what the step's selection has already done.
enum WindowHave { kWindowNothing, kWindowLists, kWindowListsUnranked, kWindowLogits };
template <typename T>
sals_status window_logits(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos, const void* Kc, const void* W, const void* Kw,
                          const void* W_hi, const int32_t* idx, const int32_t* n_sel, hipStream_t st, WindowHave have)
{
    const sals_desc& d = ctx->d;
    const TopkResolve res = topk_resolve(ctx, const_cast<int32_t*>(idx));  // (the step's own list where it is used)
    const WindowLists wl = window_lists(ctx, win);
    const int w = win->d.top_k;
    if (ctx->plan.n_parts + win->plan.n_parts > ctx->L.max_parts) return SALS_ERR_UNSUPPORTED;
    if (have == kWindowNothing) {
        hipLaunchKernelGGL(window_split_kernel, dim3(d.B), dim3(256), 0, st, idx, n_sel, d.top_k + d.n_sink + d.n_recent, w, wl.idx_hi,
                           wl.n_lo, wl.n_hi);
        if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    }
    const StatsLink lo = window_stats(ctx, win, false), hi = window_stats(ctx, win, true);
    SplitLogits split{};
    if (have == kWindowLogits) {
        const int ks = window_slices(win);
        if (ks > 1) split = split_logits(win, ks, wl.n_hi, hi.stats + hi.part0, hi.stride);
        if (ks > 1 && ctx->plan.pick == 4) {  // (tiles of several sequences do not add up on the side)
            hipLaunchKernelGGL(logits_finish_kernel, dim3(split.n_parts, split.rows), dim3(64), 0, st, split);
            if (launch_status() != SALS_OK) return SALS_ERR_HIP;
        }
    }
    const sals_status s = launch_attend<T>(ctx, q, q_pos, Kc, nullptr, W, idx, wl.n_lo, nullptr, st, nullptr, 0, kPhaseLogits, &lo,
                                           nullptr, split.ksplit > 1 && ctx->plan.pick != 4 ? &split : nullptr,
                                           have == kWindowListsUnranked ? &res : nullptr);
    if (s != SALS_OK || have == kWindowLogits) return s;
    return launch_attend<T>(win, q, q_pos, Kw, nullptr, W_hi, wl.idx_hi, wl.n_hi, nullptr, st, nullptr, w, kPhaseLogits, &hi);
}

// selection of a decode step and, where they go together, the window's logits
sals_status window_step_select(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos, const void* Kw, const void* W_hi,
                               const float* scores, const int32_t* seq_len, int32_t* idx, int32_t* n_sel, hipStream_t st, WindowHave* have)
{
    if (window_select_fits(ctx, win)) {
        *have = kWindowLogits;
        return ctx->d.dtype == SALS_BF16
                   ? launch_window_select<bf16_t>(ctx, win, q, q_pos, Kw, W_hi, scores, seq_len, idx, n_sel, st)
                   : launch_window_select<float>(ctx, win, q, q_pos, Kw, W_hi, scores, seq_len, idx, n_sel, st);
    }
    // the selection kernel also writes the two passes' token lists (they follow from the sequence lengths)
    *have = step_resolves(ctx) ? kWindowListsUnranked : kWindowLists;
    return launch_topk(ctx, scores, seq_len, idx, n_sel, st, window_lists(ctx, win), true);
}

sals_status window_attend(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos, const void* Kc,
                          const void* Vc, const void* W, const void* Kw, const void* Vw, const void* W_hi,
                          const int32_t* idx, const int32_t* n_sel, void* out, hipStream_t st, WindowHave have)
{
    const sals_desc& d = ctx->d;
    const int w = win->d.top_k;
    const WindowLists wl = window_lists(ctx, win);
    int32_t* idx_hi = wl.idx_hi;
    int32_t* n_hi = wl.n_hi;
    int32_t* n_lo = wl.n_lo;
    // One softmax over both caches: the two logits passes leave their tile statistics side by side in the main
    // context's array, each value pass normalises with the statistics of all tiles, and one output projection adds
    // both passes' value sums through their projectors.
    const bool bf = d.dtype == SALS_BF16;
    const sals_status s = bf ? window_logits<bf16_t>(ctx, win, q, q_pos, Kc, W, Kw, W_hi, idx, n_sel, st, have)
                             : window_logits<float>(ctx, win, q, q_pos, Kc, W, Kw, W_hi, idx, n_sel, st, have);
    if (s != SALS_OK) return s;
    const StatsLink l_lo = window_stats(ctx, win, false);
    {
        const PvPass lo{ctx, idx, n_lo, Vc, 0}, hi{win, idx_hi, n_hi, Vw, w};
        if (bf) launch_pv<bf16_t>(ctx, l_lo.stats, l_lo.stride, lo, &hi, nullptr, st);
        else launch_pv<float>(ctx, l_lo.stats, l_lo.stride, lo, &hi, nullptr, st);
        if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    }
    {
        ProfScope ps(ctx, SALS_K_ATTEND_OUT, st);
        const float* t_lo = reinterpret_cast<const float*>(ctx->ws + ctx->L.tpart);
        const float* t_hi = reinterpret_cast<const float*>(win->ws + win->L.tpart);
        if (bf)
            launch_out<bf16_t>(st, d, ctx->L.pv_ntr, w_section<bf16_t>(ctx, W, 3), t_lo, win->d.r, win->L.pv_ntr,
                               w_section<bf16_t>(win, W_hi, 3), t_hi, out);
        else
            launch_out<float>(st, d, ctx->L.pv_ntr, w_section<float>(ctx, W, 3), t_lo, win->d.r, win->L.pv_ntr,
                              w_section<float>(win, W_hi, 3), t_hi, out);
    }
    return launch_status();
}
}  // namespace

extern "C" {

sals_status sals_sparse_attend_window(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos,
                                      const void* Kc, const void* Vc, const void* W, const void* Kw,
                                      const void* Vw, const void* W_hi, const int32_t* idx, const int32_t* n_sel,
                                      void* out, void* hip_stream)
{
    sals_status s = window_pair_ok(ctx, win);
    if (s != SALS_OK) return s;
    if (bad(q) || !q_pos || bad(Kc) || bad(Vc) || bad(W) || bad(Kw) || bad(Vw) || bad(W_hi) || !idx || !n_sel ||
        bad(out))
        return SALS_ERR_INVALID_ARG;
    return window_attend(ctx, win, q, q_pos, Kc, Vc, W, Kw, Vw, W_hi, idx, n_sel, out, static_cast<hipStream_t>(hip_stream),
                         kWindowNothing);
}

sals_status sals_decode_step_window(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos,
                                    const void* Kc, const void* Vc, const void* W, const void* Kw, const void* Vw,
                                    const void* W_hi, const int32_t* seq_len, void* out, float* scores,
                                    int32_t* idx, int32_t* n_sel, void* hip_stream)
{
    sals_status s = window_pair_ok(ctx, win);
    if (s != SALS_OK) return s;
    if (bad(q) || !q_pos || bad(Kc) || bad(Vc) || bad(W) || bad(Kw) || bad(Vw) || bad(W_hi) || !seq_len || bad(out))
        return SALS_ERR_INVALID_ARG;
    if (scores && !aligned16(scores)) return SALS_ERR_INVALID_ARG;
    if (!scores) scores = reinterpret_cast<float*>(ctx->ws + ctx->L.scores);
    if (!idx) idx = reinterpret_cast<int32_t*>(ctx->ws + ctx->L.idx);
    if (!n_sel) n_sel = reinterpret_cast<int32_t*>(ctx->ws + ctx->L.n_sel);
    s = step_scores(ctx, q, W, Kc, seq_len, scores, static_cast<hipStream_t>(hip_stream));
    if (s != SALS_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    WindowHave have;
    s = window_step_select(ctx, win, q, q_pos, Kw, W_hi, scores, seq_len, idx, n_sel, st, &have);
    if (s != SALS_OK) return s;
    return window_attend(ctx, win, q, q_pos, Kc, Vc, W, Kw, Vw, W_hi, idx, n_sel, out, st, have);
}

// ---- recent window of the quantised value path: keys in the rank-r_hi ring, values as 8-bit codes ----

sals_status sals_window_append_qv(sals_ctx* win, const void* k_new, const void* v_new, const void* W_hi, void* Kw,
                                  void* Vqw, void* Vmeta_w, const int32_t* seq_len, void* hip_stream)
{
    if (!win || bad(k_new) || bad(v_new) || bad(W_hi) || bad(Kw) || bad(Vqw) || bad(Vmeta_w) || !seq_len)
        return SALS_ERR_INVALID_ARG;
    if (win->d.n_sink != 0 || win->d.n_recent != 0) return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    int32_t* sl = const_cast<int32_t*>(seq_len);  // read only: no length is advanced here
    const QuantArgs qa{v_new, Vqw, Vmeta_w, 8};
    const int ring = win->d.top_k;
    return win->d.dtype == SALS_BF16 ? launch_append<bf16_t>(win, W_hi, k_new, nullptr, Kw, nullptr, qa, sl, st, false, ring)
                                     : launch_append<float>(win, W_hi, k_new, nullptr, Kw, nullptr, qa, sl, st, false, ring);
}

namespace {
sals_status window_attend_qv(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos, const void* Kc,
                             const void* Vq, const void* Vmeta, int bits, const void* W, const void* Kw, const void* Vqw,
                             const void* Vmeta_w, const void* W_hi, const int32_t* idx, const int32_t* n_sel, void* out,
                             hipStream_t st, WindowHave have)
{
    const sals_desc& d = ctx->d;
    const int w = win->d.top_k;
    const WindowLists wl = window_lists(ctx, win);
    // two logits passes (low-rank cache, ring) with their tile statistics side by side, then one pass over the values
    // of the whole selection: the tokens before the window from the low-bit cache, the window's from its 8-bit ring
    const bool bf = d.dtype == SALS_BF16;
    const sals_status s = bf ? window_logits<bf16_t>(ctx, win, q, q_pos, Kc, W, Kw, W_hi, idx, n_sel, st, have)
                             : window_logits<float>(ctx, win, q, q_pos, Kc, W, Kw, W_hi, idx, n_sel, st, have);
    if (s != SALS_OK) return s;
    const StatsLink l_lo = window_stats(ctx, win, false);
    QvCache qv{Vq, Vmeta, bits};
    qv.codes_w = Vqw; qv.meta_w = Vmeta_w;
    qv.logits_w = reinterpret_cast<const float*>(win->ws + win->L.logits);
    qv.n_lo = wl.n_lo; qv.lk_w = win->L.lk; qv.ring = w;
    return bf ? launch_attend<bf16_t>(ctx, q, q_pos, Kc, nullptr, W, idx, n_sel, out, st, &qv, 0, 0, &l_lo)
              : launch_attend<float>(ctx, q, q_pos, Kc, nullptr, W, idx, n_sel, out, st, &qv, 0, 0, &l_lo);
}
}  // namespace

sals_status sals_sparse_attend_qv_window(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos,
                                         const void* Kc, const void* Vq, const void* Vmeta, int bits, const void* W,
                                         const void* Kw, const void* Vqw, const void* Vmeta_w, const void* W_hi,
                                         const int32_t* idx, const int32_t* n_sel, void* out, void* hip_stream)
{
    sals_status s = window_pair_ok(ctx, win);
    if (s != SALS_OK) return s;
    if (bad(q) || !q_pos || bad(Kc) || bad(Vq) || bad(Vmeta) || bad(W) || bad(Kw) || bad(Vqw) || bad(Vmeta_w) || bad(W_hi) ||
        !idx || !n_sel || bad(out))
        return SALS_ERR_INVALID_ARG;
    if (bits != 2 && bits != 4) return SALS_ERR_UNSUPPORTED;
    return window_attend_qv(ctx, win, q, q_pos, Kc, Vq, Vmeta, bits, W, Kw, Vqw, Vmeta_w, W_hi, idx, n_sel, out,
                            static_cast<hipStream_t>(hip_stream), kWindowNothing);
}

sals_status sals_decode_step_qv_window(sals_ctx* ctx, sals_ctx* win, const void* q, const int32_t* q_pos,
                                       const void* Kc, const void* Vq, const void* Vmeta, int bits, const void* W,
                                       const void* Kw, const void* Vqw, const void* Vmeta_w, const void* W_hi,
                                       const int32_t* seq_len, void* out, float* scores, int32_t* idx, int32_t* n_sel,
                                       void* hip_stream)
{
    sals_status s = window_pair_ok(ctx, win);
    if (s != SALS_OK) return s;
    if (bad(q) || !q_pos || bad(Kc) || bad(Vq) || bad(Vmeta) || bad(W) || bad(Kw) || bad(Vqw) || bad(Vmeta_w) || bad(W_hi) ||
        !seq_len || bad(out))
        return SALS_ERR_INVALID_ARG;
    if (bits != 2 && bits != 4) return SALS_ERR_UNSUPPORTED;
    if (scores && !aligned16(scores)) return SALS_ERR_INVALID_ARG;
    if (!scores) scores = reinterpret_cast<float*>(ctx->ws + ctx->L.scores);
    if (!idx) idx = reinterpret_cast<int32_t*>(ctx->ws + ctx->L.idx);
    if (!n_sel) n_sel = reinterpret_cast<int32_t*>(ctx->ws + ctx->L.n_sel);
    s = step_scores(ctx, q, W, Kc, seq_len, scores, static_cast<hipStream_t>(hip_stream));
    if (s != SALS_OK) return s;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    WindowHave have;
    s = window_step_select(ctx, win, q, q_pos, Kw, W_hi, scores, seq_len, idx, n_sel, st, &have);
    if (s != SALS_OK) return s;
    return window_attend_qv(ctx, win, q, q_pos, Kc, Vq, Vmeta, bits, W, Kw, Vqw, Vmeta_w, W_hi, idx, n_sel, out, st, have);
}

// ---- overlap score ----------------------------------------------------------------------------------

sals_status sals_overlap_score(sals_ctx* ctx, const void* q, const int32_t* q_pos, const void* K,
                               const int32_t* seq_len, const int32_t* idx, const int32_t* n_sel, float* os,
                               void* hip_stream)
{
    if (!ctx || bad(q) || !q_pos || bad(K) || !seq_len || !idx || !n_sel || !os) return SALS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const sals_desc& d = ctx->d;
    const Layout& L = ctx->L;
    if (ensure_rope_table(ctx, st) != SALS_OK) return SALS_ERR_HIP;
    const int k_tot = d.top_k + d.n_sink + d.n_recent;
    float2* part = reinterpret_cast<float2*>(ctx->ws + L.dn_part);  // the dense baseline's partials: larger
    const float2* rope = reinterpret_cast<const float2*>(ctx->ws + L.rope);
    const int G = d.H_q / d.H_kv;
    const dim3 grid(L.dn_chunks, d.H_kv, d.B);
    const float scale = 1.0f / std::sqrt((float)d.d);
#define SALS_OS(T, GMAX)                                                                                          \
    hipLaunchKernelGGL((overlap_stats_kernel<T, GMAX>), grid, dim3(256), 0, st, static_cast<const T*>(q), q_pos,     \
                       static_cast<const T*>(K), seq_len, idx, n_sel, rope, ctx->inv, part, d.S_max, d.H_q, d.H_kv, \
                       k_tot, L.dn_chunks, L.dn_tok, ceil_div(k_tot, L.dn_chunks), d.rope_style, scale)
#define SALS_OS_G(T)                                                                                              \
    do {                                                                                                          \
        if (G <= 1) SALS_OS(T, 1); else if (G <= 2) SALS_OS(T, 2); else if (G <= 4) SALS_OS(T, 4); else SALS_OS(T, 8); \
    } while (0)
    if (d.dtype == SALS_BF16) SALS_OS_G(bf16_t); else SALS_OS_G(float);
#undef SALS_OS_G
#undef SALS_OS
    if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    hipLaunchKernelGGL(overlap_merge_kernel, dim3(ceil_div(d.B * d.H_q, 256)), dim3(256), 0, st, part, os,
                       d.B * d.H_q, L.dn_chunks);
    return launch_status();
}


}  // extern "C"

// ---- offline calibration (Sec. 4.2) ----------------------------------------------------
namespace {
constexpr int64_t kCalChunk = 4096;  // tokens whose products are summed in fp32 before they are added to the fp64 matrix

// slices of a chunk's token axis (each a separate fp32 output of the GEMM): as many as bring the launch to about two
// workgroups per compute unit, at most 8, every slice at least 256 tokens long
int cal_slices(int D)
{
    const bool big = D % 256 == 0 && D >= 2048;
    const int n = big ? D / 256 : D / 128;
    const int tiles = big ? n * n + n : n * (n + 1) / 2;
    int z = 1;
    while (z < 8 && tiles * z < 512 && kCalChunk / (2 * z) >= 256) z *= 2;
    return z;
}

sals_status calib_accumulate_f32(const void* K, int64_t n_tok, int D, double* C, void* ws, hipStream_t st)
{
    const float* X = static_cast<const float*>(K);
    float* XT = static_cast<float*>(ws);
    float* P = reinterpret_cast<float*>(static_cast<unsigned char*>(ws) + align_up((size_t)D * kCalChunk * 4));
    const bool big = D % 256 == 0 && D >= 2048;  // (below that the larger tile leaves most of the chip without a workgroup)
    const int step_tok = kLgStep / 4;  // tokens per 64-byte step of the contraction axis
    for (int64_t t0 = 0; t0 < n_tok; t0 += kCalChunk) {
        const int64_t n = std::min(kCalChunk, n_tok - t0);
        const int64_t n_pad = (n + 63) / 64 * 64;  // whole 64-byte steps of the contraction axis, zero filled
        hipLaunchKernelGGL(calib_transpose_kernel, dim3((unsigned)(n_pad / kCalTile), (unsigned)ceil_div(D, kCalTile)),
                           dim3(256), 0, st, X + (size_t)t0 * D, XT, (long long)n, D, (long long)n_pad);
        const int steps = (int)(n_pad / step_tok);
        const int per = ceil_div(steps, std::min(cal_slices(D), std::max(1, steps / 2)));  // >= 2 steps per slice
        const int slices = ceil_div(steps, per);
        PrefillArgs a{};
        a.X[0] = XT; a.UT[0] = XT; a.cache[0] = nullptr; a.seq_len = nullptr; a.n_new = nullptr;
        a.n_tok = D; a.D = (int)n_pad; a.r = D; a.S_max = D; a.B = 1; a.nproj = 1; a.pacc = P; a.kslice_steps = per;
        // tiles that reach the upper triangle only (the kernel numbers them row by row)
        if (big) {
            const int nt = D / 256;
            hipLaunchKernelGGL((prefill_compress_kernel<256, 128, true>), dim3(nt * nt + nt, slices, 1), dim3(kPfThreads),
                               prefill_lds_bytes(256, 128), st, a);
        } else {
            const int nt = D / 128;
            hipLaunchKernelGGL((prefill_compress_kernel<128, 128, true>), dim3(nt * (nt + 1) / 2, slices, 1),
                               dim3(kPfThreads), prefill_lds_bytes(128, 128), st, a);
        }
        hipLaunchKernelGGL(calib_reduce_kernel, dim3((unsigned)(((size_t)D * D / 4 + 255) / 256)), dim3(256), 0, st, C, P, D,
                           slices, big ? 256 : 128, 128);
        if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    }
    // the lower triangle from the upper one (which also makes the matrix exactly symmetric)
    hipLaunchKernelGGL(calib_mirror_kernel, dim3(D / 32, D / 32), dim3(256), 0, st, C, D);
    return launch_status();
}

int cov_tiles(int D) { const int nt = ceil_div(D, kCovTile); return nt * (nt + 1) / 2; }
// bf16 keys: slices of the token axis per launch at most (each a separate fp32 output over at most 4096 tokens), so that the
// tile sums of a launch stay near 280 MB
int cov_max_slices(int D) { return std::min(64, std::max(2, 1088 / cov_tiles(D))); }
// Tiles of a first launch, which fill the chip (one workgroup per compute unit) a whole number of times: the second launch has
// the tiles left and, on the compute units that its part of a round leaves idle, the additions of the first.  0: one launch for
// all.  Estimated durations in us: a round 0.95 per 32 tokens and 8 to start and to store a tile; the additions 0.05 per tile and
// slice and 0.3 per tile; 12 for the start and the uneven end of another launch.
int cov_first_tiles(int tiles, int slices, int64_t slice_steps, double* us)
{
    const double round = (double)slice_steps * 0.95 + 8.0, add = 0.05 * slices + 0.3;
    const int whole = tiles * slices / 256, first = whole * 256 / slices, rest = (tiles - first) * slices;
    *us = ceil_div(tiles * slices, 256) * round + add * tiles;
    if (first == 0 || rest == 0 || rest >= 256) return 0;
    const double two = whole * round + std::max(round, add * first * 256 / (256 - rest)) + add * (tiles - first) + 12.0;
    if (two >= *us) return 0;
    *us = two;
    return first;
}
// ... and of a batch of n tokens: the number with the smallest estimated duration
int cov_slices(int D, int64_t n)
{
    const int tiles = cov_tiles(D), lo = (int)((n + kCalChunk - 1) / kCalChunk);
    const int64_t steps = (n + kCovStep - 1) / kCovStep;
    int best = lo;
    double best_us = 1e30;
    for (int s = lo; s <= cov_max_slices(D) && s <= steps; ++s) {
        double us;
        cov_first_tiles(tiles, s, (steps + s - 1) / s, &us);
        if (us < best_us) { best_us = us; best = s; }
    }
    return best;
}
sals_status calib_accumulate_bf16(const void* K, int64_t n_tok, int D, double* C, void* ws, hipStream_t st)
{
    const bf16_t* X = static_cast<const bf16_t*>(K);
    float* P = static_cast<float*>(ws);
    const int nt = ceil_div(D, kCovTile), tiles = cov_tiles(D);
    const int64_t most = kCalChunk * cov_max_slices(D);
    for (int64_t t0 = 0; t0 < n_tok; t0 += most) {
        const int64_t n = std::min(most, n_tok - t0);
        const int64_t steps = (n + kCovStep - 1) / kCovStep;
        const int want = cov_slices(D, n);
        const int slice_tok = (int)((steps + want - 1) / want) * kCovStep;   // (at most 4096: want >= n / 4096)
        const int slices = (int)((n + slice_tok - 1) / slice_tok);
        double us;
        const int first = cov_first_tiles(tiles, slices, slice_tok / kCovStep, &us);
        auto launch = [&](int tile0, int count, int add) {  // tiles' sums, and the additions of the first `add` tiles
            hipLaunchKernelGGL(calib_cov_kernel, dim3(count * slices + add * 32), dim3(512), kCovLds, st, X + (size_t)t0 * D, (long long)n,
                               D, nt, slice_tok, slices, P, tile0, count, C);
        };
        if (first > 0) launch(0, first, 0);
        launch(first, tiles - first, first);
        hipLaunchKernelGGL(calib_cov_reduce_kernel, dim3(64, tiles - first), dim3(256), 0, st, C, P, D, nt, slices, first);
        if (launch_status() != SALS_OK) return SALS_ERR_HIP;
    }
    return SALS_OK;
}

sals_status calib_lds_attr(int32_t dtype)
{
    static std::mutex m;
    static bool done[2][kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SALS_ERR_HIP;
    std::lock_guard<std::mutex> lock(m);
    bool& ok = done[dtype == SALS_BF16][dev];
    if (ok) return SALS_OK;
    auto allow = [](const void* kern, size_t bytes) {
        return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
    };
    if (dtype == SALS_BF16) ok = allow(reinterpret_cast<const void*>(calib_cov_kernel), kCovLds);
    else ok = allow(reinterpret_cast<const void*>(prefill_compress_kernel<256, 128, true>), prefill_lds_bytes(256, 128)) &&
              allow(reinterpret_cast<const void*>(prefill_compress_kernel<128, 128, true>), prefill_lds_bytes(128, 128));
    return ok ? SALS_OK : SALS_ERR_HIP;
}
}  // namespace

extern "C" {

size_t sals_calib_accumulate_workspace_bytes(int32_t dtype, int32_t D)
{
    if ((dtype != SALS_BF16 && dtype != SALS_F32) || D < 128 || D % 128 != 0 || D > kCalMaxD) return 0;
    if (dtype == SALS_BF16) return align_up((size_t)cov_tiles(D) * cov_max_slices(D) * kCovTile * kCovTile * 4);  // tile sums
    // the transposed keys of a chunk, then the fp32 tile sums of its slices
    return align_up((size_t)D * kCalChunk * 4) + align_up((size_t)cal_slices(D) * D * D * 4);
}

sals_status sals_calib_accumulate(int32_t dtype, const void* K, int64_t n_tok, int32_t D, double* C, void* workspace,
                                  size_t workspace_bytes, void* hip_stream)
{
    if ((dtype != SALS_BF16 && dtype != SALS_F32) || bad(K) || bad(C) || n_tok < 1 || D < 128 || D % 128 != 0 || D > kCalMaxD)
        return SALS_ERR_INVALID_ARG;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0 ||
        workspace_bytes < sals_calib_accumulate_workspace_bytes(dtype, D))
        return SALS_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (calib_lds_attr(dtype) != SALS_OK) return SALS_ERR_HIP;
    if (dtype == SALS_BF16) return calib_accumulate_bf16(K, n_tok, D, C, workspace, st);
    return calib_accumulate_f32(K, n_tok, D, C, workspace, st);
}

namespace {
// Column slices of the launches of a Jacobi step: of the Gram matrices (at most 8: the partial matrices are added up by every
// workgroup of the rotation) and of the rotation, as many as keep either within about two, or one, workgroups per compute unit
// (multiples of 16 columns, at least 64 of them).
int jac_gram_slices(int D)
{
    int s = 1;
    while (s < 8 && D % (32 * s) == 0 && D / (2 * s) >= 64 && D / (2 * kJacBig) * 2 * (2 * s) <= 512) s *= 2;
    return s;
}
int jac_slices(int D)
{
    int s = 1;
    while (D % (32 * s) == 0 && D / (2 * s) >= 64 && D / (2 * kJacBig) * (2 * s) <= 256) s *= 2;
    return s;
}
constexpr int kAllMaxD = 3584;   // of transformations of all rows at once (see all_first)
struct PinnedAlloc {
    static void* pin(size_t bytes)
    {
        void* p = nullptr;
        if (hipHostMalloc(&p, bytes, hipHostMallocPortable) == hipSuccess) return p;
        (void)hipGetLastError();
        return nullptr;
    }
    static void unpin(void* p) { (void)hipHostFree(p); }
};
// doubles that a call reads back: convergence slots, norms, what is found of angles (their sums, counts and squares, or two values a tile)
constexpr size_t eig_host_doubles(int D)
{
    const size_t n = D, tiles = n * n / 4096, angles = n * n / 2048;
    return n / kJacBig + n + (D <= kAllMaxD ? tiles + 2 * angles : 2 * tiles);
}
typedef HostBlock<PinnedAlloc, std::max(eig_host_doubles(kCalMaxD), eig_host_doubles(kAllMaxD)) * 8, 4> EigHost;
struct Event {
    hipEvent_t e = nullptr;
    ~Event() { if (e) (void)hipEventDestroy(e); }
};
struct EigWs {  // byte offsets into the workspace
    size_t G, conv, norm, sgn, diag, part, Y0, Y1, total;
};
// `n_part` slices of the Gram matrices; `series`: with the two partial sums that making the last rotations all at once takes.
EigWs eig_ws(int D, int n_part, bool series)
{
    EigWs w{};
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o = align_up(o + bytes); return at; };
    w.G = take((size_t)D * D * 8);               // the rotated factor
    w.conv = take((size_t)(D / kJacBig) * 8);    // convergence slots; before the sweeps, whether a pivot was not positive
    w.norm = take((size_t)D * 8);                // row norms and signs
    w.sgn = take((size_t)D * 8);
    w.diag = take((size_t)D * kCalPanel * 8);    // factored diagonal blocks
    // partial Gram matrices of a step: of the blocks, or of pairs of them
    w.part = take((size_t)n_part * (D / kJacBig) * std::max(kJacRec, kJacBigRec / 2) * 8);
    w.Y0 = take(series ? (size_t)D * D * 8 : 0);
    w.Y1 = take(series ? (size_t)D * D * 8 : 0);
    w.total = o;
    return w;
}
// What a workspace of `bytes` allows: with less than the full size sweeps alone, and as many slices as fit (a slice of the Gram
// matrices is 320 D bytes: with one of them all of it is less than 8 D^2 + 900 D).
bool eig_plan(int D, size_t bytes, EigWs* w, int* n_part, bool* series)
{
    *n_part = jac_gram_slices(D);
    *series = true;
    *w = eig_ws(D, *n_part, true);
    if (bytes >= w->total) return true;
    *series = false;
    for (;; *n_part /= 2) {
        *w = eig_ws(D, *n_part, false);
        if (bytes >= w->total) return true;
        if (*n_part == 1) return false;
    }
}
}  // namespace

namespace {
// Transformations of all rows at once (k_calib_all.hpp) in place of sweeps, up to kAllMaxD.  One takes 0.38 ms at D = 1024, where a
// sweep takes 0.85, and from the Cholesky factor on it brings the rows as far as a sweep does, or further once the angles are below
// one; its products grow with D^3 and a sweep's steps with D^2, so for large D it comes later.  A call, r = 5/8 D, in ms with the
// transformations behind one, two, three and four sweeps (and with sweeps alone): D = 256 1.8 / 1.9 / 2.0 / 2.0 (2.1), 512 2.8 / 2.8 /
// 3.0 / 3.2 (4.1), 1024 4.9 / 5.3 / 5.7 / 6.3 (9.4), 1536 12.9 / 13.3 / 13.8 / 14.3 (19.1), 2048 21.2 / 21.5 / 21.8 / 22.5 (28.7), 2560 45.6 /
// 43.8 / 43.0 / 44.1 (58.9), 3072 67.9 / 68.0 / 66.9 / 63.9 (80.3), 3584 111 / 104 / 102 / 98.6 (109), 4096 159 / 149 / 142 / 140 (141).
inline int all_first(int D) { return D <= 2048 ? 1 : D < 3072 ? 3 : 4; }
// Up to kFloatMaxD the long way, in place of the first sweep and of the transformations that follow it, is gone in floats (k_calib_all.hpp):
// transformations until one has started from |E| <= kFloatLast, V made orthogonal once, in fp32, behind the first one that starts from
// kFloatPolish or less.  A call, r = 5/8 D, in ms without and with it, D = 256 1.44 / 1.06, 512 2.34 / 1.49, 1024 4.30 / 2.63, 1536 12.2 / 6.75,
// 2048 20.5 / 12.2, 2560 42.3 / 23.4 (beyond, with all polar factors in pairs, 3072 66.3 / 65.9, 3584 99.2 / 100.8); D = 1024 with
// spectra c^-2 5.03 / 2.89, 10^(-6 c / D) 4.51 / 2.78, sixteenfold eigenvalues 8.18 / 6.70.  kFloatLast 0.3 and 0.03: 2.70 and 2.65 at D = 1024 where
// 0.1 takes 2.65, and 1.55 and 1.63 with a linear spectrum at D = 512, where it takes 1.55; kFloatPolish 1.5 and 6: 2.65 and 2.68, 1.62 and 1.55.
constexpr double kFloatLast = 0.1, kFloatPolish = 3.5;
// the series of the exponential: cut behind E^4 it differs from an orthogonal matrix by |E|^6 / 72
constexpr double kSeriesNorm = 4e-3;
// the product kernels' dynamic LDS, beyond the default limit
sals_status calib_all_lds(bool series)
{
    auto allow = [](const void* kern, size_t bytes) {
        return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
    };
    constexpr size_t nn = prod_lds<float, float, true>();
    if (!allow(reinterpret_cast<const void*>(calib_angles_kernel), kSymLds)) return SALS_ERR_HIP;
    if (!series) return SALS_OK;
    const bool ok = allow(reinterpret_cast<const void*>(calib_gram_kernel<double>), kSymLds) &&
                    allow(reinterpret_cast<const void*>(calib_gram_kernel<float>), kSymLds) &&
                    allow(reinterpret_cast<const void*>(calib_series_kernel<false>), kSymLds) &&
                    allow(reinterpret_cast<const void*>(calib_series_kernel<true>), kSymLds) &&
                    allow(reinterpret_cast<const void*>(calib_series_rest_kernel), prod_lds<float, float, false>()) &&
                    allow(reinterpret_cast<const void*>(calib_float_apply_kernel), nn) &&
                    allow(reinterpret_cast<const void*>(calib_polar_kernel<0, true, false>), kPairLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_kernel<0, false, false>), kPairLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_kernel<1, false, false>), kPairLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_kernel<1, false, true>), kPairLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_kernel<2, false, false>), kPairLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_kernel<2, false, true>), kPairLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_plain_kernel<0, true, kOutPlain, false>), kPlainLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_plain_kernel<0, false, kOutPlain, false>), kPlainLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_plain_kernel<1, false, kOutPlain, false>), kPlainLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_plain_kernel<1, false, kOutFloat, false>), kPlainLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_plain_kernel<2, false, kOutPlain, false>), kPlainLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_plain_kernel<2, false, kOutPlain, true>), kPlainLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_plain_kernel<2, false, kOutFloat, false>), kPlainLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_square_kernel), kSymLds) &&
                    allow(reinterpret_cast<const void*>(calib_polar_last_kernel), nn) &&
                    allow(reinterpret_cast<const void*>(calib_defect_kernel), kSymLds) &&
                    allow(reinterpret_cast<const void*>(calib_correction_kernel), kPairLds) &&
                    allow(reinterpret_cast<const void*>(calib_apply_kernel<float, false>), prod_lds<float, double, true>()) &&
                    allow(reinterpret_cast<const void*>(calib_apply_kernel<double, true>), prod_lds<double, double, true>());
    return ok ? SALS_OK : SALS_ERR_HIP;
}
}  // namespace

size_t sals_calib_eigenvectors_workspace_bytes(int32_t D)
{
    if (D < kCalThreads || D % kCalThreads != 0 || D > kCalMaxD) return 0;
    return eig_ws(D, jac_gram_slices(D), true).total;
}

sals_status sals_calib_eigenvectors(double* C, int32_t D, int32_t r, int32_t dtype, double* eigval, void* U, void* workspace,
                                    size_t workspace_bytes, int32_t max_sweeps, int32_t* sweeps, void* hip_stream)
{
    if ((dtype != SALS_BF16 && dtype != SALS_F32) || bad(C) || !eigval || bad(U) || D < kCalThreads || D % kCalThreads != 0 ||
        D > kCalMaxD || r < 1 || r > D || max_sweeps < 1)
        return SALS_ERR_INVALID_ARG;
    EigWs off;
    int n_part;
    bool series;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0 || !eig_plan(D, workspace_bytes, &off, &n_part, &series))
        return SALS_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    auto at = [&](size_t o) { return reinterpret_cast<double*>(ws + o); };
    double *G = at(off.G), *conv = at(off.conv), *norm = at(off.norm), *sgn = at(off.sgn), *diag = at(off.diag), *part = at(off.part);
    int* fail = reinterpret_cast<int*>(ws + off.conv);
    const int n_blocks = D / kJacBig, n_pairs = n_blocks / 2, n_steps = n_blocks - 1;
    const int slices = jac_slices(D);
    const int n_tiles = (D / 64) * (D / 64);   // of the angles, whose results lie where the partial Gram matrices do
    f64x2* const found = reinterpret_cast<f64x2*>(part);
    const int n_angles = D / kAngleRows * (D / 256);
    double *const square = part, *const all_found = square + n_tiles;   // (read with one copy, squares first)
    float* const row_off = reinterpret_cast<float*>(all_found + 2 * n_angles);
    double *rows = G, *other = at(off.Y0), *third = at(off.Y1);   // the rows, and room for two more matrices (`series`)
    double* const sorted = diag;                                  // (the factored blocks are in place by then)
    const bool all = series && D <= kAllMaxD;
    double *const scale = sgn, *const lead = diag + D;   // (behind the sorted norms; the signs are wanted at the very end only)
    auto row_norms = [&](const double* M) { hipLaunchKernelGGL(calib_rownorm_kernel, dim3(D), dim3(kCalThreads), 0, st, M, D, norm, sgn); };
    auto find_lead = [&](const double* M) {   // the squared norm of rows that count
        row_norms(M);
        hipLaunchKernelGGL(calib_lead_kernel, dim3(D), dim3(kCalThreads), 0, st, norm, D, r, lead);
    };
    auto factor = [&](double f) -> bool {
        if (hipMemcpyAsync(G, C, (size_t)D * D * 8, hipMemcpyDeviceToDevice, st) != hipSuccess ||
            hipMemsetAsync(fail, 0, sizeof(int), st) != hipSuccess)
            return false;
        for (int k0 = 0; k0 < D; k0 += kCalPanel) {
            const int rest = D - k0 - kCalPanel;
            hipLaunchKernelGGL(calib_chol_panel_kernel, dim3(std::max(1, rest / 64)), dim3(256), 0, st, G, D, k0, scale, f, diag, fail);
            if (rest > 0) hipLaunchKernelGGL(calib_chol_update_kernel, dim3(rest / 64, rest / 64), dim3(512), 0, st, G, D, k0);
        }
        hipLaunchKernelGGL(calib_chol_finish_kernel, dim3(D), dim3(256), 0, st, G, D, diag);
        return launch_status() == SALS_OK;
    };
    EigHost host;   // (behind the first launch a lack of memory would leave kernels at work in the caller's)
    if (!host.p) return SALS_ERR_HIP;
    // G = Cholesky factor of C + shift I, the shift from C's scale, which the host learns with what came of it.
    row_norms(C);
    hipLaunchKernelGGL(calib_scale_kernel, dim3(1), dim3(kCalThreads), 0, st, norm, D, scale);
    if (!factor(1.0) || calib_all_lds(series) != SALS_OK) return SALS_ERR_HIP;
    double *const h_conv = static_cast<double*>(host.p), *const h_norm = h_conv + n_blocks, *const h_found = h_norm + D;
    auto read = [&](void* to, const void* from, size_t bytes) { return hipMemcpyAsync(to, from, bytes, hipMemcpyDeviceToHost, st) == hipSuccess; };
    auto wait = [&]() { return launch_status() == SALS_OK && hipStreamSynchronize(st) == hipSuccess; };
    if (!read(h_norm, scale, 8) || !read(h_conv, fail, sizeof(int)) || !wait()) return SALS_ERR_HIP;
    const double n0 = h_norm[0];  // (between the largest diagonal entry and lambda_0)
    int done = 0;
    bool converged = !(n0 > 0.0) || !std::isfinite(n0);  // the zero matrix needs no rotation
    bool rotated = false;
    double shift = 0.0;
    // No eigenvalue lies below -sqrt(D) n0 (sqrt(D) is at most 90.5), so ten shifts, up to 180 n0, end with a positive definite matrix
    // unless C is not one of numbers (then its rows are returned as they are).
    if (!converged) {
        int failed = *reinterpret_cast<int*>(h_conv);
        double f = 1.0;
        for (int t = 1; t < 10 && failed; ++t) {
            f *= 64.0;
            if (!factor(f) || !read(h_conv, fail, sizeof(int)) || !wait()) return SALS_ERR_HIP;
            failed = *reinterpret_cast<int*>(h_conv);
        }
        shift = kCalShift * n0 * f;
        converged = failed != 0;
    }
    if (hipMemsetAsync(lead, 0, 8, st) != hipSuccess) return SALS_ERR_HIP;   // first sweep: every rotation counts
    auto block_step = [&](int step) {  // rotates the pairs of blocks of a step of a sweep, or neighbours
        hipLaunchKernelGGL((calib_jacobi_gram_kernel<double>), dim3(n_pairs, n_part, 2), dim3(256), 0, st, rows, D, D, step, D / n_part, part);
        hipLaunchKernelGGL((calib_jacobi_rotate_kernel<double>), dim3(n_pairs, slices), dim3(kJacThreads), 0, st, rows, D, D, step, D / slices,
                           part, n_part, lead, conv);
    };
    auto inside_step = [&]() {
        hipLaunchKernelGGL(calib_jacobi_inside_gram_kernel, dim3(n_blocks, n_part), dim3(256), 0, st, rows, D, D / n_part, part);
        hipLaunchKernelGGL(calib_jacobi_inside_kernel, dim3(n_blocks, slices), dim3(kJacInsideThreads), 0, st, rows, D, D / slices, part,
                           n_part, lead, conv);
    };
    const dim3 tile_grid(D / 64, D / 64), sym_grid(n_tiles), prod(kProdThreads);
    // Orthogonal polar factor of I + E in floats, X or X2, from E and A = E E^T (as pairs of bf16), with room for Y (which may be E or A).
    // `exact`: the last step in fp32 (otherwise in pairs, as all others).
    // The defect of (X X^T) X is quadratic in that of X; X (X X^T) is the same only as long as X commutes with its transpose, and what
    // rounding takes from that would stay.
    auto polar_factor = [&](const PolarPlan& P, const uint32_t* E, const uint32_t* A, uint32_t* Y, uint32_t* X, uint32_t* X2, bool exact) -> const float* {
        auto step = [&](auto n, bool fp32, const uint32_t* L, const uint32_t* R, double f, double d, double s, const uint32_t* S, double t,
                        const uint32_t* T, uint32_t* O) {
            constexpr int N = decltype(n)::value;
            if (fp32) hipLaunchKernelGGL((calib_polar_kernel<N, false, true>), tile_grid, prod, kPairLds, st, L, R, D, (float)f, (float)d,
                                         (float)s, S, (float)t, T, O, nullptr);
            else hipLaunchKernelGGL((calib_polar_kernel<N, false, false>), tile_grid, prod, kPairLds, st, L, R, D, (float)f, (float)d,
                                    (float)s, S, (float)t, T, O, nullptr);
        };
        const double w = 0.5 * P.a[0] * P.a[0] * P.a[0] / (P.top * P.top * P.top), c1 = 1.5 * P.a[0] / P.top - w;
        const bool more = P.one_more && !exact;   // (the unscaled step in pairs as well)
        const int n = P.n + (more ? 1 : 0);
        step(std::integral_constant<int, 2>{}, n == 1, A, E, w * P.tau * P.tau * P.tau, c1, c1 * P.tau, E, -w * P.tau * P.tau, A, X);
        for (int k = 1; k < n; ++k) {
            const double a = k < P.n ? P.a[k] : 1.0;
            step(std::integral_constant<int, 0>{}, false, X, X, 1.0, 0.0, 0.0, nullptr, 0.0, nullptr, Y);
            step(std::integral_constant<int, 1>{}, k == n - 1, Y, X, -0.5 * a * a * a, 0.0, 1.5 * a, X, 0.0, nullptr, X2);
            std::swap(X, X2);
        }
        if (P.one_more && exact) {
            float *const x = reinterpret_cast<float*>(X), *const x2 = reinterpret_cast<float*>(X2), *const y = reinterpret_cast<float*>(Y);
            hipLaunchKernelGGL(calib_polar_square_kernel, sym_grid, prod, kSymLds, st, x, D, D, y);
            hipLaunchKernelGGL(calib_polar_last_kernel, tile_grid, prod, (prod_lds<float, float, true>()), st, y, x, D, -0.5f, 1.5f, x2);
            std::swap(X, X2);
        }
        return reinterpret_cast<const float*>(X);
    };
    // to = X made orthogonal, times `from`, by way of `between` and C; `rounded` is room for a matrix of pairs
    auto correct_and_apply = [&](const float* X, uint32_t* rounded, const double* from, double* between, double* to) {
        hipLaunchKernelGGL(calib_defect_kernel, sym_grid, prod, kSymLds, st, X, D, C, rounded);
        hipLaunchKernelGGL(calib_correction_kernel, tile_grid, prod, kPairLds, st, rounded, D, C);
        hipLaunchKernelGGL((calib_apply_kernel<float, false>), tile_grid, prod, (prod_lds<float, double, true>()), st, X, from, nullptr, 1.0, between, D);
        hipLaunchKernelGGL((calib_apply_kernel<double, true>), tile_grid, prod, (prod_lds<double, double, true>()), st, C, between, between, 1.0, to, D);
    };
    // The long way in floats: an orthogonal matrix times the factor into `rows`, nearly orthogonal rows mostly (*near: the last angles were
    // small); *ok false: the factor is still there (and C, unless a transformation was begun, which takes rows that are not orthogonal).
    auto float_rows = [&](bool* ok, bool* near) -> sals_status {
        *ok = *near = false;
        float *cur = reinterpret_cast<float*>(at(off.Y0)), *nxt = reinterpret_cast<float*>(at(off.Y1));
        uint32_t *const c0 = reinterpret_cast<uint32_t*>(C), *const c1 = c0 + (size_t)D * D;
        float* const fpart = reinterpret_cast<float*>(part);
        int expo;
        std::frexp(std::sqrt(n0), &expo);   // (rows of the factor have norms of at most D^1/4 sqrt(n0))
        auto near_step = [&](int step, auto inside) {
            constexpr bool kInside = decltype(inside)::value;
            hipLaunchKernelGGL((calib_jacobi_gram_kernel<float>), dim3(n_pairs, n_part, 2), dim3(256), 0, st, cur, D, 2 * D, step, D / n_part, fpart);
            hipLaunchKernelGGL((calib_jacobi_rotate_kernel<float, kInside>), dim3(n_pairs, slices), dim3(kJacThreads), 0, st, cur, D, 2 * D, step,
                               2 * D / slices, fpart, n_part, lead, conv);
        };
        FloatDefect defect;
        auto polish = [&]() {   // V <- (3 I - V V^T) V / 2, and G with it
            float* const O = reinterpret_cast<float*>(c0);
            hipLaunchKernelGGL(calib_polar_square_kernel, sym_grid, prod, kSymLds, st, cur + D, D, 2 * D, O);
            hipLaunchKernelGGL(calib_float_apply_kernel, dim3(2 * D / 64, D / 64), prod, (prod_lds<float, float, true>()), st, O, cur, D, 2 * D, -0.5f, 1.5f,
                               nxt, 2 * D);
            std::swap(cur, nxt);
            defect.polish();
        };
        // The polar factor in floats, X or X2, with all steps in plain bf16 (E and A are such matrices, in the lower half of the room of one in
        // pairs).  Its first step and the square that the next one begins with can be launched before the plan is known; they are `ahead`, and made
        // again if the plan turns out to have one step only.
        auto low = [](uint32_t* M) { return reinterpret_cast<bf16_t*>(M); };
        auto high = [&](uint32_t* M) { return reinterpret_cast<bf16_t*>(M) + (size_t)D * D; };
        auto plain_square = [&](uint32_t* X, uint32_t* A) {
            hipLaunchKernelGGL((calib_polar_plain_kernel<0, false, kOutPlain, false>), tile_grid, prod, kPlainLds, st, low(X), low(X), D, 1.f, -1.f, 0.f,
                               nullptr, 0.f, high(A), nullptr, nullptr);
        };
        auto begin_plain = [&](uint32_t* E, uint32_t* A, uint32_t* X) {
            hipLaunchKernelGGL((calib_polar_plain_kernel<2, false, kOutPlain, true>), tile_grid, prod, kPlainLds, st, low(A), low(E), D, 0.f, 0.f, 0.f, low(E),
                               0.f, X, high(X), square);
            plain_square(X, A);
        };
        auto plain_factor = [&](const PolarPlan& P, bool ahead, uint32_t* E, uint32_t* A, uint32_t* X, uint32_t* X2) -> const float* {
            const int n = P.n + (P.one_more ? 1 : 0);
            const double w = 0.5 * P.a[0] * P.a[0] * P.a[0] / (P.top * P.top * P.top), c1 = 1.5 * P.a[0] / P.top - w;
            ahead = ahead && n > 1;
            auto first = [&](auto out) {
                hipLaunchKernelGGL((calib_polar_plain_kernel<2, false, (PolarOut)decltype(out)::value, false>), tile_grid, prod, kPlainLds, st, low(A), low(E),
                                   D, (float)(w * P.tau * P.tau * P.tau), (float)c1, (float)(c1 * P.tau), low(E), (float)(-w * P.tau * P.tau), X,
                                   high(X), nullptr);
            };
            if (n == 1) first(std::integral_constant<int, kOutFloat>{});
            else if (!ahead) first(std::integral_constant<int, kOutPlain>{});
            for (int k = 1; k < n; ++k) {
                const double a = k < P.n ? P.a[k] : 1.0;
                const float f = (float)(-0.5 * a * a * a), s = (float)(1.5 * a - 0.5 * a * a * a);   // of (X X^T - I) X and X
                auto step = [&](auto out) {
                    hipLaunchKernelGGL((calib_polar_plain_kernel<1, false, (PolarOut)decltype(out)::value, false>), tile_grid, prod, kPlainLds, st, high(A),
                                       high(X), D, f, 0.f, s, high(X), 0.f, X2, high(X2), nullptr);
                };
                if (k > 1 || !ahead) plain_square(X, A);
                if (k == n - 1) step(std::integral_constant<int, kOutFloat>{});
                else step(std::integral_constant<int, kOutPlain>{});
                std::swap(X, X2);
            }
            return reinterpret_cast<const float*>(X);
        };
        hipLaunchKernelGGL(calib_float_rows_kernel, dim3(D), dim3(kCalThreads), 0, st, rows, D, std::ldexp(1.0, -expo), cur);
        Event copied;
        if (hipEventCreateWithFlags(&copied.e, hipEventDisableTiming) != hipSuccess) return SALS_ERR_HIP;
        FloatWay way;
        int steps = 0;   // of the last polar factor
        bool first = true, polished = false, enough = false;
        int n_lead = r;
        do {
            near_step(kJacNearEven, std::true_type{});
            near_step(kJacNearOdd, std::false_type{});
            hipLaunchKernelGGL(calib_float_norm_kernel, dim3(D / 4), dim3(256), 0, st, cur, D, norm);
            hipLaunchKernelGGL(calib_sort_kernel, dim3(D), dim3(kCalThreads), 0, st, reinterpret_cast<const double*>(cur), norm, D,
                               reinterpret_cast<double*>(nxt), sorted);
            std::swap(cur, nxt);
            uint32_t *const A = reinterpret_cast<uint32_t*>(nxt), *const E = A + (size_t)D * D;
            hipLaunchKernelGGL((calib_gram_kernel<float>), sym_grid, prod, kSymLds, st, cur, D, 2 * D, sorted, n_lead, reinterpret_cast<float*>(A), row_off);
            const bool plain = !polished;   // (large angles)
            if (plain) {
                auto angles = first ? calib_all_angles_kernel<bf16_t, true> : calib_all_angles_kernel<bf16_t, false>;
                hipLaunchKernelGGL(angles, dim3(D / kAngleRows, D / 256), dim3(256), 0, st, reinterpret_cast<const float*>(A), D, sorted, n_lead, row_off,
                                   kFloatOpen, kFloatDamp, reinterpret_cast<bf16_t*>(E), all_found);
                hipLaunchKernelGGL((calib_polar_plain_kernel<0, true, kOutPlain, false>), tile_grid, prod, kPlainLds, st, reinterpret_cast<const bf16_t*>(E),
                                   reinterpret_cast<const bf16_t*>(E), D, 1.f, 0.f, 0.f, nullptr, 0.f, A, nullptr, square);
            } else {
                hipLaunchKernelGGL((calib_all_angles_kernel<uint32_t>), dim3(D / kAngleRows, D / 256), dim3(256), 0, st, reinterpret_cast<const float*>(A), D,
                                   sorted, n_lead, row_off, kFloatOpen, kFloatDamp, E, all_found);
                hipLaunchKernelGGL((calib_polar_kernel<0, true, false>), tile_grid, prod, kPairLds, st, E, E, D, 1.f, 0.f, 0.f, nullptr, 0.f, nullptr, A,
                                   square);
            }
            if (!read(h_found, square, (size_t)(n_tiles + (first ? 2 : 1) * n_angles) * 8) || (first && !read(h_norm, sorted, (size_t)D * 8)))
                return SALS_ERR_HIP;
            const bool ahead = plain && steps > 1;   // (not the first time, which may leave C as it is)
            if (ahead) {
                if (hipEventRecord(copied.e, st) != hipSuccess) return SALS_ERR_HIP;
                begin_plain(E, A, c0);
                if (launch_status() != SALS_OK || hipEventSynchronize(copied.e) != hipSuccess) return SALS_ERR_HIP;
            } else if (!wait()) {
                return SALS_ERR_HIP;
            }
            double e2 = 0.0, a2 = 0.0;
            for (int i = 0; i < n_tiles; ++i) a2 += h_found[i];
            for (int i = 0; i < n_angles; ++i) e2 += h_found[n_tiles + i];
            const double now = std::sqrt(e2);
            const PolarPlan P = polar_plan(a2, now <= kFloatLast && polished ? kPolarNear : kFloatPolar);
            if (!std::isfinite(now) || P.n == 0) return SALS_OK;
            if (first) {
                double open = 0.0;
                for (int i = 0; i < n_angles; ++i) open += h_found[n_tiles + n_angles + i];
                if (!float_begins(now, open, h_norm, D)) return SALS_OK;
                n_lead = float_lead(h_norm, r);
            }
            steps = P.n + (P.one_more ? 1 : 0);
            const float* const X = plain ? plain_factor(P, ahead, E, A, c0, c1) : polar_factor(P, E, A, A, c0, c1, false);
            hipLaunchKernelGGL(calib_float_apply_kernel, dim3(2 * D / 64, D / 64), prod, (prod_lds<float, float, true>()), st, X, cur, D, 2 * D, 1.f, 0.f, nxt,
                               2 * D);
            std::swap(cur, nxt);
            defect.factor(P, plain);
            const bool stuck = way.stuck(now, polished);
            first = false;
            *near = now <= kFloatLast;
            enough = stuck || (*near && polished);
            if ((now <= kFloatPolish || stuck) && !polished) { polish(); polished = true; }
        } while (!enough);
        for (int k = 0; k < 8 && !defect.correctable(); ++k) polish();   // (mostly none)
        float* const O = reinterpret_cast<float*>(c0);
        hipLaunchKernelGGL(calib_polar_square_kernel, sym_grid, prod, kSymLds, st, cur + D, D, 2 * D, O);
        hipLaunchKernelGGL(calib_float_apply_kernel, tile_grid, prod, (prod_lds<float, float, true>()), st, O, cur + D, D, 2 * D, -0.5f, 1.5f, nxt, D);
        // V, made orthogonal in fp64, times the factor
        correct_and_apply(nxt, reinterpret_cast<uint32_t*>(nxt) + (size_t)D * D, rows, reinterpret_cast<double*>(cur), rows);
        if (launch_status() != SALS_OK) return SALS_ERR_HIP;
        *ok = true;
        return SALS_OK;
    };
    bool settled = false, fresh = false, near = false;
    // (A limit of one is that of one sweep in fp64: behind the floats, which would be all that it allows, some angles are always left.)
    if (all && D <= kFloatMaxD && max_sweeps > 1 && !converged) {
        const sals_status s = float_rows(&fresh, &near);
        if (s != SALS_OK) return s;
        near = near && fresh;
    }
    if (fresh) {   // (it takes the place of a sweep, and counts as one)
        rotated = true;
        done = 1;
        // The pairs inside and next to blocks, which floats leave too far from orthogonal for the series half of the time.  (Once more in floats,
        // the angles, and if they were too large a transformation: 4 % more at D = 256 and 1024, 2 at 512 and 768.)
        inside_step();
        block_step(kJacNearEven);
        block_step(kJacNearOdd);
        find_lead(rows);
    }
    bool moved = false;    // `lead` is from before a transformation
    double last = 1e300;   // |E| of the transformation before, infinite behind a sweep
    // (The limit is one of sweeps, so that one which is enough without transformations is enough with them.  Between two sweeps |E|
    // falls by a tenth at least with each, from at most D to kSeriesNorm.)
    while (done < max_sweeps && !converged) {
        double worst = 0.0;   // largest rotation that is known to have been left behind
        if (fresh) {   // behind the floats: their rest is mostly for the series
            worst = 0.1;
            fresh = false;
        } else if (all && !settled && (near || done >= all_first(D)) && last > 0.0) {
            // One transformation of all rows; at any D where floats left small angles, but too large ones for the series (D = 2304, keys, r =
            // 5/8 D 23.2 ms with a sweep there, 21.2 so; from |E| = 100 on, 1 / c^2 at D = 2560 55.1 with transformations, 50.2 with sweeps)
            moved = true;
            inside_step();
            block_step(kJacNearEven);
            block_step(kJacNearOdd);
            hipLaunchKernelGGL(calib_rownorm_kernel, dim3(D), dim3(kCalThreads), 0, st, rows, D, norm, sgn);
            hipLaunchKernelGGL(calib_sort_kernel, dim3(D), dim3(kCalThreads), 0, st, rows, norm, D, other, sorted);
            std::swap(rows, other);
            uint32_t *const E = reinterpret_cast<uint32_t*>(third), *const A = E + (size_t)D * D;
            hipLaunchKernelGGL((calib_gram_kernel<double>), sym_grid, prod, kSymLds, st, rows, D, D, sorted, r,
                               reinterpret_cast<float*>(A), row_off);
            hipLaunchKernelGGL((calib_all_angles_kernel<uint32_t>), dim3(D / kAngleRows, D / 256), dim3(256), 0, st, reinterpret_cast<const float*>(A), D,
                               sorted, r, row_off, kAllOpen, kAllDamp, E, all_found);
            hipLaunchKernelGGL((calib_polar_kernel<0, true, false>), tile_grid, prod, kPairLds, st, E, E, D, 1.f, 0.f, 0.f, nullptr, 0.f, nullptr,
                               A, square);
            if (!read(h_found, square, (size_t)(n_tiles + n_angles) * 8) || !wait()) return SALS_ERR_HIP;
            double e2 = 0.0, a2 = 0.0;
            for (int i = 0; i < n_tiles; ++i) a2 += h_found[i];
            for (int i = 0; i < n_angles; ++i) e2 += h_found[n_tiles + i];
            // (a matrix on which the transformations gain little, as with eigenvalues that repeat or rows of very different norms
            // in no order, gets a sweep in between)
            const double now = std::sqrt(e2);
            const PolarPlan P = polar_plan(a2);
            if (now <= kSeriesNorm) {
                worst = now;
                last = 0.0;   // (what the series leaves is for sweeps)
                settled = true;
                find_lead(rows);
                moved = false;
            } else if (!std::isfinite(now) || P.n == 0) {
                last = 0.0;   // (sums that are no numbers: a sweep)
                continue;
            } else {
                last = now < 0.9 * last ? now : 0.0;
                const float* const X = polar_factor(P, E, A, E, reinterpret_cast<uint32_t*>(other), reinterpret_cast<uint32_t*>(other) + (size_t)D * D, true);
                correct_and_apply(X, reinterpret_cast<uint32_t*>(other) + (X == reinterpret_cast<float*>(other) ? (size_t)D * D : 0), rows, third, other);
                std::swap(rows, other);
                if (launch_status() != SALS_OK) return SALS_ERR_HIP;
                continue;
            }
        } else {
            if (moved) {   // (the r-th norm may have fallen far: rows below the old one would not be asked to have converged)
                find_lead(rows);
                moved = false;
            }
            if (hipMemsetAsync(conv, 0, (size_t)n_blocks * 8, st) != hipSuccess) return SALS_ERR_HIP;
            inside_step();
            for (int step = 0; step < n_steps; ++step) block_step(step);
            if (!read(h_conv, conv, (size_t)n_blocks * 8)) return SALS_ERR_HIP;
            find_lead(rows);
            if (!wait()) return SALS_ERR_HIP;
            for (int i = 0; i < n_blocks; ++i) worst = std::max(worst, h_conv[i]);
            rotated = rotated || worst > 0.0;  // (in the first sweep every rotation is recorded)
            ++done;
            last = 1e300;
            // a rotation by less than 1e-11 no longer moves an eigenvector; only pairs with a row among the r largest are asked to
            // have converged
            converged = worst <= 1e-11;
        }
        // Behind a sweep of small rotations the angles that are left decide: converged, or all of them at once, or a further sweep.
        // (Sweeps whose largest rotation was 0.26, 0.07, 0.007 left 4e-5, 1e-3, 4e-6.)  The angles lie in C, which is free until its
        // rows are written.
        for (int pass = 0; !converged && worst <= 0.3 && pass < 6; ++pass) {
            hipLaunchKernelGGL(calib_angles_kernel, sym_grid, prod, kSymLds, st, rows, D, norm, lead, C, found);
            if (!read(h_found, found, (size_t)n_tiles * sizeof(f64x2)) || !wait()) return SALS_ERR_HIP;
            double most = 0.0, square_sum = 0.0;
            for (int i = 0; i < n_tiles; ++i) { most = std::max(most, h_found[2 * i]); square_sum += h_found[2 * i + 1]; }
            converged = most <= 1e-11;
            if (converged || !series || !(square_sum <= kSeriesNorm * kSeriesNorm)) break;
            // exp(E) G = G + (exp(E) - I) G, with as many terms as are above rounding.
            const double* X = C;
            if (square_sum > 1e-18) {
                float* const P = reinterpret_cast<float*>(third), *const L = P + (size_t)D * D;
                X = other;
                if (square_sum <= 4e-8) {
                    hipLaunchKernelGGL((calib_series_kernel<false>), sym_grid, prod, kSymLds, st, C, D, other, P, L);
                } else {
                    hipLaunchKernelGGL((calib_series_kernel<true>), sym_grid, prod, kSymLds, st, C, D, other, P, L);
                    hipLaunchKernelGGL(calib_series_rest_kernel, tile_grid, prod, (prod_lds<float, float, false>()), st, L, P, D, other);
                }
            }
            hipLaunchKernelGGL((calib_apply_kernel<double, true>), tile_grid, prod, (prod_lds<double, double, true>()), st, X, rows, rows, 1.0, third, D);
            std::swap(rows, third);
            find_lead(rows);
        }
    }
    // A matrix whose factor needed no rotation is diagonal (R R^T is diagonal for an upper triangular R only if R is): its
    // own rows are the answer, without the detour through the square roots.
    if (!rotated) row_norms(C);
#define SALS_SELECT(T, ROOT, M)                                                                                              \
    hipLaunchKernelGGL((calib_select_kernel<T, ROOT>), dim3(D), dim3(kCalThreads), 0, st, M, norm, sgn, D, r, shift, eigval, \
                       static_cast<T*>(U), C)
    if (dtype == SALS_BF16) { if (rotated) SALS_SELECT(bf16_t, true, rows); else SALS_SELECT(bf16_t, false, C); }
    else { if (rotated) SALS_SELECT(float, true, rows); else SALS_SELECT(float, false, C); }
#undef SALS_SELECT
    if (sweeps) *sweeps = converged ? done : -done;
    host.idle = true;
    return launch_status();
}

}  // extern "C"
