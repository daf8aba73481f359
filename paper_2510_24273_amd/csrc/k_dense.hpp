// Dense decode attention over a full-rank KV cache: the baseline the paper's speed-ups are
// quoted against (Sec. 5.3, Table 6), here as an in-library comparison on the same hardware.
//
//   out[b,h] = softmax_j( RoPE(q[b,h], q_pos[b]) . K[b,j,g(h)] / sqrt(d) ) V[b,j,g(h)],  j < seq_len[b]
//
// K [B, S_max, H_kv, d] holds the keys as a dense model caches them (already rotated at their
// positions), V [B, S_max, H_kv, d] the values.  A pure HBM stream of 2*S*D_kv elements per
// sequence.  A workgroup covers a token chunk of one sequence and HB neighbouring KV heads: 16 lanes (one DPP row) own a
// (token, head) row of K and of V in 16-byte pieces, so with two heads a load of a wave is 512 bytes of a token's row in one
// piece; the dot product is folded with DPP rotations, softmax runs online per 16-lane group over UT tokens at a time (one in
// fp32, where rows are twice as long), whose rows are requested together and one set ahead.  The lane groups of a head and
// then the chunks are merged by log-sum-exp in a fixed order.  One workgroup per compute unit streams best (batch 16, 4096
// tokens, 32 heads: 7.1 TB/s with the merge; one head per workgroup, a token at a time, 256-token chunks: 5.9).  Batch 8, 2048
// tokens: 50.7 -> 43.3 us with the merge.
#pragma once
#include "common.hpp"
#include "k_attend.hpp"

namespace sals {

constexpr int kDnMaxChunks = 64;  // token chunks per sequence at most
constexpr int kDnRec = kHeadDim + 2;  // floats per partial record: running max, normaliser, 128 sums

// part [B, H, n_chunks, kDnRec]; grid (n_chunks, H_kv / HB, B)
template <typename T, int GMAX, int HB>
__global__ __launch_bounds__(256) void dense_attend_kernel(const T* __restrict__ q, const int32_t* __restrict__ q_pos,
                                                           const T* __restrict__ K, const T* __restrict__ V,
                                                           const int32_t* __restrict__ seq_len, int S_max, int H, int H_kv,
                                                           int n_chunks,
                                                           const float2* __restrict__ rope, InvFreq inv,
                                                           float* __restrict__ part, int rope_style, float scale)
{
    static_assert(HB == 1 || HB == 2, "heads of a workgroup share its waves' four lane groups");
    constexpr int VEC = elem<T>::vec;
    constexpr int NCH = kHeadDim / (16 * VEC);  // 16-byte pieces per lane and row: 1 (bf16) or 2 (fp32)
    constexpr int UT = NCH > 1 ? 1 : GMAX > 4 ? 2 : 4;
    constexpr int NS = 16 / HB;                 // token slots of a head
    __shared__ float sQ[HB][GMAX][kHeadDim];
    __shared__ float2 sCS[kPairs];
    __shared__ float sRed[16][kDnRec + 2];

    const int chunk = blockIdx.x, h0 = blockIdx.y * HB, b = blockIdx.z;
    const int tid = threadIdx.x, li = tid & 15, tg = tid >> 4;   // lane group tg = wave * 4 + DPP row
    const int hb = (tg & 3) % HB, slot = (tg >> 2) * (4 / HB) + (tg & 3) / HB;
    const int G = idiv(H, H_kv);
    const int S_v = ld_uniform_i32(seq_len + b), qp_v = ld_uniform_i32(q_pos + b);
    const size_t row_stride = (size_t)H_kv * kHeadDim;
    const T* kb = K + ((size_t)b * S_max * H_kv + h0 + hb) * kHeadDim + li * VEC;
    const T* vb = V + ((size_t)b * S_max * H_kv + h0 + hb) * kHeadDim + li * VEC;

    struct Rows { u32x4 k[UT][NCH], v[UT][NCH]; };
    // tokens j, j + NS, ... of this lane's slot, from clamped addresses (slots past the end re-read the last row)
    auto load_rows = [&](Rows& R, int j, int last) {
#pragma unroll
        for (int u = 0; u < UT; ++u) {
            const size_t off = (size_t)min(j + u * NS, last) * row_stride;
#pragma unroll
            for (int n = 0; n < NCH; ++n) {
                R.k[u][n] = ld16_stream(kb + off + 16 * n * VEC);
                R.v[u][n] = ld16_stream(vb + off + 16 * n * VEC);
            }
        }
    };
    // the chunks are shares of the tokens present, not of the capacity (the first loads wait for the length)
    const int S = min(wave_uniform(S_v), S_max);
    const int tok_per_chunk = ((max(S, 0) + n_chunks - 1) / n_chunks + 15) & ~15;
    const int j0 = chunk * tok_per_chunk, j1 = min(S, j0 + tok_per_chunk);
    Rows R0, R1;
    load_rows(R0, j0 + slot, max(S - 1, 0));

    // the rotated, pre-scaled query of these KV heads' query heads
    const int qp = wave_uniform(qp_v);
    if (tid < kPairs) {
        if (qp >= 0 && qp <= S_max) {
            sCS[tid] = rope[(size_t)qp * kPairs + tid];
        } else {
            double sn, c;
            sincos((double)qp * inv.f[tid], &sn, &c);
            sCS[tid] = make_float2((float)c, (float)sn);
        }
    }
    __syncthreads();
    for (int t = tid; t < HB * G * kPairs; t += 256) {
        const int p = t & (kPairs - 1), hm = t >> 6;  // (head of the block, head of its group)
        const int c1 = pair_first(p, rope_style), c2 = pair_second(p, rope_style);
        const T* qh = q + ((size_t)b * H + (size_t)h0 * G + hm) * kHeadDim;
        const float a = elem<T>::load(qh + c1), bb = elem<T>::load(qh + c2);
        const float2 cs = sCS[p];
        float* dst = sQ[hm / G][hm % G];
        dst[c1] = (a * cs.x - bb * cs.y) * scale;
        dst[c2] = (bb * cs.x + a * cs.y) * scale;
    }
    __syncthreads();
    float qf[GMAX][NCH][VEC];
#pragma unroll
    for (int m = 0; m < GMAX; ++m)
#pragma unroll
        for (int n = 0; n < NCH; ++n)
#pragma unroll
            for (int v = 0; v < VEC; ++v) qf[m][n][v] = m < G ? sQ[hb][m][(li + 16 * n) * VEC + v] : 0.f;

    float mx[GMAX], l[GMAX], acc[GMAX][NCH][VEC];
#pragma unroll
    for (int m = 0; m < GMAX; ++m) {
        mx[m] = -INFINITY; l[m] = 0.f;
#pragma unroll
        for (int n = 0; n < NCH; ++n)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[m][n][v] = 0.f;
    }
    auto consume = [&](Rows& R, int base) {
        const int j = base + slot;
        // The value words of slots past the chunk count as zero: the row they re-read is a live one, and its weight of zero
        // would make a NaN of an infinity.  (The last set of a chunk only; the scores are masked below.)
        if (base + UT * NS > j1) {  // uniform
#pragma unroll
            for (int u = 0; u < UT; ++u)
#pragma unroll
                for (int n = 0; n < NCH; ++n)
#pragma unroll
                    for (int e = 0; e < 4; ++e) R.v[u][n][e] = j + u * NS < j1 ? R.v[u][n][e] : 0u;
        }
#pragma unroll
        for (int m = 0; m < GMAX; ++m) {
            if (m < G) {  // uniform
                float x[UT];
#pragma unroll
                for (int u = 0; u < UT; ++u) {
                    x[u] = 0.f;
#pragma unroll
                    for (int n = 0; n < NCH; ++n) {
                        float kf[VEC];
                        elem<T>::unpack(R.k[u][n], kf);
#pragma unroll
                        for (int v = 0; v < VEC; ++v) x[u] = fmaf(qf[m][n][v], kf[v], x[u]);
                    }
                }
                float mn = mx[m];
#pragma unroll
                for (int u = 0; u < UT; ++u) {
                    x[u] = row16_sum(x[u]);
                    x[u] = j + u * NS < j1 ? x[u] : -INFINITY;
                    mn = fmaxf(mn, x[u]);
                }
                const float ref = mn > -INFINITY ? mn : 0.f;  // (no token yet)
                const float r = __expf(mx[m] - ref);
                mx[m] = mn;
                l[m] *= r;
#pragma unroll
                for (int n = 0; n < NCH; ++n)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[m][n][v] *= r;
#pragma unroll
                for (int u = 0; u < UT; ++u) {
                    const float p = __expf(x[u] - ref);
                    l[m] += p;
#pragma unroll
                    for (int n = 0; n < NCH; ++n) {
                        float vf[VEC];
                        elem<T>::unpack(R.v[u][n], vf);
#pragma unroll
                        for (int v = 0; v < VEC; ++v) acc[m][n][v] = fmaf(p, vf[v], acc[m][n][v]);
                    }
                }
            }
        }
    };
    // two register sets take turns (a copy between them would wait for the loads it moves); trip counts are the chunk's, the
    // same for every lane group
    for (int j = j0; j < j1; j += 2 * UT * NS) {
        if (j + UT * NS < j1) load_rows(R1, j + UT * NS + slot, S - 1);
        consume(R0, j);
        if (j + UT * NS < j1) {
            if (j + 2 * UT * NS < j1) load_rows(R0, j + 2 * UT * NS + slot, S - 1);
            consume(R1, j + UT * NS);
        }
    }

    // the lane groups of every head, merged in slot order
#pragma unroll
    for (int m = 0; m < GMAX; ++m) {
        if (m < G) {  // uniform
            __syncthreads();
            if (li == 0) { sRed[tg][0] = mx[m]; sRed[tg][1] = l[m]; }
#pragma unroll
            for (int n = 0; n < NCH; ++n)
#pragma unroll
                for (int v = 0; v < VEC; ++v) sRed[tg][2 + (li + 16 * n) * VEC + v] = acc[m][n][v];
            __syncthreads();
            for (int t = tid; t < HB * kHeadDim; t += 256) {
                const int h = t / kHeadDim, c = t % kHeadDim;
                auto group = [&](int s) { return (s / (4 / HB)) * 4 + (s % (4 / HB)) * HB + h; };
                float M = -INFINITY;
#pragma unroll
                for (int s = 0; s < NS; ++s) M = fmaxf(M, sRed[group(s)][0]);
                float L = 0.f, A = 0.f;
                if (M > -INFINITY) {
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const float w = __expf(sRed[group(s)][0] - M);
                        L = fmaf(sRed[group(s)][1], w, L);
                        A = fmaf(sRed[group(s)][2 + c], w, A);
                    }
                }
                float* rec = part + (((size_t)b * H + (size_t)(h0 + h) * G + m) * n_chunks + chunk) * kDnRec;
                if (c == 0) { rec[0] = M; rec[1] = L; }
                rec[2 + c] = A;
            }
        }
    }
}

// out[b,h] = merged chunks / normaliser, rounded once to T.  grid (B*H), 128 threads.  Sixteen chunk records are requested
// together and merged online (a loop with one load per round would cost a memory round trip per chunk).
template <typename T>
__global__ __launch_bounds__(128) void dense_merge_kernel(const float* __restrict__ part, T* __restrict__ out,
                                                          int n_chunks)
{
    const size_t bh = blockIdx.x;
    const int c = threadIdx.x;
    const float* rec = part + bh * n_chunks * kDnRec;
    float M = -INFINITY, L = 0.f, A = 0.f;
    for (int k0 = 0; k0 < n_chunks; k0 += 16) {
        float m[16], l[16], a[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const float* r = rec + (size_t)min(k0 + u, n_chunks - 1) * kDnRec;
            m[u] = r[0]; l[u] = r[1]; a[u] = r[2 + c];
        }
        float mn = M;
#pragma unroll
        for (int u = 0; u < 16; ++u) mn = fmaxf(mn, m[u]);  // (a clamped slot repeats the last record)
        if (mn > -INFINITY) {  // uniform
            const float w0 = __expf(M - mn);
            L *= w0;
            A *= w0;
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const bool live = k0 + u < n_chunks;  // (a repeated record adds nothing, an infinity in it neither)
                const float w = __expf(m[u] - mn);
                L = fmaf(live ? l[u] : 0.f, w, L);
                A = fmaf(live ? a[u] : 0.f, w, A);
            }
            M = mn;
        }
    }
    elem<T>::store(out + bh * kHeadDim + c, L > 0.f ? A / L : 0.f);
}

}  // namespace sals
