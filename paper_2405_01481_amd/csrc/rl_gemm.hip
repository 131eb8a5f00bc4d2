// MFMA GEMMs for gfx950:  C[M,N] = A[M,K] (fp16, row-major) * W[N,K]^T (bf16, row-major).
//
// Weights stay bf16 in HBM and are converted to fp16 on their way to the MFMA operand registers
// (exact for every weight of normal fp16 magnitude) -- or are read from an fp16 copy where a weight set
// has one; the contraction runs on fp16 MFMAs (v_mfma_f32_32x32x16_f16 in the first kernel,
// v_mfma_f32_16x16x32_f16 in the others) with fp32 accumulation.  Four kernels (the decode step's
// weight-streaming GEMMs are in rl_gemm_stream.hip):
//   * gemm_mfma_kernel: 128 x 128, 64 x 128 and 64 x 64 tiles staged through registers -- small M on bf16 weights, and split-K
//     for decode batches above 128 rows;
//   * gemm_ring_kernel: the same tiles staged by global -> LDS loads -- small M where a weight set has its fp16 copy;
//   * gemm_dma8_kernel: tiles of 96 to 256 rows x 256 columns, eight waves, operands staged by global ->
//     LDS loads -- the large-M GEMMs of prefill and scoring;
//   * gemm_kl8_kernel:  the same loop run twice on tiles of 128 rows -- the exact full-vocabulary KL, which needs the
//     policy's and the reference's logits of a tile together.
// Epilogues: fp32 store / split-K partial, residual add, SwiGLU, RoPE + q/k/v split for
// the QKV projection, log-sum-exp + target gather for the scoring LM head; mg_epilogue for the first kernel, d8_half for
// the second and third.  Both round alike: a row's results do not depend on which of them its GEMM's size picks.
#include <type_traits>

#include "rl_common.h"
#include "rl_gemm.h"
#include "rl_gemm_dev.h"

#define BK 64

// Which row of W feeds LDS row r of the B tile of column-block nb.
//  EPI_SWIGLU: the tile holds BN/2 gate rows and the matching BN/2 up rows, interleaved in
//              blocks of 32 so that a wave's adjacent 32-column MFMA tiles are (gate, up).
//  MG_QKV with head_dim 128: the halves of each head (128 tile columns) are interleaved in blocks of
//              32 so that a wave holds columns j and j + 64 in the same lane.
template <int EPI, int BN>
__device__ __forceinline__ int w_row_of(int r, int nb, const GemmArgs& a) {
    if (EPI == MG_SWIGLU) {
        int blk = r >> 5, within = r & 31;
        int col = nb * (BN / 2) + (blk >> 1) * 32 + within;
        return (blk & 1) ? a.up_offset + col : col;
    } else if (EPI == MG_QKV) {
        if (a.hd == 128) {
            int blk = (r & 127) >> 5, within = r & 31;   // per head, LDS blocks: [0:32) [64:96) [32:64) [96:128)
            int src = ((blk & 1) ? 64 : 0) + (blk >> 1) * 32 + within;
            return nb * BN + (r & ~127) + src;
        }
        return nb * BN + r;
    } else {
        return nb * BN + r;
    }
}

// Tile order.  The tile sequence walks bands of 8 row blocks column by column, so that consecutive
// tiles share few A row blocks and few W column blocks.  Workgroup ids are dealt round-robin to the 8
// XCDs, each with its own L2: XCD x takes the contiguous run [x*C, (x+1)*C) of the sequence, so the
// tiles resident on one XCD at any time form a compact block and re-use their operands from that L2.
// The grid holds 8*C ids; returns false for the (at most 7) ids past the end.
__device__ __forceinline__ bool tile_of(int id, int MB, int NB, int& mb, int& nb) {
    const int T = MB * NB, C = (T + 7) >> 3;
    const int pos = (id & 7) * C + (id >> 3);
    if (pos >= T) return false;
    const int per_group = 8 * NB;
    const int group = pos / per_group, first = group * 8, gsz = min(MB - first, 8), r = pos % per_group;
    mb = first + r % gsz;
    nb = r / gsz;
    return true;
}

// Row blocks of BM rows: a block's rows belong to one weight set.
__host__ __device__ __forceinline__ int row_blocks(const GemmArgs& a, int BM) {
    return a.Wb ? (a.M1 + BM - 1) / BM + (a.M - a.M1 + BM - 1) / BM : (a.M + BM - 1) / BM;
}
// First row of row block mb; with two weight sets a becomes the GEMM of the block's own (its weights, its end of rows).
__device__ __forceinline__ int enter_row_block(GemmArgs& a, int BM, int mb) {
    if (a.Wb) {
        const int mb1 = (a.M1 + BM - 1) / BM;
        if (mb >= mb1) {
            a.W = a.Wb;
            return a.M1 + (mb - mb1) * BM;
        }
        a.M = a.M1;
    }
    return mb * BM;
}

// Maximum / sum over the 32 lanes of a half-wave (the lanes that hold one row of a 32-column MFMA tile); every lane
// ends with the same bits.  Four steps inside each row of 16 lanes are data-parallel-primitive moves (swap lanes 1
// apart, 2 apart, mirror 8, mirror 16: each lane always meets a partner that holds the complementary set, and both
// form the same commutative combination), the step across the two rows is one cross-lane shuffle.
__device__ __forceinline__ float row32_max(float v) {
    v = fmaxf(v, dpp_move<0xB1>(v));    // quad_perm [1,0,3,2]
    v = fmaxf(v, dpp_move<0x4E>(v));    // quad_perm [2,3,0,1]
    v = fmaxf(v, dpp_move<0x141>(v));   // row_half_mirror
    v = fmaxf(v, dpp_move<0x140>(v));   // row_mirror
    return fmaxf(v, __shfl_xor(v, 16, RL_WAVE));
}
// The same two reductions for all register rows of a band at once, level by level: the chains are independent,
// so consecutive instructions never wait on one another (a data-parallel-primitive move needs two idle slots after
// the instruction that wrote its source).  Same operations per row, in the same order, as row32_max / row32_sum.
template <int CTRL, int N>
__device__ __forceinline__ void rows_max_step(float (&v)[N]) {
    float t[N];
#pragma unroll
    for (int r = 0; r < N; ++r) t[r] = dpp_move<CTRL>(v[r]);
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = fmaxf(v[r], t[r]);
}
template <int CTRL, int N>
__device__ __forceinline__ void rows_sum_step(float (&v)[N]) {
    float t[N];
#pragma unroll
    for (int r = 0; r < N; ++r) t[r] = dpp_move<CTRL>(v[r]);
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] += t[r];
}
template <int N>
__device__ __forceinline__ void rows_max(float (&v)[N]) {
    rows_max_step<0xB1>(v); rows_max_step<0x4E>(v); rows_max_step<0x141>(v); rows_max_step<0x140>(v);
    float t[N];
#pragma unroll
    for (int r = 0; r < N; ++r) t[r] = __shfl_xor(v[r], 16, RL_WAVE);
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = fmaxf(v[r], t[r]);
}
template <int N>
__device__ __forceinline__ void rows_sum(float (&v)[N]) {
    rows_sum_step<0xB1>(v); rows_sum_step<0x4E>(v); rows_sum_step<0x141>(v); rows_sum_step<0x140>(v);
    float t[N];
#pragma unroll
    for (int r = 0; r < N; ++r) t[r] = __shfl_xor(v[r], 16, RL_WAVE);
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] += t[r];
}
__device__ __forceinline__ float row32_sum(float v) {
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    return v + __shfl_xor(v, 16, RL_WAVE);
}

// Element of dimension d of token m in v_out, plane of one (lo / hi, kv head): [vt_cap / 32 tiles][hd][32 tokens].
__device__ __forceinline__ int64_t v_tile_off(const GemmArgs& a, int plane, int m, int d) {
    return (((int64_t)plane * (a.vt_cap >> 5) + (m >> 5)) * a.hd + d) * 32 + (m & 31);
}

// Epilogue of gemm_mfma_kernel for one 32-row band of a wave's accumulators: acc[j][r] of the
// wave in tile-column position wn is C(row, col) with
//   row = m_base + 8*(r/4) + 4*(lane/32) + r%4,   col(tile-local) = wn*TN*32 + j*32 + lane%32
template <int EPI, int BN, int TN, int WGN>
__device__ __forceinline__ void mg_epilogue(floatx16 (&acc)[TN], const GemmArgs& a, int m_base, int nb, int wn,
                                            int ks, int lane) {
    constexpr int NR = 16;
    const int lg = lane >> 5, lrow = lane & 31;
    if (EPI == MG_RESID) {
        // read-modify-write of the fp32 residual stream: all of the band's loads are issued before the
        // first add (rows past M read row M-1 instead of branching, so nothing separates the loads)
        float old[TN][NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int m = min(m_base + 8 * (r >> 2) + 4 * lg + (r & 3), a.M - 1);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                old[j][r] = a.outF[(int64_t)m * a.ldc + min(nb * BN + wn * TN * 32 + j * 32 + lrow, a.N - 1)];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int m = m_base + 8 * (r >> 2) + 4 * lg + (r & 3);
            if (m >= a.M) continue;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                int n = nb * BN + wn * TN * 32 + j * 32 + lrow;
                if (n < a.N) a.outF[(int64_t)m * a.ldc + n] = old[j][r] + acc[j][r];
            }
        }
        return;
    }
    if constexpr (EPI == MG_QKV) {
        // Columns of a wave belong to one head (hd 128) or two (hd 64); the rotation pairs (jj, jj + hd/2) sit in
        // adjacent 32-column MFMA tiles of a lane (acc[j], acc[j + 1]).  Everything the stores depend on is fetched
        // first, in batches -- positions and cache slots of the lane's 16 rows, their pages, the rotation factors
        // -- so that the band pays a few memory latencies instead of one per row: the stores that follow may
        // alias anything as far as the compiler knows, and a load behind a store waits for it.
        __builtin_amdgcn_sched_barrier(0);                    // one band at a time: the loads of the next one stay behind
        const int hd = a.hd, half = hd >> 1, Hq = a.Hq, Hkv = a.Hkv;
        const int c_first = wn * TN * 32;                     // tile-local column of acc[0], lane 0
        auto col_of = [&](int j) {                            // global qkv column of acc[j][.] of this lane
            const int c0 = c_first + j * 32 + lrow;
            return hd == 128 ? nb * BN + (c0 & ~127) + (((c0 & 127) >> 5) >> 1) * 32 + (c0 & 31) : nb * BN + c0;
        };
        const int head_hi = col_of(TN - 2) / hd;              // wave-uniform
        int pos[NR];                                           // < 0: padding row of the packed token list
        int page[NR];
        const bool to_pool = a.pool != nullptr && head_hi >= Hq;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int m = m_base + 8 * (r >> 2) + 4 * lg + (r & 3);
            const int p_ = a.tok_pos[min(m, a.M - 1)];
            pos[r] = m < a.M ? p_ : -1;
        }
        if (to_pool) {
            int slot[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) slot[r] = a.tok_slot[min(m_base + 8 * (r >> 2) + 4 * lg + (r & 3), a.M - 1)];
#pragma unroll
            for (int r = 0; r < NR; ++r)
                page[r] = a.block_table[(int64_t)(pos[r] >= 0 ? slot[r] : 0) * a.mpps + max(pos[r], 0) / a.geo.PT];
        }
        const int S = a.split_out ? 2 : 1;                     // fp16 pairs: rows of q and k are [hi heads | lo heads]
#pragma unroll
        for (int jp = 0; jp < TN / 2; ++jp) {
            const int j = 2 * jp, col0 = col_of(j);
            const int head = col0 / hd, jj = col0 % hd;        // jj < half; the partner column is jj + half
            if (head < Hq + Hkv) {
                float2 cs[NR];
#pragma unroll
                for (int r = 0; r < NR; ++r) cs[r] = a.rope[(int64_t)max(pos[r], 0) * half + jj];
                __builtin_amdgcn_sched_barrier(0);
                // q and k: rotate, round (and keep what the rounding left over), store token-major; k also to its page
#pragma unroll
                for (int r = 0; r < NR; ++r) {
                    const int m = m_base + 8 * (r >> 2) + 4 * lg + (r & 3);
                    if (m >= a.M) continue;
                    const bool pad = pos[r] < 0;               // padding rows get zeros: nothing non-finite is ever read back
                    const float x0 = pad ? 0.f : acc[j][r], x1 = pad ? 0.f : acc[j + 1][r];
                    const float v0 = rope_lo(x0, x1, cs[r].x, cs[r].y), v1 = rope_hi(x0, x1, cs[r].x, cs[r].y);
                    f16_t h0, l0, h1, l1;
                    split_f16(v0, h0, l0);
                    split_f16(v1, h1, l1);
                    if (head < Hq) {
                        f16_t* o = a.q_out + (int64_t)m * Hq * hd * S + head * hd + jj;
                        o[0] = h0; o[half] = h1;
                        if (a.split_out) { o[Hq * hd] = l0; o[Hq * hd + half] = l1; }
                    } else {
                        const int g = head - Hq;
                        if (a.k_out) {
                            f16_t* o = a.k_out + ((int64_t)m * Hkv * S + g) * hd + jj;
                            o[0] = h0; o[half] = h1;
                            if (a.split_out) { o[Hkv * hd] = l0; o[Hkv * hd + half] = l1; }
                        }
                        if (a.pool && !pad) {
                            const int st = pos[r] % a.geo.PT;
                            a.pool[a.geo.k_off(a.layer, page[r], g, st, jj)] = h0;
                            a.pool[a.geo.k_off(a.layer, page[r], g, st, jj + half)] = h1;
                            if (a.split_out) {
                                a.pool[a.geo.k_off(a.layer_lo, page[r], g, st, jj)] = l0;
                                a.pool[a.geo.k_off(a.layer_lo, page[r], g, st, jj + half)] = l1;
                            }
                        }
                    }
                }
                continue;
            }
            const int g = head - Hq - Hkv;
            // V with dim-major destinations (tiles of 32 tokens of v_out, and the V pages of the cache): the four
            // registers r = 4k .. 4k+3 of a lane are four consecutive tokens of one dimension, so they leave as one
            // 8-byte store instead of four 2-byte stores a cache line apart from their neighbours'.
#pragma unroll
            for (int rq = 0; rq < NR / 4; ++rq) {
                const int m4 = m_base + 8 * rq + 4 * lg;
                if (m4 >= a.M) continue;
                typedef _Float16 half4 __attribute__((ext_vector_type(4)));
                const int* p = &pos[4 * rq];
                const bool all = p[0] >= 0 && p[1] >= 0 && p[2] >= 0 && p[3] >= 0;
                // plane 0: the values rounded to fp16; plane 1 (split_out): what the rounding left over
                auto emit = [&](const int pl) {
                    half4 h0, h1;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float f0 = p[t] >= 0 ? acc[j][4 * rq + t] : 0.f, f1 = p[t] >= 0 ? acc[j + 1][4 * rq + t] : 0.f;
                        f16_t r0, r1, e0, e1;
                        split_f16(f0, r0, e0);
                        split_f16(f1, r1, e1);
                        h0[t] = pl == 0 ? r0 : e0;
                        h1[t] = pl == 0 ? r1 : e1;
                    }
                    if (a.v_out) {
                        f16_t* o0 = a.v_out + v_tile_off(a, pl * Hkv + g, m4, jj);
                        f16_t* o1 = o0 + half * 32;
                        if (m4 + 3 < a.M) {
                            *reinterpret_cast<half4*>(o0) = h0;
                            *reinterpret_cast<half4*>(o1) = h1;
                        } else {
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                if (m4 + t < a.M) { o0[t] = h0[t]; o1[t] = h1[t]; }
                        }
                    }
                    if (a.pool) {
                        const int lay = pl == 0 ? a.layer : a.layer_lo;
                        if (all && p[0] % 4 == 0 && p[3] == p[0] + 3) {   // four tokens of one sequence: same page, adjacent slots
                            const int st = p[0] % a.geo.PT;
                            *reinterpret_cast<half4*>(a.pool + a.geo.v_off(lay, page[4 * rq], g, st, jj)) = h0;
                            *reinterpret_cast<half4*>(a.pool + a.geo.v_off(lay, page[4 * rq], g, st, jj + half)) = h1;
                        } else {
#pragma unroll
                            for (int t = 0; t < 4; ++t)
                                if (p[t] >= 0) {
                                    const int st = p[t] % a.geo.PT;
                                    a.pool[a.geo.v_off(lay, page[4 * rq + t], g, st, jj)] = h0[t];
                                    a.pool[a.geo.v_off(lay, page[4 * rq + t], g, st, jj + half)] = h1[t];
                                }
                        }
                    }
                };
                emit(0);
                if (a.split_out) emit(1);
            }
        }
        return;
    }
    if constexpr (EPI == MG_SWIGLU) {
        // A band that lies wholly inside the matrix and leaves as plain fp16: no per-element bounds checks or branches, one row pointer per register row.  Same values as the general path.
        const int n_first = nb * (BN / 2) + wn * TN * 16;      // of this wave's TN * 16 output columns
        if (m_base + 2 * NR <= a.M && n_first + TN * 16 <= a.N && !a.split_out) {   // wave-uniform
            f16_t* o = a.outH + (int64_t)(m_base + 4 * lg) * a.ldc + n_first + lrow;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                f16_t* orow = o + (int64_t)(8 * (r >> 2) + (r & 3)) * a.ldc;
#pragma unroll
                for (int j = 0; j < TN; j += 2) orow[(j / 2) * 32] = (f16_t)swiglu_act(acc[j][r], acc[j + 1][r]);
            }
            return;
        }
    }
    if constexpr (EPI == MG_LSE) {
        // A band that lies wholly inside the matrix: the 16 rows' reductions run level by level, then the stores.  Same
        // values as the row-by-row form below.
        if (m_base + 2 * NR <= a.M) {                               // wave-uniform
            int tg[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) tg[r] = a.tgt[m_base + 8 * (r >> 2) + 4 * lg + (r & 3)];
            float mx[NR], se[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                mx[r] = acc[0][r];
#pragma unroll
                for (int j = 1; j < TN; ++j) mx[r] = fmaxf(mx[r], acc[j][r]);
            }
            rows_max(mx);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                se[r] = 0.f;
#pragma unroll
                for (int j = 0; j < TN; ++j) se[r] += __expf(acc[j][r] - mx[r]);
            }
            rows_sum(se);
            const int nparts = (a.N / BN) * WGN;
            const int c_first = nb * BN + wn * TN * 32 + lrow;   // this lane's column of acc[0]
            float2* part = a.lse_part + (int64_t)(m_base + 4 * lg) * nparts + nb * WGN + wn;
            float* zt = a.z_tgt + m_base + 4 * lg;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int ro = 8 * (r >> 2) + (r & 3);
                if (lrow == 0) part[(int64_t)ro * nparts] = make_float2(mx[r], se[r]);
                const int d = tg[r] - c_first;                  // 0, 32, ..: the target is this lane's column of acc[d / 32]
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (d == j * 32) zt[ro] = acc[j][r];
            }
            return;
        }
    }
    {
        // the targets of the lane's 16 rows, fetched before the first store (a load behind a store that may alias it
        // waits for the store)
        int tgt[EPI == MG_LSE ? NR : 1];
        if constexpr (EPI == MG_LSE) {
#pragma unroll
            for (int r = 0; r < NR; ++r) tgt[r] = a.tgt[min(m_base + 8 * (r >> 2) + 4 * lg + (r & 3), a.M - 1)];
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int m = m_base + 8 * (r >> 2) + 4 * lg + (r & 3);
            if (m >= a.M) continue;
            if (EPI == MG_STORE_F32) {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    int n = nb * BN + wn * TN * 32 + j * 32 + lrow;
                    if (n < a.N) a.outF[(int64_t)ks * a.split_stride + (int64_t)m * a.ldc + n] = acc[j][r];
                }
            } else if (EPI == MG_SWIGLU) {
#pragma unroll
                for (int j = 0; j < TN; j += 2) {
                    int n = nb * (BN / 2) + (wn * TN + j) / 2 * 32 + lrow;
                    const float act = swiglu_act(acc[j][r], acc[j + 1][r]);
                    if (n < a.N) {
                        if (a.split_out) {
                            f16_t hi, lo;
                            split_f16(act, hi, lo);
                            a.outH[(int64_t)m * a.ldc + n] = hi;
                            a.outH[(int64_t)m * a.ldc + a.N + n] = lo;
                        } else {
                            a.outH[(int64_t)m * a.ldc + n] = (f16_t)act;
                        }
                    }
                }
            } else if (EPI == MG_LSE) {
                // this wave's TN*32 columns of row m: running (max, sum of exponentials) over the
                // lanes that share the row (the 32 lanes of a half-wave), and the target's logit
                float mx = acc[0][r];
#pragma unroll
                for (int j = 1; j < TN; ++j) mx = fmaxf(mx, acc[j][r]);
                mx = row32_max(mx);
                float se = 0.f;
#pragma unroll
                for (int j = 0; j < TN; ++j) se += __expf(acc[j][r] - mx);
                se = row32_sum(se);
                const int nparts = (a.N / BN) * WGN;
                if (lrow == 0) a.lse_part[(int64_t)m * nparts + nb * WGN + wn] = make_float2(mx, se);
                const int t = tgt[EPI == MG_LSE ? r : 0];
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (t == nb * BN + wn * TN * 32 + j * 32 + lrow) a.z_tgt[m] = acc[j][r];
            }
        }
    }
}

// WF16: W points at an fp16 copy of the weights (nothing to convert on the way to LDS).
template <int BM, int BN, int WGM, int WGN, int EPI, int BKT, bool WF16>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(GemmArgs a) {
    constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
    constexpr int LSTR = BKT + 8;   // halfs per LDS row (+16 B pad: conflict-free ds_read_b128)
    constexpr int CPR = BKT / 8;    // 16-byte chunks per tile row
    constexpr int A_CH = BM * CPR / 256, W_CH = BN * CPR / 256;   // chunks per thread per k-tile
    extern __shared__ __attribute__((aligned(16))) char smem[];
    f16_t* As = reinterpret_cast<f16_t*>(smem);                   // [2][BM][LSTR]
    f16_t* Ws = As + 2 * BM * LSTR;                         // [2][BN][LSTR]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WGN, wn = wave % WGN;
    const int NB = a.n_blocks_n, MB = row_blocks(a, BM), ks = blockIdx.z;
    int nb, mb;
    if (!tile_of(blockIdx.x, MB, NB, mb, nb)) return;
    const int m0 = enter_row_block(a, BM, mb);
    const int kbeg = ks * a.k_per_split, kend = min(a.K, kbeg + a.k_per_split);
    const int nk = (kend - kbeg + BKT - 1) / BKT;

    // per-thread global source rows for the staged loads
    const f16_t* a_src[A_CH];
    const bf16_t* w_src[W_CH];
    int a_dst[A_CH], w_dst[W_CH];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
        int c = tid + i * 256, r = c / CPR, kc = c % CPR;
        int m = m0 + r;
        a_src[i] = a.A + (int64_t)min(m, a.M - 1) * a.lda + kc * 8;   // rows >= M: any finite-or-not data, never stored
        a_dst[i] = r * LSTR + kc * 8;
    }
#pragma unroll
    for (int i = 0; i < W_CH; ++i) {
        int c = tid + i * 256, r = c / CPR, kc = c % CPR;
        int wr = w_row_of<EPI, BN>(r, nb, a);
        w_src[i] = a.W + (int64_t)min(wr, a.Wrows - 1) * a.Kw + kc * 8;
        w_dst[i] = r * LSTR + kc * 8;
    }

    // Two register sets alternate between k-tiles: a tile is requested at the start of step kt-2's
    // successor... concretely, tile kt+2 is requested at the start of step kt and parked in LDS at
    // the end of step kt+1, so every global load has two full steps to arrive.  The steady-state
    // loop issues the same requests on every path (vector loads return in order; a wait count is
    // exact only then); prologue and the last two steps are peeled.
    u32x4_t ra0[A_CH], rw0[W_CH], ra1[A_CH], rw1[W_CH];
#define MG_LOAD(sl, kt)                                                                          \
    {                                                                                            \
        _Pragma("unroll") for (int i_ = 0; i_ < A_CH; ++i_)                                      \
            ra##sl[i_] = *reinterpret_cast<const u32x4_t*>(a_src[i_] + kbeg + (kt) * BKT);        \
        _Pragma("unroll") for (int i_ = 0; i_ < W_CH; ++i_)                                      \
            rw##sl[i_] = *reinterpret_cast<const u32x4_t*>(w_src[i_] + wrap_k(kbeg + (kt) * BKT, a.Kw));  \
    }
#define MG_PARK(sl, buf)                                                                         \
    {                                                                                            \
        _Pragma("unroll") for (int i_ = 0; i_ < A_CH; ++i_)                                      \
            *reinterpret_cast<u32x4_t*>(As + (buf) * BM * LSTR + a_dst[i_]) = ra##sl[i_];  \
        _Pragma("unroll") for (int i_ = 0; i_ < W_CH; ++i_)                                      \
            *reinterpret_cast<half8*>(Ws + (buf) * BN * LSTR + w_dst[i_]) =                      \
                WF16 ? __builtin_bit_cast(half8, rw##sl[i_]) : bf16x8_to_half8(rw##sl[i_]);      \
    }
    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    const int lrow = lane & 31, lk = (lane >> 5) * 8;
#define MG_FRAGS(dst_a, dst_b, kk)                                                               \
    _Pragma("unroll") for (int i = 0; i < TM; ++i)                                               \
        dst_a[i] = *reinterpret_cast<const half8*>(Ab + i * 32 * LSTR + (kk));             \
    _Pragma("unroll") for (int j = 0; j < TN; ++j)                                               \
        dst_b[j] = *reinterpret_cast<const half8*>(Wb + j * 32 * LSTR + (kk));
#define MG_MFMAS(src_a, src_b)                                                                   \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) _Pragma("unroll") for (int j = 0; j < TN; ++j) \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(src_a[i], src_b[j], acc[i][j], 0, 0, 0);
    // fragments of k-slice kk+16 are fetched from LDS while the MFMAs of slice kk run
#define MG_COMPUTE(buf)                                                                          \
    {                                                                                            \
        const f16_t* Ab = As + (buf) * BM * LSTR + (wm * TM * 32 + lrow) * LSTR + lk;            \
        const f16_t* Wb = Ws + (buf) * BN * LSTR + (wn * TN * 32 + lrow) * LSTR + lk;            \
        half8 afA[TM], bfA[TN], afB[TM], bfB[TN];                                                \
        MG_FRAGS(afA, bfA, 0)                                                                    \
        _Pragma("unroll") for (int kk = 0; kk < BKT; kk += 32) {                                 \
            MG_FRAGS(afB, bfB, kk + 16)                                                          \
            MG_MFMAS(afA, bfA)                                                                   \
            if (kk + 32 < BKT) { MG_FRAGS(afA, bfA, kk + 32) }                                   \
            MG_MFMAS(afB, bfB)                                                                   \
        }                                                                                        \
    }
    // step with tile parity p: request tile kt+2 into set p (its previous tile is already parked),
    // consume LDS buffer p, park set 1-p (tile kt+1) into buffer 1-p
#define MG_STEP_FULL(p, q, kt) { MG_LOAD(p, (kt) + 2) __builtin_amdgcn_sched_barrier(0); MG_COMPUTE(p) MG_PARK(q, q) __syncthreads(); }
#define MG_STEP_PARK(p, q)     { MG_COMPUTE(p) MG_PARK(q, q) __syncthreads(); }
#define MG_STEP_LAST(p)        { MG_COMPUTE(p) }
    if (nk >= 3) {
        MG_LOAD(0, 0)
        MG_LOAD(1, 1)
        MG_PARK(0, 0)
        __syncthreads();
        int kt = 0;
        for (; kt + 3 < nk; kt += 2) {
            MG_STEP_FULL(0, 1, kt)
            MG_STEP_FULL(1, 0, kt + 1)
        }
        if (nk - kt == 3) {
            MG_STEP_FULL(0, 1, kt)
            MG_STEP_PARK(1, 0)
            MG_STEP_LAST(0)
        } else {
            MG_STEP_PARK(0, 1)
            MG_STEP_LAST(1)
        }
    } else {
        for (int kt = 0; kt < nk; ++kt) {
            MG_LOAD(0, kt)
            MG_PARK(0, 0)
            __syncthreads();
            MG_COMPUTE(0)
            __syncthreads();
        }
    }
#undef MG_LOAD
#undef MG_PARK
#undef MG_COMPUTE
#undef MG_FRAGS
#undef MG_MFMAS
#undef MG_STEP_FULL
#undef MG_STEP_PARK
#undef MG_STEP_LAST

    // written out: with the largest epilogue the unroller gives up on a loop over the bands
    static_assert(TM <= 2, "bands written out below");
    mg_epilogue<EPI, BN, TN, WGN>(acc[0], a, m0 + wm * TM * 32, nb, wn, ks, lane);
    if (TM > 1) mg_epilogue<EPI, BN, TN, WGN>(acc[TM > 1 ? 1 : 0], a, m0 + wm * TM * 32 + 32, nb, wn, ks, lane);
}

// Row metadata of the MG_QKV epilogue held across a wave: lane l keeps position and cache page of rows row0 + l and
// row0 + 64 + l (fetched before the main loop, so that the epilogue starts without a chain of dependent loads).
struct QkvRowMeta {
    int pos[2] = {-1, -1};    // < 0: padding row / past M
    int page[2] = {0, 0};
};
__device__ __forceinline__ QkvRowMeta qkv_row_meta(const GemmArgs& a, int row0, int lane) {
    QkvRowMeta q;
    int slot[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int m = row0 + h * 64 + lane;
        const int p_ = a.tok_pos[min(m, a.M - 1)];
        slot[h] = a.pool ? a.tok_slot[min(m, a.M - 1)] : 0;
        q.pos[h] = m < a.M ? p_ : -1;
    }
    if (a.pool) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            q.page[h] = a.block_table[(int64_t)(q.pos[h] >= 0 ? slot[h] : 0) * a.mpps + max(q.pos[h], 0) / a.geo.PT];
    }
    return q;
}

// ------------------------------------------------------------------ tile GEMM with global -> LDS staging
// Stages of gemm_ring_kernel: what fits in 160 KB of LDS, at most eight.
static constexpr int ring_stages(int MI, int WGM, int WGN) {
    const int fit = 160 * 1024 / ((16 * MI * WGM + 64 * WGN) * 128);
    return fit < 8 ? fit : 8;
}

// Large-M GEMM, tiles of 32 MI rows x 256 columns (MI = 3 .. 8, by the number of rows: big_row_blocks), eight waves
// (2 x 4; 16 MI x 64 of C per wave; what follows says 128 x 64, MI = 8; two waves per SIMD, so a wave that waits
// -- at a barrier, for its fragment reads, behind a queued staging load -- leaves the SIMD's matrix core to the other
// one), operands staged global -> LDS through FIVE stages of 32 k with the loads of two consecutive k-tiles issued
// together.  A stage row is 64 B, half a 128-byte cache line, and a request for half a line makes the L2 deliver the
// whole line: with one k-tile per request group the L2 -> L1 path carries twice the operand bytes (counted: 4 sectors
// per request, the vector L1 stalled on pending requests for most of the kernel).  The loads of k-tiles 2p and 2p+1 --
// the two halves of the same lines -- go out back to back, so the second finds the line already on its way and one
// request per line reaches the L2.  A pair needs two free stages; with five stages the pair (p+4, p+5) is issued from
// the second slice of tile p (whose stage the barrier before it has released) to the end of tile p+1, spread over
// those three slices: bunched, the loads queue up in the vector memory path and hold back the MFMAs behind them.
// The matrix cores run 16x16x32 MFMAs, the shape that draws less power per flop (a register-only probe sustains 5 %
// more on it than on 32x32x16).  Per wave and k-tile: 2 + 2 staging loads, 8 A fragments (16 rows x 32 k each: one
// 16-byte read per lane) and 4 W fragments, 32 MFMAs in two slices of 16: slice 0 on rows 0-63 of the wave, slice 1 on
// rows 64-127.  During slice 0 the A fragments of rows 64-127 are read (same stage); during slice 1, behind the
// barrier that publishes the next k-tile, its W fragments and its A fragments of rows 0-63; of the pair's 4 loads per
// tile 2, 1, 1 go out in the three slices that may issue them.  Loads complete in issue order, so the waits are
// counts: inside an even k-tile p everything but the youngest 8 loads (pair p+2, p+3) has landed, i.e. tile p+1;
// inside an odd tile p+1 everything but the youngest 7 (tile p+3's last load and the 6 of pair p+4, p+5 issued so
// far), i.e. tile p+2.  The last four k-tiles, behind which nothing is left to ask for, are written out with counts of their
// own (re-requesting the final tile instead, for one form of the trip, kept the epilogue waiting for a memory latency: 0.3 % of a
// pass at 1B width, 4600 rows, and of the exact KL; within the noise of the other passes).
// WF16: W points at an fp16 copy of the weights and its fragments go from LDS straight into the MFMAs; otherwise W is
// bf16 and each fragment is converted (exactly) next to the MFMAs of slice 1, which costs 5-10 % of the loop.  Both
// forms feed the MFMAs the same values in the same order: their results are identical bit for bit.
// Requires K % 64 == 0 and K >= 128, no split over K, 5 * 512 * 64 bytes of LDS.
typedef float floatx4_t __attribute__((ext_vector_type(4)));
template <int EPI, bool WF16, int MI>
__device__ __forceinline__ void dma8_loop(const GemmArgs& a, const f16_t* Aop, int lda, const bf16_t* Wop, int m0, int nb, int wave,
                                          int lane, char* smem, floatx4_t (&acc)[MI][4], QkvRowMeta& meta) {
    constexpr int BM = 32 * MI, BN = 256, WGN = 4;
    constexpr int MI0 = (MI + 1) / 2, MI1 = MI / 2;      // 16-row blocks of the wave in slice 0 and in slice 1
    constexpr int STAGE = (BM + BN) * 64;
    constexpr int LPA = (BM + 127) / 128, LPT = LPA + 2;  // staging loads per wave and k-tile: of A, in all
    const int wm = wave / WGN, wn = wave % WGN;
    const int nk = a.K / 32, nkw = a.Kw / 32;
    // 16-row block of its operand that load l of this wave stages; where A has fewer blocks than 8 LPA, the waves left
    // over stage a block twice (same bytes to the same place), so that every wave counts the same loads
#define X8_BLOCK(l)                                                                                             \
    ((l) >= LPA ? ((l) - LPA) * 8 + wave                                                                        \
                : (l) * 8 + wave < BM / 16 ? (l) * 8 + wave : (l) * 8 + wave - ((l) > 0 ? 8 : BM / 16))
    unsigned g_off[LPT];
    {
        const int lc = (lane & 3) ^ ((lane >> 4) & 3);
#pragma unroll
        for (int l = 0; l < LPT; ++l) {
            const int r = X8_BLOCK(l) * 16 + (lane >> 2);
            g_off[l] = l < LPA ? ((unsigned)min(m0 + r, a.M - 1) * (unsigned)lda + lc * 8) * 2u   // rows >= M: clamped, never stored
                             : ((unsigned)min(w_row_of<EPI, BN>(r, nb, a), a.Wrows - 1) * (unsigned)a.Kw + lc * 8) * 2u;
        }
    }
    const char* Ag = reinterpret_cast<const char*>(Aop);
    const char* Wg = reinterpret_cast<const char*>(Wop);
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
#define X8_LOAD(st, kt, l)                                                                                      \
    {                                                                                                           \
        const int kt_ = (kt);                                                                                   \
        const unsigned sa_ = lds_base + (st) * STAGE + ((l) >= LPA ? BM * 64 : 0) + X8_BLOCK(l) * 1024;         \
        const char* g_ = (l) < LPA ? Ag + (size_t)kt_ * 64 : Wg + (size_t)wrap_k(kt_, nkw) * 64;                \
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"                            \
                     :: "s"(sa_), "v"(g_off[l]), "s"(g_) : "memory");                                           \
    }
    // fragment offsets inside a stage: row lane % 16 of a 16-row block, logical 16-byte chunk lane / 16, swizzled
    const int fr = lane & 15;
    const int fko = ((lane >> 4) ^ ((fr >> 2) & 3)) * 16;
    const int fa = (wm * MI * 16 + fr) * 64 + fko;                 // + i * 1024 for the i-th 16-row block of the wave
    const int fw = BM * 64 + (wn * 64 + fr) * 64 + fko;        // + j * 1024
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    half8 af[2][MI0];
    u32x4_t wf[2][4], bw[WF16 ? 1 : 4];   // W fragments as they go into the MFMAs; bf16 fragments waiting for their conversion
#define X8_CVT2(w) __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(__uint_as_float((w) << 16), __uint_as_float((w) & 0xffff0000u)))
#define X8_LDA(so, i) *reinterpret_cast<const half8*>(smem + (so) + fa + (i) * 1024)
#define X8_LDW(so, j) *reinterpret_cast<const u32x4_t*>(smem + (so) + fw + (j) * 1024)
    // One slice: NQ = 4 MI0 or 4 MI1 MFMAs on A set AS (slice 0: the wave's first MI0 row blocks, slice 1: the others) and
    // W set WS.  The fragment reads are spread behind the first MFMAs (slice 0: the row blocks of slice 1, stage NSO,
    // into A set 1; slice 1: W of stage NSO into W set 1 - WS, then the row blocks of slice 0 into A set 0), LOADS pairs
    // of staging loads behind the last quarter.  With MI = 8: reads behind MFMAs 0, 2, 4, 6 / 0 - 3 and 4, 6, 8, 10,
    // conversions behind 8 - 15, loads behind 12, 14.  The MFMAs walk the row blocks back and forth, so that each shares an
    // operand with the one before it: 0.3 - 0.7 % on whole passes (8B width, 4000 to 16384 rows), where power sets the pace.
#define X8_SLICE(AS, WS, NSO, LOADS, LB, PT, PS0, PS1) X8_SLICE_(AS, WS, true, NSO, LOADS, LB, PT, PS0, PS1)
#define X8_SLICE_(AS, WS, READS, NSO, LOADS, LB, PT, PS0, PS1)                                                  \
    _Pragma("unroll") for (int q = 0; q < 4 * ((AS) ? MI1 : MI0); ++q) {                                        \
        constexpr int NI_ = (AS) ? MI1 : MI0, NQ_ = 4 * NI_;                                                    \
        const int j_ = q / NI_, i_ = (j_ & 1) ? NI_ - 1 - q % NI_ : q % NI_;                                    \
        acc[(AS) * MI0 + i_][j_] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, wf[WS][j_]), af[AS][i_], acc[(AS) * MI0 + i_][j_], 0, 0, 0); \
        if (!(READS)) {                                                                                         \
        } else if ((AS) == 0) {                                                                                 \
            _Pragma("unroll") for (int u_ = 0; u_ < MI1; ++u_)                                                  \
                if (u_ * (NQ_ / 2) / MI1 == q) af[1][u_] = X8_LDA(NSO, MI0 + u_);                               \
        } else {                                                                                                \
            _Pragma("unroll") for (int u_ = 0; u_ < 4; ++u_)                                                    \
                if (u_ * NQ_ / 16 == q) {                                                                       \
                    if (WF16) wf[1 - (WS)][u_] = X8_LDW(NSO, u_);                                               \
                    else bw[WF16 ? 0 : u_] = X8_LDW(NSO, u_);                                                   \
                }                                                                                               \
            _Pragma("unroll") for (int u_ = 0; u_ < MI0; ++u_)                                                  \
                if (NQ_ / 4 + u_ * (NQ_ / 2) / MI0 == q) af[0][u_] = X8_LDA(NSO, u_);                           \
            _Pragma("unroll") for (int c_ = 0; c_ < 8; ++c_)   /* half a bf16 fragment -> fp16 per unit */      \
                if (!WF16 && NQ_ / 2 + c_ * (NQ_ / 2) / 8 == q) {                                               \
                    const int jj_ = c_ >> 1, h_ = (c_ & 1) * 2;                                                 \
                    wf[1 - (WS)][jj_][h_] = X8_CVT2(bw[WF16 ? 0 : jj_][h_]);                                    \
                    wf[1 - (WS)][jj_][h_ + 1] = X8_CVT2(bw[WF16 ? 0 : jj_][h_ + 1]);                            \
                }                                                                                               \
        }                                                                                                       \
        _Pragma("unroll") for (int u_ = 0; u_ < (LOADS); ++u_)                                                  \
            if (NQ_ - NQ_ / 4 + u_ * (NQ_ / 8) == q) {                                                          \
                X8_LOAD(PS0, PT, (LB) + u_)                                                                     \
                X8_LOAD(PS1, (PT) + 1, (LB) + u_)                                                               \
            }                                                                                                   \
        __builtin_amdgcn_sched_barrier(0);                                                                      \
    }
    int s0 = 0, s1 = 1, s2 = 2, s3 = 3, s4 = 4;
#pragma unroll
    for (int l = 0; l < LPT; ++l) { X8_LOAD(0, 0, l) X8_LOAD(1, 1, l) }
#pragma unroll
    for (int l = 0; l < LPT; ++l) { X8_LOAD(2, 2, l) X8_LOAD(3, 3, l) }
    if constexpr (EPI == MG_QKV) meta = qkv_row_meta(a, m0 + wm * MI * 16, lane);
    __builtin_amdgcn_s_waitcnt(dma_waitcnt(EPI == MG_QKV ? 0 : 2 * LPT + 1, 15));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MI0; ++i) af[0][i] = X8_LDA(0, i);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const u32x4_t w_ = X8_LDW(0, j);
#pragma unroll
        for (int c = 0; c < 4; ++c) wf[0][j][c] = WF16 ? w_[c] : X8_CVT2(w_[c]);
    }
    // Even k-tile kt (W set 0): slice 0, barrier (tile kt+1 complete, stage of tile kt released after this slice's reads), slice 1
    // with the first loads of pair (kt+4, kt+5); odd k-tile kt+1 (W set 1) alike, its barrier completing tile kt+2.
    int kt = 0;
    for (; kt < nk - 4; kt += 2) {
        const int o0 = s0 * STAGE, o1 = s1 * STAGE, o2 = s2 * STAGE;
        X8_SLICE(0, 0, o0, 0, 0, 0, 0, 0)
        __builtin_amdgcn_s_waitcnt(dma_waitcnt(2 * LPT, 0));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        X8_SLICE(1, 0, o1, LPT - 2, 0, kt + 4, s4, s0)
        X8_SLICE(0, 1, o1, 1, LPT - 2, kt + 4, s4, s0)
        __builtin_amdgcn_s_waitcnt(dma_waitcnt(2 * (LPT - 1) + 1, 0));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        X8_SLICE(1, 1, o2, 1, LPT - 1, kt + 4, s4, s0)
        const int t0 = s0, t1 = s1;
        s0 = s2; s1 = s3; s2 = s4; s3 = t0; s4 = t1;
    }
    // The last four k-tiles, nothing left to ask for (asking for the final tile again, to keep one form of the trip, leaves a
    // memory latency between the last MFMAs and the epilogue).  Behind tile nk - 2 only its pair's last load is younger.
    {
        const int o0 = s0 * STAGE, o1 = s1 * STAGE, o2 = s2 * STAGE, o3 = s3 * STAGE;
        X8_SLICE(0, 0, o0, 0, 0, 0, 0, 0)
        __builtin_amdgcn_s_waitcnt(dma_waitcnt(2 * LPT, 0));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        X8_SLICE(1, 0, o1, 0, 0, 0, 0, 0)
        X8_SLICE(0, 1, o1, 0, 0, 0, 0, 0)
        __builtin_amdgcn_s_waitcnt(dma_waitcnt(1, 0));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        X8_SLICE(1, 1, o2, 0, 0, 0, 0, 0)
        X8_SLICE(0, 0, o2, 0, 0, 0, 0, 0)
        __builtin_amdgcn_s_waitcnt(dma_waitcnt(0, 0));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        X8_SLICE(1, 0, o3, 0, 0, 0, 0, 0)
        X8_SLICE(0, 1, o3, 0, 0, 0, 0, 0)
        X8_SLICE_(1, 1, false, 0, 0, 0, 0, 0, 0)
    }
    __builtin_amdgcn_s_waitcnt(dma_waitcnt(0, 0));    // nothing is on its way to LDS
#undef X8_LOAD
#undef X8_BLOCK
#undef X8_CVT2
#undef X8_LDA
#undef X8_LDW
#undef X8_SLICE
#undef X8_SLICE_
}

// ---- epilogues of the large-M kernel.  A wave's accumulators pass through its own LDS patch, 64 rows x 64 columns of
// fp32 at a time, and come back with whole row pieces in each lane, so that everything that leaves is 16 bytes per lane
// and stores and LDS accesses are few: with all 256 tiles of a round ending together, the matrix cores idle for as
// long as an epilogue takes.  Row stride 68 floats: eight lanes on eight rows, or on two rows, meet no bank conflict.
// W goes into the MFMAs as the first operand, so that a lane holds row lane % 16 of a 16 x 16 block and its
// columns 4 * (lane / 16) .. + 3: 16-byte writes as well.  Against stores of one element per lane, 16384 rows of the 8B
// shape: LM head 13.33 -> 12.21 ms, QKV 712 -> 647 us, residual and gate/up the same within 1 %: theirs wait for memory.
static constexpr int PATCH_LD = 68;

// Blocks FIRST .. FIRST + NB - 1 (16 rows each) of the wave's accumulators into the patch.
template <int NB, int FIRST, int MI>
__device__ __forceinline__ void patch_put(const floatx4_t (&acc)[MI][4], float* patch, int lane) {
    float* const p = patch + (lane & 15) * PATCH_LD + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<floatx4_t*>(p + i * 16 * PATCH_LD + j * 16) = acc[FIRST + i][j];
    __builtin_amdgcn_wave_barrier();          // LDS accesses of a wave complete in order
}
template <int N>
__device__ __forceinline__ void patch_get(float (&v)[N], const float* patch, int row, int col) {
#pragma unroll
    for (int x = 0; x < N / 4; ++x) {
        const floatx4_t t = *reinterpret_cast<const floatx4_t*>(patch + row * PATCH_LD + col + 4 * x);
#pragma unroll
        for (int y = 0; y < 4; ++y) v[4 * x + y] = t[y];
    }
}
// Maximum and sum of a lane's 16 values, columns c .. c + 7 and c + 32 .. c + 39 of a wave's 64 where its quad holds the
// others (c = 0, 8, 16, 24).  The sum pairs the columns 32 apart, then 1, 2 and 4 apart (quad_sum goes on with 8 and 16): a
// term is rounded at six additions, one after the other it would be at up to 17, and the exact KL is a small difference of
// such sums (error against 64 bits 0.5 to 16 % larger, V = 131072 to 256).
__device__ __forceinline__ float max_of(const float (&v0)[8], const float (&v1)[8]) {
    float m = v0[0];
#pragma unroll
    for (int x = 0; x < 8; ++x) m = fmaxf(m, fmaxf(v0[x], v1[x]));
    return m;
}
__device__ __forceinline__ float sum_of(const float (&v)[8]) {
    return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
}
// over the four lanes of a quad, every lane with the same bits
__device__ __forceinline__ float quad_max(float v) {
    v = fmaxf(v, dpp_move<0xB1>(v));          // quad_perm [1,0,3,2]
    return fmaxf(v, dpp_move<0x4E>(v));       // quad_perm [2,3,0,1]
}
__device__ __forceinline__ float quad_sum(float v) {
    v += dpp_move<0xB1>(v);
    return v + dpp_move<0x4E>(v);
}
// eight floats as fp16 pairs
__device__ __forceinline__ void split8(const float (&v)[8], half8& hi, half8& lo) {
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        f16_t h, l;
        split_f16(v[x], h, l);
        hi[x] = h;
        lo[x] = l;
    }
}

// Rows HF * 64 .. of the wave (at most 64; m0 the first of them) of a tile in column block nb, wave column wn.
template <int EPI, int MI, int HF>
__device__ __forceinline__ void d8_half(const floatx4_t (&acc)[MI][4], float* patch, const GemmArgs& a, int m0, int nb,
                                        int wn, int lane, const QkvRowMeta& meta) {
    constexpr int NB = MI - HF * 4 < 4 ? MI - HF * 4 : 4;            // its 16-row blocks
    if constexpr (EPI == MG_RESID || EPI == MG_STORE_F32) {
        // four rows of 256 bytes per access.  The residual's loads all go out first (rows past M read row M - 1)
        const int row = lane >> 4, c = nb * 256 + wn * 64 + (lane & 15) * 4;
        floatx4_t old[NB * 4];
        if constexpr (EPI == MG_RESID) {
#pragma unroll
            for (int it = 0; it < NB * 4; ++it)
                old[it] = *reinterpret_cast<const floatx4_t*>(a.outF + (int64_t)min(m0 + it * 4 + row, a.M - 1) * a.ldc + c);
            __builtin_amdgcn_sched_barrier(0);
        }
        patch_put<NB, HF * 4>(acc, patch, lane);
#pragma unroll
        for (int it = 0; it < NB * 4; ++it) {
            const int m = m0 + it * 4 + row;
            floatx4_t v = *reinterpret_cast<const floatx4_t*>(patch + (it * 4 + row) * PATCH_LD + (lane & 15) * 4);
            if constexpr (EPI == MG_RESID) {
#pragma unroll
                for (int x = 0; x < 4; ++x) v[x] = old[it][x] + v[x];
            }
            if (m < a.M) *reinterpret_cast<floatx4_t*>(a.outF + (int64_t)m * a.ldc + c) = v;
        }
    } else if constexpr (EPI == MG_SWIGLU) {
        // columns 0 .. 31 of the wave are gates, 32 .. 63 the up projections of the same output columns; a quad of
        // lanes holds a row
        const int row = lane >> 2, c = (lane & 3) * 8;
        f16_t* const o = a.outH + nb * 128 + wn * 32 + c;
        patch_put<NB, HF * 4>(acc, patch, lane);
#pragma unroll
        for (int it = 0; it < NB; ++it) {
            const int m = m0 + it * 16 + row;
            float g[8], u[8], act[8];
            patch_get(g, patch, it * 16 + row, c);
            patch_get(u, patch, it * 16 + row, 32 + c);
#pragma unroll
            for (int x = 0; x < 8; ++x) act[x] = swiglu_act(g[x], u[x]);
            half8 hi, lo;
            split8(act, hi, lo);
            if (m < a.M) {
                *reinterpret_cast<half8*>(o + (int64_t)m * a.ldc) = hi;
                if (a.split_out) *reinterpret_cast<half8*>(o + (int64_t)m * a.ldc + a.N) = lo;
            }
        }
    } else if constexpr (EPI == MG_QKV) {
        // The wave's columns belong to one head: columns w and w + 32 are the rotation pair (jb + w, jb + w + hd / 2)
        const int hd = a.hd, half = hd >> 1, Hq = a.Hq, Hkv = a.Hkv;
        const int head = hd == 128 ? nb * 2 + (wn >> 1) : nb * 4 + wn, jb = hd == 128 ? (wn & 1) * 32 : 0;
        const int S = a.split_out ? 2 : 1;                     // fp16 pairs: rows of q and k are [hi heads | lo heads]
        if (head < Hq + Hkv) {
            // q and k: a quad of lanes per row rotates eight pairs each, rounds (and keeps what the rounding left over),
            // stores token-major; k also to its page.  The rotation factors go out first
            const int row = lane >> 2, c = (lane & 3) * 8;
            int pos[NB], page[NB];
            floatx4_t cs[NB][4];                               // (cos, sin) of two columns each
#pragma unroll
            for (int it = 0; it < NB; ++it) {
                pos[it] = __shfl(meta.pos[HF], it * 16 + row, RL_WAVE);
                page[it] = __shfl(meta.page[HF], it * 16 + row, RL_WAVE);
                const float2* t = a.rope + (int64_t)max(pos[it], 0) * half + jb + c;
#pragma unroll
                for (int x = 0; x < 4; ++x) cs[it][x] = *reinterpret_cast<const floatx4_t*>(t + 2 * x);
            }
            __builtin_amdgcn_sched_barrier(0);
            patch_put<NB, HF * 4>(acc, patch, lane);
#pragma unroll
            for (int it = 0; it < NB; ++it) {
                const int m = m0 + it * 16 + row;
                const bool pad = pos[it] < 0;                  // padding rows get zeros: nothing non-finite is ever read back
                float x0[8], x1[8], v0[8], v1[8];
                patch_get(x0, patch, it * 16 + row, c);
                patch_get(x1, patch, it * 16 + row, 32 + c);
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    const float cx = cs[it][x >> 1][(x & 1) * 2], sx = cs[it][x >> 1][(x & 1) * 2 + 1];
                    v0[x] = pad ? 0.f : rope_lo(x0[x], x1[x], cx, sx);
                    v1[x] = pad ? 0.f : rope_hi(x0[x], x1[x], cx, sx);
                }
                if (m >= a.M) continue;
                auto put = [](f16_t* p, int far, half8 h0, half8 h1) {
                    *reinterpret_cast<half8*>(p) = h0;
                    *reinterpret_cast<half8*>(p + far) = h1;
                };
                half8 h0, l0, h1, l1;
                split8(v0, h0, l0);
                split8(v1, h1, l1);
                const int jj = jb + c;
                if (head < Hq) {
                    f16_t* o = a.q_out + (int64_t)m * Hq * hd * S + head * hd + jj;
                    put(o, half, h0, h1);
                    if (a.split_out) put(o + Hq * hd, half, l0, l1);
                } else {
                    const int g = head - Hq;
                    if (a.k_out) {
                        f16_t* o = a.k_out + ((int64_t)m * Hkv * S + g) * hd + jj;
                        put(o, half, h0, h1);
                        if (a.split_out) put(o + Hkv * hd, half, l0, l1);
                    }
                    if (a.pool && !pad) {
                        const int st = pos[it] % a.geo.PT;
                        put(a.pool + a.geo.k_off(a.layer, page[it], g, st, jj), half, h0, h1);
                        if (a.split_out) put(a.pool + a.geo.k_off(a.layer_lo, page[it], g, st, jj), half, l0, l1);
                    }
                }
            }
        } else {
            // V with dim-major destinations (tiles of 32 tokens of v_out, and the V pages of the cache): a lane takes eight
            // consecutive tokens of one dimension, 16 dimensions x 32 tokens per step
            const int g = head - Hq - Hkv;
            patch_put<NB, HF * 4>(acc, patch, lane);
#pragma unroll
            for (int rb = 0; rb < (NB + 1) / 2; ++rb) {
                const int r0 = rb * 32 + (lane >> 4) * 8;      // first token; m0 + r0 is a multiple of 8
                int pos[8], page[8];
                bool run = r0 < NB * 16 && m0 + r0 + 7 < a.M;  // eight tokens of one sequence in one page
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    pos[t] = __shfl(meta.pos[HF], (r0 + t) & 63, RL_WAVE);
                    page[t] = __shfl(meta.page[HF], (r0 + t) & 63, RL_WAVE);
                    run = run && pos[t] == pos[0] + t;
                }
                run = run && pos[0] >= 0 && pos[0] % 8 == 0;
                if (r0 >= NB * 16) continue;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) {
                    const int w = cb * 16 + (lane & 15);
                    const int dim = w < 32 ? jb + w : half + jb + w - 32;
                    float v[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) v[t] = pos[t] < 0 ? 0.f : patch[(r0 + t) * PATCH_LD + w];
                    half8 hi, lo;
                    split8(v, hi, lo);
                    for (int pl = 0; pl < S; ++pl) {           // plane 1: what the rounding left over
                        const half8 h = pl == 0 ? hi : lo;
                        if (a.v_out) {
                            f16_t* o = a.v_out + v_tile_off(a, pl * Hkv + g, m0 + r0, dim);
                            if (m0 + r0 + 7 < a.M) *reinterpret_cast<half8*>(o) = h;
                            else {
#pragma unroll
                                for (int t = 0; t < 8; ++t)
                                    if (m0 + r0 + t < a.M) o[t] = h[t];
                            }
                        }
                        if (a.pool) {
                            const int lay = pl == 0 ? a.layer : a.layer_lo;
                            if (run) *reinterpret_cast<half8*>(a.pool + a.geo.v_off(lay, page[0], g, pos[0] % a.geo.PT, dim)) = h;
                            else {
#pragma unroll
                                for (int t = 0; t < 8; ++t)
                                    if (pos[t] >= 0) a.pool[a.geo.v_off(lay, page[t], g, pos[t] % a.geo.PT, dim)] = h[t];
                            }
                        }
                    }
                }
            }
        }
    } else if constexpr (EPI == MG_LSE) {
        // maximum and sum of exponentials of the wave's 64 columns: a quad of lanes per row, lane q taking columns 8 q ..
        // 8 q + 7 and those 32 further on: the sums form the tree of the 128 x 128 kernel's reduction (columns 32 apart, then
        // 1, 2, 4, 8, 16 apart), and its bits
        const int row = lane >> 2, c = (lane & 3) * 8, n0 = nb * 256 + wn * 64;
        int tg[NB];
#pragma unroll
        for (int it = 0; it < NB; ++it) tg[it] = a.tgt[min(m0 + it * 16 + row, a.M - 1)];
        __builtin_amdgcn_sched_barrier(0);
        patch_put<NB, HF * 4>(acc, patch, lane);
        const int nparts = a.N / 64;
#pragma unroll
        for (int it = 0; it < NB; ++it) {
            const int m = m0 + it * 16 + row;
            float z0[8], z1[8], e[8];
            patch_get(z0, patch, it * 16 + row, c);
            patch_get(z1, patch, it * 16 + row, 32 + c);
            const float mx = quad_max(max_of(z0, z1));
#pragma unroll
            for (int x = 0; x < 8; ++x) e[x] = __expf(z0[x] - mx) + __expf(z1[x] - mx);
            const float se = quad_sum(sum_of(e));
            if ((lane & 3) == 0 && m < a.M) {
                a.lse_part[(int64_t)m * nparts + nb * 4 + wn] = make_float2(mx, se);
                const int d = tg[it] - n0;
                if (d >= 0 && d < 64) a.z_tgt[m] = patch[(it * 16 + row) * PATCH_LD + d];
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
}

template <int EPI, bool WF16, int MI>
__global__ __launch_bounds__(512, 1) void gemm_dma8_kernel(GemmArgs a) {
    constexpr int BM = 32 * MI, WGN = 4;
    extern __shared__ __attribute__((aligned(1024))) char smem[];   // [5 stages][A BM x 64 B | W 256 x 64 B]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    int nb, mb;
    if (!tile_of(blockIdx.x, row_blocks(a, BM), a.n_blocks_n, mb, nb)) return;
    const int m0 = enter_row_block(a, BM, mb);
    floatx4_t acc[MI][4];
    QkvRowMeta meta;
    dma8_loop<EPI, WF16, MI>(a, a.A, a.lda, a.W, m0, nb, wave, lane, smem, acc, meta);
    __syncthreads();                                   // every wave is done with the stages: LDS is free
    float* const patch = reinterpret_cast<float*>(smem) + wave * (64 * PATCH_LD);
    const int m_w = m0 + wm * MI * 16;
    d8_half<EPI, MI, 0>(acc, patch, a, m_w, nb, wn, lane, meta);
    if constexpr (MI > 4) d8_half<EPI, MI, 1>(acc, patch, a, m_w + 64, nb, wn, lane, meta);
}

// GEMMs below the large-M kernel whose weights are there as fp16: tiles of 16 MI WGM rows x 64 WGN columns, WGM x WGN waves of
// 16 MI x 64 each, operands global -> LDS in k-tiles of 64 through as many stages as fit.  Such a GEMM has at most one workgroup
// per CU and is bound by what that workgroup draws: measured, a CU has about 64 KB on its way at once, which is 115 - 145
// KB/us from L2, 95 behind it and 62 - 65 from memory, whatever the row stride and however many stages wait.  So all of them are
// kept on their way and nothing else may show: one barrier per k-tile, in its middle; the fragments of the second 32 k are read
// under the MFMAs of the first, those of the next k-tile under the second's, and the k-tile that fills the freed stage is
// requested among the same MFMAs.  0.53 us per k-tile of 128 x 128 tiles (0.37 with its operands in L2; the MFMAs alone 0.25)
// against 0.66 staged through registers.  bf16 weights stay with that kernel: it converts them once on their way to LDS, here
// every wave would on its own.
// 16-byte chunks of a 128-byte row are XOR-swizzled with (row / 2) % 8 on the source side of the loads (fragment reads: 16 rows,
// one 16-byte read per lane).  MFMAs, their order along k and the epilogues are the large-M kernel's: a row's bits do not depend
// on which of the kernels runs.  The tile's columns are half or a quarter of a 256-column tile there.  Offsets count from the
// tile's first row of A and of W.
template <int EPI, int MI, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_ring_kernel(GemmArgs a) {
    constexpr int BM = 16 * MI * WGM, BN = 64 * WGN, NWV = WGM * WGN, RB = 128, QC = 256 / BN;   // QC: tiles per 256 columns
    constexpr int S = ring_stages(MI, WGM, WGN), ST = (BM + BN) * RB, NI = (BM + BN) / 8 / NWV;
    static_assert((BM + BN) / 8 % NWV == 0, "every wave counts the same loads");
    extern __shared__ __attribute__((aligned(1024))) char smem[];   // [S][A BM x 128 B | W BN x 128 B]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    int nt, mb;
    if (!tile_of(blockIdx.x, row_blocks(a, BM), a.n_blocks_n, mb, nt)) return;
    const int m0 = enter_row_block(a, BM, mb);
    const int nb = nt / QC, c0 = nt % QC * BN;                       // 256-column tile, first column in it
    const int nk = a.K / 64, nkw = a.Kw / 64;
    const int w_first = w_row_of<EPI, 256>(c0, nb, a);
    const char* const Ag = reinterpret_cast<const char*>(a.A + (int64_t)m0 * a.lda);
    const char* const Wg = reinterpret_cast<const char*>(a.W + (int64_t)min(w_first, a.Wrows - 1) * a.Kw);
    // request t of a wave: the 1 KB block t * NWV + wave = 8 rows of a stage; lane -> row + lane / 8, chunk lane % 8
    unsigned off[NI];
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        const int row = (t * NWV + wave) * 8 + (lane >> 3);
        const unsigned ch = (unsigned)((lane & 7) ^ ((row >> 1) & 7)) * 16u;
        if ((t * NWV + wave) * 8 < BM) off[t] = (unsigned)min(row, a.M - 1 - m0) * (unsigned)a.lda * 2u + ch;   // rows >= M: clamped, never stored
        else off[t] = (unsigned)(min(w_row_of<EPI, 256>(c0 + row - BM, nb, a), a.Wrows - 1) - min(w_first, a.Wrows - 1)) * (unsigned)a.Kw * 2u + ch;
    }
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem + wave * 1024;
    // request t of k-tile kt
#define RG_ISSUE1(stage, kt, t)                                                                                 \
    {                                                                                                           \
        const int k_ = (kt);                                                                                    \
        const unsigned l_ = lds0 + (stage) * ST + (t) * (NWV * 1024);                                           \
        const char* g_ = ((t) * NWV + wave) * 8 < BM ? Ag + (size_t)k_ * RB : Wg + (size_t)wrap_k(k_, nkw) * RB; \
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(l_), "v"(off[t]), "s"(g_) : "memory"); \
    }
    floatx4_t acc[MI][4];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    const int fr = lane & 15, q = lane >> 4, sw = (fr >> 1) & 7;
    const int fa = (wm * MI * 16 + fr) * RB, fw = (BM + wn * 64 + fr) * RB;
    const int ch0 = (q ^ sw) * 16, ch1 = ((4 + q) ^ sw) * 16;        // this lane's chunk of the first and of the second 32 k
    half8 af[2][MI];
    half8 wf[2][4];
#define RG_READ(set, u, so, ch)                                                                                 \
    if ((u) < 4) wf[set][(u) & 3] = *reinterpret_cast<const half8*>((so) + fw + (u) * 16 * RB + (ch));        \
    else if ((u) < 4 + MI) af[set][(u) < 4 + MI && (u) >= 4 ? (u) - 4 : 0] = *reinterpret_cast<const half8*>((so) + fa + ((u) - 4) * 16 * RB + (ch));
    // 4 MI MFMAs on fragment set `set`; behind them the reads of the other set, and LOADS: the requests of k-tile PT
#define RG_SLICE(set, READS, so, ch, LOADS, stage, PT)                                                          \
    _Pragma("unroll") for (int n = 0; n < 4 * MI; ++n) {                                                        \
        const int j_ = n / MI, i_ = (j_ & 1) ? MI - 1 - n % MI : n % MI;                                        \
        acc[i_][j_] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[set][j_], af[set][i_], acc[i_][j_], 0, 0, 0);   \
        _Pragma("unroll") for (int u = 0; u < 4 + MI; ++u)                                                      \
            if ((READS) && u * 4 * MI / (4 + MI) == n) { RG_READ(1 - (set), u, so, ch) }                        \
        _Pragma("unroll") for (int t = 0; t < NI; ++t)                                                          \
            if ((LOADS) && (t * 4 * MI + 2 * MI) / NI == n) { RG_ISSUE1(stage, PT, t) }                         \
        __builtin_amdgcn_sched_barrier(0);                                                                      \
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s < nk) {
#pragma unroll
            for (int t = 0; t < NI; ++t) RG_ISSUE1(s, s, t)
        }
    QkvRowMeta meta;
    if constexpr (EPI == MG_QKV) meta = qkv_row_meta(a, m0 + wm * MI * 16, lane);
    if (EPI == MG_QKV || nk < S) __builtin_amdgcn_s_waitcnt(dma_waitcnt(0, 15));
    else __builtin_amdgcn_s_waitcnt(dma_waitcnt(NI * (S - 1), 15));
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4 + MI; ++u) { RG_READ(0, u, smem, ch0) }
    int st = 0, kt = 0;
    // k-tile kt: its first 32 k, barrier (k-tile kt + 1 landed; every wave has read its fragments of k-tile kt, whose stage is
    // free), its second 32 k
    for (; kt < nk - S; ++kt) {
        const int nx = st + 1 == S ? 0 : st + 1;
        RG_SLICE(0, true, smem + st * ST, ch1, false, 0, 0)
        __builtin_amdgcn_s_waitcnt(dma_waitcnt(NI * (S - 2), 0));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        RG_SLICE(1, true, smem + nx * ST, ch0, true, st, kt + S)
        st = nx;
    }
    // the last S, all requested: r k-tiles behind this one.  With fewer than S in all everything has landed
    auto tail = [&](auto rc) __attribute__((always_inline)) {
        constexpr int r = decltype(rc)::value;
        if (r >= S || nk <= r) return;
        const int nx = st + 1 == S ? 0 : st + 1;
        RG_SLICE(0, true, smem + st * ST, ch1, false, 0, 0)
        if (r > 0) {
            __builtin_amdgcn_s_waitcnt(dma_waitcnt(r > 0 ? NI * (r - 1) : 0, 0));
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
        }
        RG_SLICE(1, r > 0, smem + nx * ST, ch0, false, 0, 0)
        st = nx;
    };
    static_assert(S <= 8, "tails written out below");
    tail(std::integral_constant<int, 7>{}); tail(std::integral_constant<int, 6>{});
    tail(std::integral_constant<int, 5>{}); tail(std::integral_constant<int, 4>{});
    tail(std::integral_constant<int, 3>{}); tail(std::integral_constant<int, 2>{});
    tail(std::integral_constant<int, 1>{}); tail(std::integral_constant<int, 0>{});
#undef RG_READ
#undef RG_SLICE
    __builtin_amdgcn_s_waitcnt(dma_waitcnt(0, 0));      // nothing is on its way to LDS
#undef RG_ISSUE1
    __syncthreads();
    float* const patch = reinterpret_cast<float*>(smem) + wave * (16 * MI * PATCH_LD);
    d8_half<EPI, MI, 0>(acc, patch, a, m0 + wm * MI * 16, nb, c0 / 64 + wn, lane, meta);
}

// Exact-KL epilogue of a wave's 64 rows x 64 columns: per row five numbers leave the kernel,
//   m_p = max z_p, S_p = sum exp(z_p - m_p), T = sum exp(z_p - m_p) (z_p - z_r), m_r = max z_r, S_r = sum exp(z_r - m_r)
// from which  KL(pi_p || pi_r) = T/S_p - (m_p + log S_p) + (m_r + log S_r)  once all column groups are combined.  Four
// lanes share a row as in the log-sum-exp epilogue; the reference's logits wait in registers while the policy's take the
// patch.
__device__ __forceinline__ void kl_epilogue(const floatx4_t (&acc_p)[4][4], const floatx4_t (&acc_r)[4][4], float* patch,
                                            const GemmArgs& a, int m0, int group, int lane) {
    const int row = lane >> 2, c = (lane & 3) * 8;
    float r0[4][8], r1[4][8];
    patch_put<4, 0>(acc_r, patch, lane);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        patch_get(r0[it], patch, it * 16 + row, c);
        patch_get(r1[it], patch, it * 16 + row, 32 + c);
    }
    __builtin_amdgcn_wave_barrier();
    patch_put<4, 0>(acc_p, patch, lane);
    const int nparts = a.N / 64;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        float p0[8], p1[8], sp[8], st[8], sr[8];
        patch_get(p0, patch, it * 16 + row, c);
        patch_get(p1, patch, it * 16 + row, 32 + c);
        const float mp = quad_max(max_of(p0, p1)), mr = quad_max(max_of(r0[it], r1[it]));
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const float e0 = __expf(p0[x] - mp), e1 = __expf(p1[x] - mp);
            sp[x] = e0 + e1;
            st[x] = e0 * (p0[x] - r0[it][x]) + e1 * (p1[x] - r1[it][x]);
            sr[x] = __expf(r0[it][x] - mr) + __expf(r1[it][x] - mr);
        }
        const float s_p = quad_sum(sum_of(sp)), t = quad_sum(sum_of(st)), s_r = quad_sum(sum_of(sr));
        const int m = m0 + it * 16 + row;
        if ((lane & 3) == 0 && m < a.M) {
            float* o = a.kl_part + ((int64_t)m * nparts + group) * 5;
            o[0] = mp; o[1] = s_p; o[2] = t; o[3] = mr; o[4] = s_r;
        }
    }
}

// Both LM heads of the exact KL on one tile: the reference's logits first (kept in the accumulators), then the policy's, by
// the loop above on tiles of 128 x 256 -- two sets of 64 accumulator registers per lane; taller tiles would spill.  Bound by
// the matrix cores.  2942 rows, d = 4096, V = 128256, fp16 copies: 6.2 ms (1.0 PFLOP/s); four waves on 128 x 128 tiles with bf16 weights, which
// this replaced, 8.4 ms.  N a multiple of 64: column groups past it are left out.
template <bool WF16>
__global__ __launch_bounds__(512, 1) void gemm_kl8_kernel(GemmArgs a) {
    constexpr int MI = 4, BM = 32 * MI, WGN = 4;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    int nb, mb;
    if (!tile_of(blockIdx.x, (a.M + BM - 1) / BM, a.n_blocks_n, mb, nb)) return;
    const int m0 = mb * BM;
    floatx4_t acc_r[MI][4], acc_p[MI][4];
    QkvRowMeta meta;
    dma8_loop<MG_KLFULL, WF16, MI>(a, a.A2, a.lda2, a.W2, m0, nb, wave, lane, smem, acc_r, meta);
    __syncthreads();                                   // the stages are filled again
    dma8_loop<MG_KLFULL, WF16, MI>(a, a.A, a.lda, a.W, m0, nb, wave, lane, smem, acc_p, meta);
    __syncthreads();
    const int group = nb * WGN + wn;
    if (group * 64 >= a.N) return;
    float* const patch = reinterpret_cast<float*>(smem) + wave * (64 * PATCH_LD);
    kl_epilogue(acc_p, acc_r, patch, a, m0 + wm * 64, group, lane);
}

template <int BM, int BN, int WGM, int WGN, int EPI, int BKT = 64, bool WF16 = false>
static void launch(const GemmArgs& a, int n_blocks_n, int splits, hipStream_t s) {
    constexpr size_t lds = (size_t)2 * (BM + BN) * (BKT + 8) * sizeof(f16_t);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void*)gemm_mfma_kernel<BM, BN, WGM, WGN, EPI, BKT, WF16>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr_set = true;
    }
    GemmArgs b = a;
    b.n_blocks_n = n_blocks_n;
    dim3 grid(8 * ((n_blocks_n * row_blocks(a, BM) + 7) / 8), 1, splits);
    gemm_mfma_kernel<BM, BN, WGM, WGN, EPI, BKT, WF16><<<grid, 256, lds, s>>>(b);
}

template <int EPI, int MI, int WGM, int WGN>
static void launch_ring_t(const GemmArgs& a, int cols, hipStream_t s) {
    constexpr int BM = 16 * MI * WGM, BN = 64 * WGN, lds = ring_stages(MI, WGM, WGN) * (BM + BN) * 128;
    static_assert(lds >= WGM * WGN * 16 * MI * PATCH_LD * 4, "the epilogue's patches reuse the stages");
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void*)gemm_ring_kernel<EPI, MI, WGM, WGN>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    GemmArgs b = a;
    b.n_blocks_n = cols / BN;
    gemm_ring_kernel<EPI, MI, WGM, WGN><<<8 * ((b.n_blocks_n * row_blocks(a, BM) + 7) / 8), 64 * WGM * WGN, lds, s>>>(b);
}
// The smallest tile of which the 256 CUs have at most one each (128 x 128 are, see use_ring).  Against the register-staged kernel on
// bf16 weights, us: 1B O projection at 512 / 1024 / 2048 rows 13.2 / 19.7 / 30.9 -> 12.5 / 15.6 / 22.4, down 50 / 60 / 90 -> 36 / 49 / 67,
// gate/up at 96 / 256 rows 21.0 / 25.6 -> 19.1 / 21.1; 8B O at 256 / 512 / 1024 rows 27.6 / 34.6 / 48.8 -> 21 / 30 / 40, down 92 / 112 /
// 148 -> 69 / 101 / 138.  The other tiles at these sizes: 128 x 128 at 512 rows of 1B down 63, 64 x 128 at 2048 101, 64 x 64 137.
template <int EPI>
static void launch_ring(const GemmArgs& a, int cols, hipStream_t s) {
    if (row_blocks(a, 64) * (cols / 64) <= 256) launch_ring_t<EPI, 1, 4, 1>(a, cols, s);            // 64 x 64
    else if (row_blocks(a, 64) * (cols / 128) <= 256) launch_ring_t<EPI, 1, 4, 2>(a, cols, s);      // 64 x 128
    else launch_ring_t<EPI, 2, 4, 2>(a, cols, s);                                                   // 128 x 128
}
template <bool WF16>
static void launch_kl8(const GemmArgs& a, hipStream_t s) {
    constexpr int BM = 128, stages = 5 * (BM + 256) * 64, patches = 8 * 64 * PATCH_LD * 4, lds = stages > patches ? stages : patches;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void*)gemm_kl8_kernel<WF16>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    GemmArgs b = a;
    b.n_blocks_n = (a.N + 255) / 256;
    dim3 grid(8 * ((b.n_blocks_n * ((a.M + BM - 1) / BM) + 7) / 8), 1, 1);
    gemm_kl8_kernel<WF16><<<grid, 512, lds, s>>>(b);
}
template <int EPI, bool WF16, int MI>
static void launch_dma8_t(const GemmArgs& a, int n_blocks_n, hipStream_t s) {
    constexpr int BM = 32 * MI, stages = 5 * (BM + 256) * 64, patches = 8 * 64 * PATCH_LD * 4;
    constexpr int lds = stages > patches ? stages : patches;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void*)gemm_dma8_kernel<EPI, WF16, MI>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    GemmArgs b = a;
    b.n_blocks_n = n_blocks_n;
    dim3 grid(8 * ((n_blocks_n * row_blocks(a, BM) + 7) / 8), 1, 1);
    gemm_dma8_kernel<EPI, WF16, MI><<<grid, 512, lds, s>>>(b);
}
template <int EPI, bool WF16>
static void launch_dma8(const GemmArgs& a, int n_blocks_n, int mi, hipStream_t s) {
    switch (mi) {
        case 3: launch_dma8_t<EPI, WF16, 3>(a, n_blocks_n, s); break;
        case 4: launch_dma8_t<EPI, WF16, 4>(a, n_blocks_n, s); break;
        case 5: launch_dma8_t<EPI, WF16, 5>(a, n_blocks_n, s); break;
        case 6: launch_dma8_t<EPI, WF16, 6>(a, n_blocks_n, s); break;
        case 7: launch_dma8_t<EPI, WF16, 7>(a, n_blocks_n, s); break;
        default: launch_dma8_t<EPI, WF16, 8>(a, n_blocks_n, s); break;
    }
}
// Tile height of the large-M kernel in units of 32 rows: the one whose rounds of 256 tiles (one workgroup per CU) cost
// least.  A round costs its k loop -- relative to 256 rows 0.575 .. 1 below, measured: short tiles reread W more often
// and feed fewer MFMAs per fragment -- plus an epilogue that goes with the rows (24 k-tiles' worth for the residual's
// read-modify-write, 8 for the others); the last, incomplete round runs at a higher clock: 0.7 + 0.3 x its filling.
// Over the layer shapes of the 1B, 8B and 70B models, 352 to 16384 rows, fp16 and bf16 weights, the height taken is
// within 0.3 % of the best of the six on average (6 % at worst); against 256 rows throughout: O projection of the 8B
// shape at 4928 rows 185 -> 150 us, 1B gate/up at 2240 rows 140 -> 124 us, 70B down projection at 12544 rows 5599 ->
// 5361 us.  Every height gives the same bits: a row's sums run over k in the same order.
static int big_row_blocks(int epi, const GemmArgs& a, int n_blocks_n) {
    static const float loop[9] = {0, 0, 0, 0.575f, 0.62f, 0.76f, 0.855f, 0.95f, 1.0f};
    int best = 8;
    float best_cost = 0.f;
    for (int mi = 8; mi >= 3; --mi) {
        const int64_t tiles = (int64_t)row_blocks(a, 32 * mi) * n_blocks_n;
        const float rem = (float)(tiles % 256) / 256.f;
        const float rounds = (float)(tiles / 256) + (rem > 0.f ? 0.7f + 0.3f * rem : 0.f);
        const float cost = rounds * (loop[mi] * (float)(a.K / 32) + (epi == MG_RESID ? 24.f : 8.f) * (float)mi / 8.f);
        if (mi == 8 || cost < best_cost) { best = mi; best_cost = cost; }
    }
    return best;
}
template <int EPI>
static void launch_big(const GemmArgs& a, int n_blocks_n, hipStream_t s) {
    GemmArgs b = a;
    b.k_per_split = a.K;
    const int mi = big_row_blocks(EPI, a, n_blocks_n);
    if (a.w_f16) launch_dma8<EPI, true>(b, n_blocks_n, mi, s);
    else launch_dma8<EPI, false>(b, n_blocks_n, mi, s);
}

// GEMMs below the large-M kernel on bf16 weights: 128 x 128 tiles, or where these are at most half of the CUs' number tiles of 64 rows, for
// the residual's also of 64 columns.  A workgroup's k-tile takes as long as its operands take to arrive (about 50 KB/us per
// CU: 0.65 us for 32 KB), so a GEMM with idle CUs is as fast as its tiles are small.
// Measured against 128 x 128 throughout (32 to 1024 rows, plain and pair layers): nowhere slower.  O projection, 1B to 512 rows
// 26 -> 16 us, to 1024 27 -> 20; 8B to 256 rows 45 -> 29, to 512 46 -> 35; 70B to 128 rows 84 -> 56, to 256 86 -> 68; down projections
// alike.  QKV, 1B to 640 rows 30 -> 21, 8B to 256 51 -> 37, 70B to 128 90 -> 70; gate/up, 1B to 128 rows 25 -> 18.  At 144 tiles of 128 x
// 128 twice as many would double up on some CUs.
// All of them sum a row over k in the same order: the bits do not depend on the choice.
template <int EPI>
static void launch_small(const GemmArgs& a, int n_blocks_n, hipStream_t s) {
    if (a.w_f16) { launch_ring<EPI>(a, n_blocks_n * 128, s); return; }
    if (row_blocks(a, 128) * n_blocks_n > 128) { launch<128, 128, 2, 2, EPI>(a, n_blocks_n, 1, s); return; }
    if constexpr (EPI == MG_RESID) {
        if (row_blocks(a, 64) * n_blocks_n <= 128) { launch<64, 64, 2, 2, EPI>(a, 2 * n_blocks_n, 1, s); return; }
    }
    launch<64, 128, 2, 2, EPI>(a, n_blocks_n, 1, s);
}

bool k_gemm_mfma_supported(int epi, int N, int K, int hd) {
    if (epi == MG_KLFULL) return N % 128 == 0 && K % 128 == 0 && (uint64_t)N * K * 2 < (1ull << 32);
    if (K % BK != 0) return false;
    if (epi == MG_SWIGLU) return N % 64 == 0;
    if (epi == MG_QKV) return N % 128 == 0 && (hd == 64 || hd == 128);
    return N % 128 == 0;
}

// Whether the large-M kernel takes this GEMM (a.Wrows filled in): where 128 x 128 tiles would be more than one per CU.
// Up to there the kernel of launch_small is faster (8B O projection, 352 rows: 35 us on its 64 x 128 tiles, which read bf16;
// 46 here on fp16 weights, 62 on bf16); beyond it, two of its 128 x 128 workgroups share a CU and lose (2240 rows: 119 against
// 74 and 85 us).
// The rule does not look at the weights' type, so that a set with an fp16 copy and one without give the same bits.
static bool use_big(int epi, const GemmArgs& a, int splits) {
    if (!a.big_mode || splits != 1) return false;
    const int out_cols = epi == MG_SWIGLU ? 2 * a.N : a.N;   // tile columns
    if (out_cols % 256 != 0 || a.K % 128 != 0) return false;
    if ((uint64_t)a.M * a.lda * 2 >= (1ull << 32) || (uint64_t)a.Wrows * a.Kw * 2 >= (1ull << 32)) return false;
    const int64_t tiles = (int64_t)row_blocks(a, 128) * (out_cols / 128);
    return a.big_mode >= 2 || tiles > 256;
}

// Below it: fp16 weights and at most one 128 x 128 tile per CU.
static bool use_ring(int epi, const GemmArgs& a, int splits) {
    if (splits != 1 || (epi != MG_RESID && epi != MG_SWIGLU && epi != MG_QKV && epi != MG_LSE) || use_big(epi, a, splits)) return false;
    if (a.K % 64 != 0 || a.Kw % 64 != 0 || (uint64_t)a.Wrows * a.Kw * 2 >= (1ull << 32) || (uint64_t)a.lda * 256 >= (1ull << 31)) return false;
    return row_blocks(a, 128) * ((epi == MG_SWIGLU ? 2 * a.N : a.N) / 128) <= 256;
}

int k_gemm_mfma_lse_parts(int M, int N, int K, int big_mode) {
    // column groups are as wide as a wave's share of the tile: 64 columns on the 256-column and on the 128 x 128 kernel
    (void)M; (void)K; (void)big_mode;
    return N / 64;
}

// Whether k_gemm_mfma will run this GEMM on a kernel that can read an fp16 copy of W (GemmArgs.w_f16).
bool k_gemm_mfma_reads_f16_copy(int epi, GemmArgs a, int splits) {
    if (a.M <= 0 || a.N <= 0) return false;
    if (epi == MG_KLFULL) return true;
    if (a.Kw <= 0) a.Kw = a.K;
    if (splits < 1) splits = 1;
    const int kt = a.K / BK, per = (kt + splits - 1) / splits;
    splits = (kt + per - 1) / per;
    a.Wrows = epi == MG_SWIGLU ? a.up_offset + a.N : a.N;
    return use_big(epi, a, splits) || use_ring(epi, a, splits);
}

void k_gemm_mfma(int epi, GemmArgs a, int splits, hipStream_t s) {
    if (a.M <= 0 || a.N <= 0) return;
    if (a.Kw <= 0) a.Kw = a.K;
    if (splits < 1) splits = 1;
    int kt = a.K / BK;
    int per = (kt + splits - 1) / splits;
    a.k_per_split = per * BK;
    splits = (kt + per - 1) / per;
    a.Wrows = epi == MG_SWIGLU ? a.up_offset + a.N : a.N;
    const bool big = use_big(epi, a, splits);
    if (a.w_f16 && !big && epi != MG_KLFULL && !use_ring(epi, a, splits)) return;     // callers check k_gemm_mfma_reads_f16_copy first
    switch (epi) {
        case MG_STORE_F32:
            if (big) launch_big<MG_STORE_F32>(a, a.N / 256, s);
            else launch<128, 128, 2, 2, MG_STORE_F32>(a, a.N / 128, splits, s);
            break;
        case MG_RESID:
            if (big) launch_big<MG_RESID>(a, a.N / 256, s);
            else launch_small<MG_RESID>(a, a.N / 128, s);
            break;
        case MG_SWIGLU:
            if (big) launch_big<MG_SWIGLU>(a, a.N / 128, s);
            else launch_small<MG_SWIGLU>(a, a.N / 64, s);
            break;
        case MG_LSE:
            if (big) launch_big<MG_LSE>(a, a.N / 256, s);
            else launch_small<MG_LSE>(a, a.N / 128, s);
            break;
        case MG_QKV:
            if (big) launch_big<MG_QKV>(a, a.N / 256, s);
            else launch_small<MG_QKV>(a, a.N / 128, s);
            break;
        case MG_KLFULL:
            if (a.w_f16) launch_kl8<true>(a, s);
            else launch_kl8<false>(a, s);
            break;
        default: break;
    }
}

// fp16 copy of a bf16 weight tensor, by the conversion the kernels themselves apply (so that a GEMM on the copy
// gives the same bits); n multiple of 8.  Bound by memory: four 16-byte loads of a thread are in flight before its
// first store.
__global__ __launch_bounds__(256) void bf16_to_f16_kernel(const u32x4_t* src, half8* dst, int64_t n8) {
    const int64_t i0 = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    u32x4_t v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (i0 + t * 256 < n8) v[t] = __builtin_nontemporal_load(src + i0 + t * 256);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (i0 + t * 256 < n8) dst[i0 + t * 256] = bf16x8_to_half8(v[t]);
}
void k_bf16_to_f16(const void* src, void* dst, int64_t n, hipStream_t s) {
    const int64_t n8 = n / 8;
    if (n8 <= 0) return;
    bf16_to_f16_kernel<<<(unsigned)((n8 + 1023) / 1024), 256, 0, s>>>((const u32x4_t*)src, (half8*)dst, n8);
}

void k_gemm_tile_decode(int epi, const GemmArgs& a, int splits, hipStream_t s) {
    if (epi == MG_SWIGLU) {
        if (a.w_f16) launch<128, 128, 2, 2, MG_SWIGLU, 64, true>(a, a.N / 64, 1, s);
        else launch<128, 128, 2, 2, MG_SWIGLU>(a, a.N / 64, 1, s);
    } else {
        if (a.w_f16) launch<128, 128, 2, 2, MG_STORE_F32, 64, true>(a, a.N / 128, splits, s);
        else launch<128, 128, 2, 2, MG_STORE_F32>(a, a.N / 128, splits, s);
    }
}

int k_gemm_mfma_splits_used(int K, int splits) {
    int kt = K / BK;
    if (splits < 1) splits = 1;
    int per = (kt + splits - 1) / splits;
    return (kt + per - 1) / per;
}
