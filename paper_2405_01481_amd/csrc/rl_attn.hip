// MFMA attention kernels for gfx950 (fp16 K/V, fp32 softmax and accumulation).
//
// Both kernels compute the transposed problem so that nothing has to be shuffled
// between the two contractions:
//     S^T = K * Q^T        (rows = keys,  cols = queries / query heads)
//     O^T = V^T * P^T      (rows = dims,  cols = queries / query heads)
// In the MFMA C layout a lane owns one column, i.e. one query (head): its softmax
// statistics are lane-local, and the four S^T values a lane holds per 16-key block
// are exactly the four k-values the B operand of the 16x16x16 MFMA wants from that
// lane for P^T.  K is read token-major, V dim-major (the paged pool stores V pages
// as [kv head][dim][token] for this reason), both straight from global memory in
// operand layout -- a (page, kv head) tile is one contiguous 4 KB block.
#include <algorithm>

#include "rl_common.h"
#include "rl_attn.h"

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

#define LOG2E 1.4426950408889634f

// s_waitcnt operand: at most vm vector loads outstanding
constexpr int vm_only(int vm) { return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | (15 << 8); }
// 2^x as the hardware instruction alone.  The library's exp2f wraps it in a rescaling for results in the denormal
// range (six instructions per value); softmax weights that small are zero for every purpose here.  2^-inf = 0.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// ------------------------------------------------------------------ decode: one new query per sequence
// Workgroup = (sequence b, kv head g, split).  Its NW waves take pages round-robin
// from the split's page range; query heads g*G .. g*G+G-1 are the MFMA columns 0..G-1
// (columns >= G are zero padding).  Per-wave results are merged through LDS; with more
// than one split the workgroup writes an unnormalised partial (o, m, l) per head.
// SP: queries, keys and values are fp16 pairs (value = hi + lo; the lo planes of the cache live in layer
// a.layer_lo, the lo halves of a query row after its hi halves).  Scores take the three leading terms
// k_hi q_hi + k_lo q_hi + k_hi q_lo, the probabilities are split the same way for the second contraction, and
// the output leaves as a pair: the layer then carries about 22 significant bits instead of 11.
// FU: the kernel is also the consumer of the QKV projection's split-K partial sums.  While its first page is on the
// way, the workgroup sums the partials of its own G query heads and of its kv head's new key and value (in split
// order), rotates q and k, keeps them in LDS as fp16, and -- split 0 only, after its loop -- appends k and v to the
// cache page.
// Queries are then read from LDS, and the wave that holds the page of the new token takes that token's key row and
// value column from LDS instead of from the page, so nothing depends on when the appended values become visible.
// A wave's page numbers are fetched once, one per lane (64 iterations' worth; without splits even before the position
// is known), so that a page's loads wait for no index load; with up to 8 waves per workgroup short contexts need no
// splits and no merge kernel.  32 rows, 8 kv heads, 200 keys, head_dim 64: 2 splits x 4 waves + merge 10.0 us, 8 waves
// 6.5 us; 3 rows, 100 keys, head_dim 128: 4 waves 6.2 us, 8 waves 5.7.
// ST: the cache is read as non-temporal (k_attn_decode_streams).
template <typename V, bool ST>
__device__ __forceinline__ V kv_load(const char* p) {
    if constexpr (ST) return __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
    else return *reinterpret_cast<const V*>(p);
}
template <int HD, int PT, bool SP, bool FU, int NW, bool ST>
__global__ __launch_bounds__(NW * 64, SP ? 2 : 4) void attn_decode_kernel(DecodeAttnArgs a) {
    static_assert(!(SP && FU), "the pair layers keep the separate consumer kernel");
    static_assert(PT == 16, "page tile is one 16-row MFMA block");
    constexpr int KS = HD / 32;    // k-steps of the 16x16x32 S^T MFMAs
    constexpr int DB = HD / 16;    // 16-dim blocks of O^T
    constexpr int NT = NW * 64, PS = 512 / NT;   // threads; column pairs of q, k, v per thread (FU)
    __shared__ float sm_m[NW][16], sm_l[NW][16];
    __shared__ float sm_o[NW][8][HD + 4];
    __shared__ __attribute__((aligned(16))) f16_t sm_q[FU ? 8 : 1][HD], sm_k[HD], sm_v[HD];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, g4 = lane >> 4;
    const int b = blockIdx.x, g = blockIdx.y, split = blockIdx.z;
    const int G = a.Hq / a.Hkv;
    // FU: the partial sums of this thread's (at most PS) column pairs are requested before anything else -- they
    // depend on nothing but the row -- so they travel together with the position, the page index and the first page.
    // Pair i = (head hh = i / (hd/2), j = i % (hd/2)) covers columns j and j + hd/2 of head hh; hh < G a query head,
    // hh == G the key, hh == G + 1 the value.
    constexpr int NE = 6;                           // splits requested up front (the rest, if any, later)
    constexpr int HALF = HD / 2;
    float pe0[FU ? PS : 1][NE], pe1[FU ? PS : 1][NE];
    const float* prow[PS] = {};
    if (FU) {
        const int width = (a.Hq + 2 * a.Hkv) * HD;
#pragma unroll
        for (int sl = 0; sl < PS; ++sl) {
            // no branches here (a thread without a second pair re-reads the last pair, a split past the last one
            // re-reads the last split): conditional loads would be waited for one by one
            const int i = min((int)threadIdx.x + sl * NT, (G + 2) * HALF - 1);
            const int hh = i / HALF, j = i % HALF;
            prow[sl] = a.qkv_part + (int64_t)b * width + (hh < G ? g * G + hh : hh == G ? a.Hq + g : a.Hq + a.Hkv + g) * HD + j;
#pragma unroll
            for (int sp = 0; sp < NE; ++sp) {
                const int64_t o = min(sp, a.qkv_nsplit - 1) * a.qkv_split_stride;
                pe0[sl][sp] = prow[sl][o];
                pe1[sl][sp] = prow[sl][o + HALF];
            }
        }
    }
    const int* bt = a.block_table + (int64_t)b * a.mpps;
    // page numbers of the wave's pages pbeg + wave + NW * (0 .. 63): lane l keeps the l-th.  Without splits pbeg is 0 and the
    // load goes out together with the position's; entries past the last page are never used.
    int pages = 0;
    if (gridDim.z == 1) pages = bt[min(wave + NW * lane, a.mpps - 1)];
    const int ctx = a.tok_pos[b] + 1;
    float2 cs_new[FU ? PS : 1];                      // (cos, sin) of the new token's position for this thread's pairs
    if (FU) {
#pragma unroll
        for (int sl = 0; sl < PS; ++sl)
            cs_new[sl] = a.rope[(int64_t)max(ctx - 1, 0) * HALF + min((int)threadIdx.x + sl * NT, (G + 2) * HALF - 1) % HALF];
    }
    const int npages = (ctx + PT - 1) / PT;
    const int chunk = (npages + (int)gridDim.z - 1) / (int)gridDim.z;
    const int pbeg = split * chunk, pend = min(npages, pbeg + chunk);
    if (gridDim.z != 1) pages = bt[min(pbeg + wave + NW * lane, a.mpps - 1)];
    const int p_new = (ctx - 1) / PT, st_new = (ctx - 1) % PT;   // page and slot of the new token
    const int64_t page_new = FU && ctx > 0 ? bt[p_new] : 0;
    const f16_t* const kbase = a.pool + a.geo.k_off(a.layer, 0, g, 0, 0);
    const f16_t* const vbase = a.pool + a.geo.v_off(a.layer, 0, g, 0, 0);
    const int64_t page_stride = a.geo.page_elems();
    const int64_t lo_off = SP ? (int64_t)(a.layer_lo - a.layer) * a.geo.layer_elems() : 0;   // hi plane -> lo plane
    const int qrow = (SP ? 2 : 1) * a.Hq * HD;       // elements per query / output row

    // Q^T operand: lane (head col, k-group g4) holds q[head][s*32 + g4*8 .. +8)
    half8 qf[KS], ql[SP ? KS : 1];
    if (!FU) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const f16_t* qp = a.q + (int64_t)b * qrow + (g * G + col) * HD + s * 32 + g4 * 8;
            if (col < G) qf[s] = *reinterpret_cast<const half8*>(qp);
            else qf[s] = half8{0, 0, 0, 0, 0, 0, 0, 0};
            if (SP) {
                if (col < G) ql[s] = *reinterpret_cast<const half8*>(qp + a.Hq * HD);
                else ql[s] = half8{0, 0, 0, 0, 0, 0, 0, 0};
            }
        }
    }
    const float scale = a.scale * LOG2E;       // softmax in base 2
    float m_run = -INFINITY, l_run = 0.f;
    floatx4 acc[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[d] = floatx4{0.f, 0.f, 0.f, 0.f};

    // One page per iteration; the next page's K and V tiles are requested before the current
    // page is consumed, so a wave always has a page in flight.
    half8 kf[KS], kn[KS], kfl[SP ? KS : 1], knl[SP ? KS : 1];
    half4 vf[DB], vn[DB], vfl[SP ? DB : 1], vnl[SP ? DB : 1];
    int p = pbeg + wave;
    // A page's address is the wave's, a lane adds 32 bits.  The lanes' parts count as changed with every page (nothing is executed
    // for that): as constants they are added to the 64-bit bases ahead of the loop, and at head_dim 128 the registers
    // these take, with the two pages live across the branch below, were 8 to 12 bytes of scratch per lane.
    unsigned k_lane = (col * HD + g4 * 8) * 2, v_lane = (col * PT + g4 * 4) * 2;
    auto fetch = [&](int64_t pg) __attribute__((always_inline)) {
        const char* const kp = (const char*)(kbase + pg * page_stride);
        const char* const vp = (const char*)(vbase + pg * page_stride);
        asm("" : "+v"(k_lane), "+v"(v_lane) : "s"(pg));
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            kn[s] = kv_load<half8, ST>(kp + k_lane + s * 64);
            if (SP) knl[s] = kv_load<half8, ST>(kp + lo_off * 2 + k_lane + s * 64);
        }
#pragma unroll
        for (int d = 0; d < DB; ++d) {
            vn[d] = kv_load<half4, ST>(vp + v_lane + d * 32 * PT);
            if (SP) vnl[d] = kv_load<half4, ST>(vp + lo_off * 2 + v_lane + d * 32 * PT);
        }
    };
    if (p < pend) fetch(__builtin_amdgcn_readlane(pages, 0));
    if (FU) {
        if (ctx > 0) {   // uniform over the workgroup; a parked row has no keys and no query
#pragma unroll
            for (int sl = 0; sl < PS; ++sl) {
                const int i = threadIdx.x + sl * NT;
                if (i < (G + 2) * HALF) {
                    const int hh = i / HALF, j = i % HALF;
                    const float2 cs = cs_new[sl];
                    float x0 = 0.f, x1 = 0.f;       // summed in split order
#pragma unroll
                    for (int sp = 0; sp < NE; ++sp) {
                        x0 = sp < a.qkv_nsplit ? x0 + pe0[sl][sp] : x0;
                        x1 = sp < a.qkv_nsplit ? x1 + pe1[sl][sp] : x1;
                    }
                    for (int sp = NE; sp < a.qkv_nsplit; ++sp) {
                        x0 += prow[sl][sp * a.qkv_split_stride];
                        x1 += prow[sl][sp * a.qkv_split_stride + HALF];
                    }
                    if (hh <= G) {
                        const float r0 = x0 * cs.x - x1 * cs.y, r1 = x1 * cs.x + x0 * cs.y;
                        x0 = r0; x1 = r1;
                    }
                    const f16_t h0 = (f16_t)x0, h1 = (f16_t)x1;
                    if (hh < G) {
                        sm_q[hh][j] = h0; sm_q[hh][j + HALF] = h1;
                    } else if (hh == G) {
                        sm_k[j] = h0; sm_k[j + HALF] = h1;
                    } else {
                        sm_v[j] = h0; sm_v[j + HALF] = h1;
                    }
                }
            }
            __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if (col < G && ctx > 0) qf[s] = *reinterpret_cast<const half8*>(&sm_q[col][s * 32 + g4 * 8]);
            else qf[s] = half8{0, 0, 0, 0, 0, 0, 0, 0};
        }
    }
    int it = 0;                                     // the wave's pages so far
    for (; p < pend; p += NW) {
#pragma unroll
        for (int s = 0; s < KS; ++s) { kf[s] = kn[s]; if (SP) kfl[s] = knl[s]; }
#pragma unroll
        for (int d = 0; d < DB; ++d) { vf[d] = vn[d]; if (SP) vfl[d] = vnl[d]; }
        if (FU && p == p_new) {   // the new token's key row and value column come from LDS
            if (col == st_new) {
#pragma unroll
                for (int s = 0; s < KS; ++s) kf[s] = *reinterpret_cast<const half8*>(&sm_k[s * 32 + g4 * 8]);
            }
            if (g4 == (st_new >> 2)) {
#pragma unroll
                for (int d = 0; d < DB; ++d) {
                    const f16_t v = sm_v[d * 16 + col];
#pragma unroll
                    for (int i = 0; i < 4; ++i) vf[d][i] = i == (st_new & 3) ? v : vf[d][i];
                }
            }
        }
        if (p + NW < pend) {
            // a wave's last page asks for nothing: a re-read of that page, unused, was still waited for at the end and
            // read twice by waves of few pages (8 rows at 200 tokens 8.4 -> 7.5 us, 128 at 592 62 -> 59.5).  The pair kernel takes
            // 208 VGPRs for it, two waves per SIMD: with the re-read three (156), 128 rows 103 instead of 105.5, 32 at 1600
            // 80.6 and 80.9, head_dim 64, 64 at 280, 16.7 and 16.4
            ++it;
            if ((it & 63) == 0) pages = bt[min(p + NW + NW * lane, a.mpps - 1)];
            fetch(__builtin_amdgcn_readlane(pages, it & 63));
        }
        floatx4 s0 = {0.f, 0.f, 0.f, 0.f};
        if (SP) {   // the two small terms first, the leading one last
#pragma unroll
            for (int s = 0; s < KS; ++s) s0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(kfl[s], qf[s], s0, 0, 0, 0);
#pragma unroll
            for (int s = 0; s < KS; ++s) s0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[s], ql[s], s0, 0, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) s0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[s], qf[s], s0, 0, 0, 0);
        // lane holds keys p*16 + g4*4 + i of head `col`
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int t0 = p * PT + g4 * 4 + i;
            s0[i] = (t0 < ctx) ? s0[i] * scale : -INFINITY;
            mx = fmaxf(mx, s0[i]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, RL_WAVE));
        mx = fmaxf(mx, __shfl_xor(mx, 32, RL_WAVE));
        const float m_new = fmaxf(m_run, mx);       // finite: the first key of page p is always valid
        const float alpha = fast_exp2(m_run - m_new);
        half4 pf0, pl0;
        float ps = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float e0 = fast_exp2(s0[i] - m_new);
            ps += e0;
            pf0[i] = (f16_t)e0;
            if (SP) pl0[i] = (f16_t)(e0 - (float)pf0[i]);
        }
        l_run = l_run * alpha + ps;
        m_run = m_new;
#pragma unroll
        for (int d = 0; d < DB; ++d) {
            acc[d] *= alpha;
            if (SP) {
                acc[d] = __builtin_amdgcn_mfma_f32_16x16x16f16(vfl[d], pf0, acc[d], 0, 0, 0);
                acc[d] = __builtin_amdgcn_mfma_f32_16x16x16f16(vf[d], pl0, acc[d], 0, 0, 0);
            }
            acc[d] = __builtin_amdgcn_mfma_f32_16x16x16f16(vf[d], pf0, acc[d], 0, 0, 0);
        }
    }
    // FU: the new token's key and value go to the cache only now -- stores count towards the same in-order
    // completion counter as loads, so stores issued before the loop would hold back every page load behind them
    if (FU && split == 0 && ctx > 0) {
        for (int i = threadIdx.x; i < HD; i += NT) {
            a.pool_w[a.geo.k_off(a.layer, page_new, g, st_new, i)] = sm_k[i];
            a.pool_w[a.geo.v_off(a.layer, page_new, g, st_new, i)] = sm_v[i];
        }
    }
    // wave totals: l over the four key groups
    l_run += __shfl_xor(l_run, 16, RL_WAVE);
    l_run += __shfl_xor(l_run, 32, RL_WAVE);
    if (col < G) {
        if (g4 == 0) { sm_m[wave][col] = m_run; sm_l[wave][col] = l_run; }
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) sm_o[wave][col][d * 16 + g4 * 4 + i] = acc[d][i];
    }
    __syncthreads();
    const int nsplit = gridDim.z;
    for (int idx = threadIdx.x; idx < G * HD; idx += NT) {
        const int hh = idx / HD, d = idx % HD;
        float mt = sm_m[0][hh];
#pragma unroll
        for (int w = 1; w < NW; ++w) mt = fmaxf(mt, sm_m[w][hh]);
        float o = 0.f, l = 0.f;
        if (mt > -INFINITY) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                float wt = fast_exp2(sm_m[w][hh] - mt);
                o += wt * sm_o[w][hh][d];
                l += wt * sm_l[w][hh];
            }
        }
        const int64_t head = (int64_t)b * a.Hq + g * G + hh;
        if (nsplit == 1) {
            const float r = l > 0.f ? o / l : 0.f;                          // parked row (position -1): no keys, zeros
            f16_t* op = a.out + (int64_t)b * qrow + (g * G + hh) * HD + d;
            const f16_t hi = (f16_t)r;
            op[0] = hi;
            if (SP) op[a.Hq * HD] = (f16_t)(r - (float)hi);
        } else {
            a.part_o[(head * nsplit + split) * HD + d] = o;
            if (d == 0) {
                a.part_ml[(head * nsplit + split) * 2 + 0] = mt;
                a.part_ml[(head * nsplit + split) * 2 + 1] = l;
            }
        }
    }
}

// Merge of split partials: out = sum_s w_s o_s / sum_s w_s l_s, w_s = 2^(m_s - max m).
// split: the output row holds fp16 pairs, [Hq heads of hi | Hq heads of lo].
template <int HD>
__global__ __launch_bounds__(HD) void attn_merge_kernel(const float* part_o, const float* part_ml, f16_t* out,
                                                        int nsplit, int Hq, int split) {
    const int64_t head = blockIdx.x;
    const int d = threadIdx.x;
    float mt = -INFINITY;
    for (int s = 0; s < nsplit; ++s) mt = fmaxf(mt, part_ml[(head * nsplit + s) * 2]);
    float o = 0.f, l = 0.f;
    for (int s = 0; s < nsplit; ++s) {
        float m = part_ml[(head * nsplit + s) * 2];
        if (m == -INFINITY) continue;
        float wt = fast_exp2(m - mt);
        o += wt * part_o[(head * nsplit + s) * HD + d];
        l += wt * part_ml[(head * nsplit + s) * 2 + 1];
    }
    const float r = l > 0.f ? o / l : 0.f;
    const f16_t hi = (f16_t)r;
    f16_t* op = out + (head / Hq) * (int64_t)((split ? 2 : 1) * Hq * HD) + (head % Hq) * HD + d;
    op[0] = hi;
    if (split) op[Hq * HD] = (f16_t)(r - (float)hi);
}

// The consumer form of the kernel gives its threads at most 512 (column, column + hd/2) pairs of the group's G query
// heads, key and value, and keeps the queries of at most 8 heads in LDS.
bool k_attn_decode_consumes_qkv(int Hq, int Hkv, int hd) {
    const int G = Hq / Hkv;
    return (hd == 64 || hd == 128) && G <= 8 && (G + 2) * (hd / 2) <= 512;
}

// From the context's limits: a workgroup draws up to 38 KB/us, four waves of it as much as eight, so 256 workgroups are
// enough to read the cache at memory speed, and a split costs a merge kernel and the query's preparation once more.  Hence
// only as many splits as it takes to reach 256 workgroups, rounded up (25 rows of 8 kv heads: 2 splits, 400 workgroups), of
// at least 16 pages of the longest sequence each; eight waves where fewer than 512
// workgroups leave room (short contexts: 32 rows x 200 keys 7.6 -> 6.5 us; 64 rows x 300 keys at head_dim 128 19.4 ->
// 18.9, non-temporal 18.1 -> 18.6).  8 kv heads, head_dim 128, merge included, splits 1 / 2 / 4 / 8: 32 rows x 1600 keys 38 / 41 / 43 / 50 us,
// 16 x 4000 73 / 49 / 48 / 52, 8 x 1600 23.5 / 18.1 / 16.4 / 18.7, 1 x 4000 46 / 29 / 19.4 / 15.9, 8 x 300 8.7 / 10.3 / 9.8 / 11.8.
void k_attn_decode_plan(int max_batch, int Hkv, int mpps, int max_splits, int* waves, int* nsplit) {
    const int wgs = max_batch * Hkv;
    *waves = wgs < 512 ? 8 : 4;
    *nsplit = std::max(1, std::min(std::min((256 + wgs - 1) / wgs, mpps / 16), max_splits));
}

template <int HD, bool SP, bool FU, bool ST>
static void launch_attn_decode(const DecodeAttnArgs& a, int B, int waves, int nsplit, hipStream_t s) {
    const dim3 grid(B, a.Hkv, nsplit);
    if (waves == 8) attn_decode_kernel<HD, 16, SP, FU, 8, ST><<<grid, 512, 0, s>>>(a);
    else attn_decode_kernel<HD, 16, SP, FU, 4, ST><<<grid, 256, 0, s>>>(a);
}
template <int HD, bool ST>
static void launch_attn_decode_hd(const DecodeAttnArgs& a, int B, int waves, int nsplit, hipStream_t s) {
    if (a.split) launch_attn_decode<HD, true, false, ST>(a, B, waves, nsplit, s);
    else if (a.qkv_part) launch_attn_decode<HD, false, true, ST>(a, B, waves, nsplit, s);
    else launch_attn_decode<HD, false, false, ST>(a, B, waves, nsplit, s);
    if (nsplit > 1)
        attn_merge_kernel<HD><<<B * a.Hq, HD, 0, s>>>(a.part_o, a.part_ml, a.out, nsplit, a.Hq, a.split);
}

// Non-temporal where the keys and values of one layer would be far more than the L2s hold if all rows had the longest context: that
// of the run, never the context's limit, which may be many times longer.  Whole generations of 64 tokens, per launch: 8B
// width 139 MB (128 rows, 264 keys) 2.4 us shorter, 113 MB (32, 864) 1.5, 109 (64, 414) 1.0, 1B 139 (64, 1064) 1.4, 87 (64, 664) 0.5; 70B 95
// MB, rows of 100 to 300 keys 1.2 us longer, of 300 2.3 shorter; 61 and 64 MB 0.5 shorter; small ones are longer: 1B 44 MB 0.3, 17
// MB 0.4, 8B 9 MB (8, 264) 0.9 of 8.
static const int64_t kStreamBytes = (int64_t)100 << 20;
bool k_attn_decode_streams(int B, int max_ctx, int Hkv, int hd, int pair) {
    return (int64_t)B * max_ctx * Hkv * hd * (pair ? 8 : 4) > kStreamBytes;
}

void k_attn_decode(const DecodeAttnArgs& a, int B, int waves, int nsplit, hipStream_t s) {
    if (B <= 0) return;
    if (a.qkv_part && (a.split || !k_attn_decode_consumes_qkv(a.Hq, a.Hkv, a.geo.hd))) return;   // callers check first
    if (a.geo.hd == 128) {
        if (a.stream) launch_attn_decode_hd<128, true>(a, B, waves, nsplit, s);
        else launch_attn_decode_hd<128, false>(a, B, waves, nsplit, s);
    } else {
        if (a.stream) launch_attn_decode_hd<64, true>(a, B, waves, nsplit, s);
        else launch_attn_decode_hd<64, false>(a, B, waves, nsplit, s);
    }
}

// ------------------------------------------------------------------ prefill / scoring: causal attention over packed sequences
// Workgroup = (NQ consecutive 32-query blocks of one sequence, HW query heads of kv head g), four waves: wave w < HW x NQ
// handles head h0 + w % HW of query block w / HW (a wave left over only helps staging), so the waves of a workgroup need the
// SAME keys and values.  Keys are walked in steps of TS tiles of 32.  Per tile K (32 keys x hd) and V^T (hd dims x 32
// keys, one contiguous piece of the value buffer) are staged ONCE per workgroup into LDS by global -> LDS loads of whole
// lines (step ks + NS - 1 is requested right after the barrier that opens step ks), and every wave reads its operand
// fragments from there.
// What bounds it is a wave's own chain of scores -> maximum -> exponentials -> products, and for short sequences what a
// workgroup costs before and after its loop.  Hence steps of 64 keys (two independent chains of score MFMAs; one maximum,
// one cross-lane exchange, one rescaling per 64 keys), V^T fragments read before the softmax, two independent workgroups
// per CU, one's start and end behind the other's loop, and an output that leaves as whole lines.  Where
// kv heads (times two for groups of more than four) are a multiple of eight, a kv head's workgroups stay on one XCD (ids go
// round-robin to the eight, each with its own L2).
// 16 x 1024 tokens of the 8B shape 257 -> 205 us (0.67 PFLOP/s; MFMAs busy a third of the time), 5 sequences of 1500 to 4096
// tokens of the 70B shape 1065 -> 690 us (1.0 PFLOP/s), 8 of 70 to 512 of the 1B shape 21.9 -> 13.7, against steps of 32 keys
// with a wait for the next tile in each and 16-byte output stores.  Eight waves per workgroup: 239, 747, 24.2; steps of 32
// keys, three workgroups per CU: 218, 725, 16.8.
// 16-byte chunks are XOR-swizzled on the source side of the loads (K: chunk ^ row%16 for 256-byte rows, chunk ^ (row/2)%8
// for 128-byte rows; V^T: chunk ^ (row/4)%4) so that the fragment reads spread over the banks.  The loads are issued from
// inline assembly and waited for by count (the compiler would otherwise make each of them complete at the next barrier).
//   S^T (32 keys x 32 queries) by 32x32x16 MFMAs with K rows as A and Q^T as B; base-2 online softmax per
//   query (a lane owns one query column); O^T += V^T P^T where the lane's own S^T registers, rounded to
//   fp16, are the B operand.
typedef float floatx16 __attribute__((ext_vector_type(16)));

static constexpr int ap_tiles(bool SP) { return SP ? 1 : 2; }                      // 32-key tiles of a step
static constexpr int AP_NW = 4;                                                    // waves of a workgroup
static constexpr int AP_NS = 2;                                                    // stages
// query heads of a group of G that a workgroup takes (the group is cut in two where it has more than four)
__host__ __device__ constexpr int ap_heads(int G) { return G <= AP_NW ? G : (G + 1) / 2; }
static constexpr int ap_stage_bytes(int HD, bool SP) { return ap_tiles(SP) * (SP ? 4 : 2) * 32 * HD * 2; }

// SP: q, k, v are fp16 pairs (value = hi + lo; rows of q, k and the output are [hi heads | lo heads], the lo plane
// of V^T follows the hi plane).  A tile then has four parts (K hi, V^T hi, K lo, V^T lo), the scores take the
// three leading terms k_hi q_hi + k_lo q_hi + k_hi q_lo, and the probabilities are split the same way for the
// second contraction: three MFMAs where the plain kernel has one.
template <int HD, bool SP>
__global__ __launch_bounds__(AP_NW * 64, HD == 64 ? 3 : 2) void attn_prefill_kernel(PrefillAttnArgs a) {
    constexpr int KSTEPS = HD / 16, DB = HD / 32, TS = ap_tiles(SP), NS = AP_NS;
    constexpr int KT = 32 * HD * 2;              // bytes of a K tile; a V^T tile is as large
    constexpr int NT = SP ? 4 : 2;               // parts of a tile: K, V^T (hi), then K, V^T (lo)
    constexpr int STG = ap_stage_bytes(HD, SP);
    constexpr int NIT = KT / 1024;               // 1 KB load instructions per part
    constexpr int PER = TS * NT * NIT / AP_NW;       // of a step, per wave
    constexpr int KCH = HD / 8;                  // 16-byte chunks per K row
    constexpr int KRPI = 64 / KCH;               // K rows per load instruction
    extern __shared__ __attribute__((aligned(1024))) char smem[];   // [NS stages][STG]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, g2 = lane >> 5;
    const int G = a.Hq / a.Hkv, HW = ap_heads(G), NQ = AP_NW / HW, parts = (G + HW - 1) / HW;
    const int pg = blockIdx.x % (a.Hkv * parts), g = pg % a.Hkv, h0 = pg / a.Hkv * HW;   // kv head; first head of its group
    const int4 blk = a.blocks[blockIdx.x / (a.Hkv * parts)];  // (row start, length, group of NQ query blocks, -)
    const int start = blk.x, len = blk.y;
    const int h = g * G + min(h0 + wave % HW, G - 1);
    const int nqb = (len + 31) / 32;
    const int qb = wave < HW * NQ && h0 + wave % HW < G ? blk.z * NQ + wave / HW : nqb;    // this wave's query block; nqb and later: none
    const int last = min((blk.z + 1) * NQ, nqb) - 1;               // the workgroup's last key block
    const int qi = qb * 32 + col;                   // this lane's query (position in the sequence)
    const int qrow = start + min(qi, len - 1);
    const int kvw = (SP ? 2 : 1) * a.Hkv * HD;      // elements per K row
    const int qw = (SP ? 2 : 1) * a.Hq * HD;        // elements per query / output row

    // Staging: load n of a wave moves 1 KB of part (wave + 4 n) / NIT of the step.
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem + wave * 1024;
    const int64_t v_plane = (int64_t)a.vt_cap * HD;                       // V of one head: tiles of [HD dims][32 tokens]
    unsigned s_off[PER];
    const char* s_base[PER];
    int s_blk[PER];                                                       // bytes from one key block to the next
#pragma unroll
    for (int n = 0; n < PER; ++n) {
        const int t = (wave + AP_NW * n) / NIT % NT, ii = (wave + AP_NW * n) % NIT;
        if ((t & 1) == 0) {                      // K: KRPI rows of KCH chunks
            const int r = ii * KRPI + lane / KCH, pc = lane % KCH;
            const int lc = pc ^ (HD == 128 ? (r & 15) : ((r >> 1) & 7));
            // tile row r holds key rho(r): the middle two 4-row groups of every 16 are swapped, so that a lane's S^T
            // registers 8kk .. 8kk+7 are eight CONSECUTIVE keys (one 16-byte V^T chunk)
            const int key = (r & ~12) | ((r & 4) << 1) | ((r & 8) >> 1);
            s_off[n] = (unsigned)(key * kvw + lc * 8) * 2u;
            s_base[n] = reinterpret_cast<const char*>(a.k + (int64_t)start * kvw + (g + (t >> 1) * a.Hkv) * HD);
            s_blk[n] = 32 * kvw * 2;
        } else {                                 // V^T: 16 dims of 4 chunks (32 keys)
            const int r = ii * 16 + (lane >> 2), pc = lane & 3;
            const int lc = pc ^ ((r >> 2) & 3);
            s_off[n] = (unsigned)(r * 32 + lc * 8) * 2u;
            s_base[n] = reinterpret_cast<const char*>(a.vT + (g + (t >> 1) * a.Hkv) * v_plane + (int64_t)start * HD);
            s_blk[n] = 32 * HD * 2;
        }
    }
    // (blocks past the last one: that one again, its keys masked)
#define AP_STAGE(stage, ks)                                                                                      \
    _Pragma("unroll") for (int n_ = 0; n_ < PER; ++n_) {                                                         \
        const int kb_ = min((ks) * TS + (wave + AP_NW * n_) / (NIT * NT), last);                                     \
        const unsigned sa_ = lds_base + (stage) * STG + n_ * (AP_NW * 1024);                                               \
        const char* g_ = s_base[n_] + (int64_t)kb_ * s_blk[n_];                                                  \
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"                             \
                     :: "s"(sa_), "v"(s_off[n_]), "s"(g_) : "memory");                                           \
    }

    half8 qf[KSTEPS], ql[SP ? KSTEPS : 1];
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) {
        const f16_t* qp = a.q + (int64_t)qrow * qw + h * HD + s * 16 + g2 * 8;
        qf[s] = *reinterpret_cast<const half8*>(qp);
        if (SP) ql[s] = *reinterpret_cast<const half8*>(qp + a.Hq * HD);
    }
    floatx16 o[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float scale = a.scale * LOG2E;
    // this lane's fragment addresses inside a tile
    const int ksw = HD == 128 ? (col & 15) : ((col >> 1) & 7);
    const int k_row = col * (HD * 2);                       // K row `col`
    const int v_row = col * 64, vsw = (col >> 2) & 3;       // V^T rows d*32 + col

#pragma unroll
    for (int t = 0; t < NS - 1; ++t) AP_STAGE(t, t)
    int st = 0, fill = NS - 1;
    for (int ks = 0; ks * TS <= last; ++ks) {
        // the tiles of step ks have landed (this wave's part: the NS - 2 younger steps may be on their way); after the
        // barrier every wave's part has, and every wave is done with the stage of step ks - 1
        __builtin_amdgcn_s_waitcnt(vm_only((NS - 2) * PER));
        __syncthreads();
        AP_STAGE(fill, ks + NS - 1)                         // the last trips' are not used: the counts hold
        const char* const kt = smem + st * STG;
        st = st + 1 == NS ? 0 : st + 1;
        fill = fill + 1 == NS ? 0 : fill + 1;
        if (ks * TS > qb || qb >= nqb) continue;            // wave-uniform: behind its query block, or none
        // S^T = K Q^T
        floatx16 stt[TS];
#pragma unroll
        for (int t = 0; t < TS; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) stt[t][r] = 0.f;
        if (SP) {   // the two small terms first, the leading one last
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s)
#pragma unroll
                for (int t = 0; t < TS; ++t) {
                    const char* kr = kt + t * NT * KT + k_row + (((s * 2 + g2) ^ ksw) * 16);
                    const half8 kl = *reinterpret_cast<const half8*>(kr + 2 * KT);
                    const half8 kf = *reinterpret_cast<const half8*>(kr);
                    stt[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kl, qf[s], stt[t], 0, 0, 0);
                    stt[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf, ql[SP ? s : 0], stt[t], 0, 0, 0);
                }
        }
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s)
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                const half8 kf = *reinterpret_cast<const half8*>(kt + t * NT * KT + k_row + (((s * 2 + g2) ^ ksw) * 16));
                stt[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf, qf[s], stt[t], 0, 0, 0);
            }
        // V^T fragments: the lane needs keys kk*16 + 8*g2 .. +8 of dim d*32 + col, one 16-byte chunk.  (Pairs: read when used)
        half8 vf[SP ? 1 : TS][SP ? 1 : DB][2];
        if constexpr (!SP) {
#pragma unroll
            for (int t = 0; t < TS; ++t)
#pragma unroll
                for (int d = 0; d < DB; ++d)
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
                        vf[t][d][kk] = *reinterpret_cast<const half8*>(kt + (t * NT + 1) * KT + d * 2048 + v_row + ((kk * 2 + g2) ^ vsw) * 16);
        }
        // register r of this lane is tile row 8*(r/4) + 4*g2 + r%4, which holds key kb*32 + 16*(r/8) + 8*g2 + r%8.
        // Only the diagonal step needs the causal mask; the running maximum is kept in raw (unscaled) units,
        // so that exp2(scale * (s - m)) is one fused multiply-add and one exp2 per element.
        if ((ks + 1) * TS > qb) {
#pragma unroll
            for (int t = 0; t < TS; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = (ks * TS + t) * 32 + 16 * (r >> 3) + 8 * g2 + (r & 7);
                    if (key > qi) stt[t][r] = -INFINITY;
                }
            // A tile wholly behind the query block has no weight, whatever its values are: 0 times an infinity is not 0
            if constexpr (!SP) {
#pragma unroll
                for (int t = 1; t < TS; ++t)
                    if (ks * TS + t > qb) {
#pragma unroll
                        for (int d = 0; d < DB; ++d) vf[t][d][0] = vf[t][d][1] = half8{};
                    }
            }
        }
        float mx = stt[0][0];
#pragma unroll
        for (int t = 0; t < TS; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, stt[t][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, RL_WAVE));
        const float m_new = fmaxf(m_run, mx);        // finite: key ks*TS*32 <= qi in every step taken
        const float alpha = fast_exp2((m_run - m_new) * scale);
        const float nms = -m_new * scale;
        half8 pf[TS][2], pl[SP ? TS : 1][2];
        float ps[2] = {0.f, 0.f};
#pragma unroll
        for (int t = 0; t < TS; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float e = fast_exp2(fmaf(stt[t][r], scale, nms));
                ps[r & 1] += e;
                const f16_t eh = (f16_t)e;
                pf[t][r >> 3][r & 7] = eh;
                if (SP) pl[SP ? t : 0][r >> 3][r & 7] = (f16_t)(e - (float)eh);
            }
        l_run = l_run * alpha + (ps[0] + ps[1]);
        m_run = m_new;
        // the accumulators are rescaled only when some query's maximum moved (rare after the first blocks)
        if (__any(alpha != 1.0f)) {
#pragma unroll
            for (int d = 0; d < DB; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
        }
        // O^T += V^T P^T
#pragma unroll
        for (int t = 0; t < TS; ++t)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int d = 0; d < DB; ++d) {
                    if constexpr (SP) {
                        const char* vr = kt + (t * NT + 1) * KT + d * 2048 + v_row + ((kk * 2 + g2) ^ vsw) * 16;
                        const half8 vh = *reinterpret_cast<const half8*>(vr), vl = *reinterpret_cast<const half8*>(vr + 2 * KT);
                        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl, pf[t][kk], o[d], 0, 0, 0);
                        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, pl[t][kk], o[d], 0, 0, 0);
                        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, pf[t][kk], o[d], 0, 0, 0);
                    } else {
                        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[t][d][kk], pf[t][kk], o[d], 0, 0, 0);
                    }
                }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // nothing may land in LDS after the workgroup has ended
#undef AP_STAGE
    __syncthreads();                                   // every wave is done with the stages
    // The output leaves as whole rows of a head: through this wave's own LDS patch ([32 queries][hd], rows padded by 16
    // bytes), 16 bytes per lane.  (Straight from the registers it is 16 bytes of a row per store: eight times the requests.)
    // The writes into the patch are the kernel's only LDS bank conflicts: counted 96 cycles per wave, at any length.
    l_run += __shfl_xor(l_run, 32, RL_WAVE);
    const float inv = qb < nqb ? 1.0f / l_run : 0.f;
    constexpr int LD = HD + 8, RPI = 512 / HD;         // rows per store instruction
    static_assert(AP_NW * 32 * LD * 2 <= NS * STG, "the patches reuse the stages");
    f16_t* const patch = reinterpret_cast<f16_t*>(smem) + wave * 32 * LD;
#pragma unroll
    for (int pl = 0; pl < (SP ? 2 : 1); ++pl) {        // plane 1: what the rounding left over
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                half4 w4;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float r = o[d][4 * j + i] * inv;
                    const f16_t hi = (f16_t)r;
                    w4[i] = pl == 0 ? hi : (f16_t)(r - (float)hi);
                }
                *reinterpret_cast<half4*>(patch + col * LD + d * 32 + 8 * j + 4 * g2) = w4;
            }
        __builtin_amdgcn_wave_barrier();               // LDS accesses of a wave complete in order
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int r = it * RPI + lane / (64 / RPI), c = lane % (64 / RPI) * 8;
            const half8 v = *reinterpret_cast<const half8*>(patch + r * LD + c);
            if (qb * 32 + r < len)
                *reinterpret_cast<half8*>(a.out + (int64_t)(start + qb * 32 + r) * qw + (pl * a.Hq + h) * HD + c) = v;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// 32-query blocks per workgroup: as many as give its four waves work, one per query head and query block.
int k_attn_prefill_blocks(int Hq, int Hkv) { return AP_NW / ap_heads(Hq / Hkv); }

template <int HD, bool SP>
static void launch_prefill(const PrefillAttnArgs& a, int nblocks, hipStream_t s) {
    constexpr int lds = AP_NS * ap_stage_bytes(HD, SP);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void*)attn_prefill_kernel<HD, SP>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    const int G = a.Hq / a.Hkv, HW = ap_heads(G);
    attn_prefill_kernel<HD, SP><<<a.Hkv * ((G + HW - 1) / HW) * nblocks, AP_NW * 64, lds, s>>>(a);
}

void k_attn_prefill(const PrefillAttnArgs& a, int nblocks, hipStream_t s) {
    if (nblocks <= 0) return;
    if (a.hd == 128) {
        if (a.split) launch_prefill<128, true>(a, nblocks, s);
        else launch_prefill<128, false>(a, nblocks, s);
    } else {
        if (a.split) launch_prefill<64, true>(a, nblocks, s);
        else launch_prefill<64, false>(a, nblocks, s);
    }
}
