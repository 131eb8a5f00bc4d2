// Weight-streaming GEMMs of a decode step of at most 128 rows:  C[M,N] = A[M,K] (fp16) * W[N,K]^T (bf16 or fp16 copy).
//
// Bound by reading W once.  What a plain read of these matrices reaches here, launch included, sets the floor: 12.6 MB
// in 3.8 us, 33.5 MB in 6.5, 117 MB in 20, 235 MB in 38 (3.3, 5.2, 5.8, 6.2 TB/s).  A comes on top, from L2: every workgroup
// reads its rows once, and they take their part of the about 64 KB that a CU has on its way at once (gate/up of the 8B shape,
// a plain layer: 38, 37.5, 39, 48.6 us at 3, 32, 64, 128 rows).  Three things decide how close a GEMM comes, all measured:
//   * how rows are read.  64-byte pieces of 16 rows (operands straight into MFMA layout) reach 60 - 80 % of the plain
//     read on the short matrices, 256-byte pieces 95 %.  So operands go global -> LDS in k-tiles of 128 (a 1 KB
//     request = 4 rows x 256 B), 16-byte chunks XOR-swizzled with the row on the source side, so that the fragment
//     reads (16 rows x 64 B, one 16-byte read per lane) meet no bank conflict.
//   * where the workgroups stand in k.  Rows whose length is a power of two put the same k of all rows on the same
//     memory channels, and workgroups start together: workgroup b therefore starts at k-tile b (mod its range) and
//     wraps.  235 MB gate/up 47.5 -> 39.3 us, 1B gate/up 16.3 -> 13.7, 70B O projection 34.7 -> 28.4.  Where rows are
//     not a power of two long it only costs (70B down projection 88 -> 98 us), and where a split has fewer than 16 k-tiles the
//     splits stand apart anyway (1B down, 8 splits of 8: 9.4 us rotated, 8.9 not): not done there.
//   * the shape of the work.  One workgroup per CU with no remainder: the tile is CT x 16 columns, CT = 1 .. 8, and K is
//     split over Z workgroups whose partial sums the consumer reduces (stream_plan).
// Eight waves: four along the k-tile (32 k each), two along the columns, so that every W fragment is read, and on bf16
// weights converted, by one wave only; each wave holds all MT x 16 rows.  The four partial accumulators meet in LDS after
// the loop, in wave order.  Three stages (above 64 rows two of A: LDS is full; four of small tiles, gs_nw), one barrier per
// k-tile; the loads are issued from inline assembly (the compiler would wait for them at every barrier) and counted by hand: two
// k-tiles of W are in flight while one is consumed.
// Against a kernel on 128 x 128 tiles with k-tiles of 64 (which it replaced), per launch: 8B at 3 rows QKV 12.8 -> 10.4 us, O 9.8
// -> 8, gate/up 52 -> 40, down 23 -> 21, LM head 222 -> 177; at 128 rows 18.1 -> 17.3, 15.3 -> 14, 58 -> 54.5, 33.5 -> 33.5, 227 ->
// 230; 1B at 32 rows 8.2 -> 5.3, 7.0 -> 4.2, 21.7 -> 13.9, 11.3 -> 9.3; 70B (bf16) at 64 rows 38 -> 33, 38 -> 29.5, 171 -> 170, 84 -> 82.
#include <type_traits>

#include "rl_common.h"
#include "rl_gemm.h"
#include "rl_gemm_dev.h"

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef f16_t half4 __attribute__((ext_vector_type(4)));

static constexpr int GS_KT = 128, GS_RB = 256, GS_WK = 4;                 // k-tile, its bytes per row, waves along k
// Stages of W and of A.  Tiles of up to 6 x 16 rows of A and W together ask for three k-tiles at a time: a split of the 1B shape has
// four in all (O at 32 rows 4.5 -> 4.4 us, down 8.7 -> 8.5; 8B O 8.3 -> 8.0; QKV 5.3 -> 5.4).  More in flight is nothing to larger tiles.
static constexpr int gs_nw(int MT, int CT) { return MT < 8 && MT + CT <= 6 ? 4 : 3; }
static constexpr int gs_na(int MT, int CT) { return MT == 8 ? 2 : gs_nw(MT, CT); }
static constexpr int gs_lds(int MT, int CT) { return (gs_nw(MT, CT) * CT + gs_na(MT, CT) * MT) * 16 * GS_RB; }

// Row of W behind row rr of the 16-row tile t.  MG_SWIGLU: 8 gate rows and the 8 up rows of the same columns.
template <int EPI>
__device__ __forceinline__ int stream_w_row(int t, int rr, const GemmArgs& a) {
    if (EPI == MG_SWIGLU) return (rr < 8 ? 0 : a.up_offset - 8) + t * 8 + rr;
    return t * 16 + rr;
}

// SwiGLU of two 16 x 16 tiles held as row r, columns 4 q .. 4 q + 3, the first 8 of them gate and the others up columns: lanes q <
// 2 finish the first tile, the others the second, each at row m and columns n .. n + 3.  One tile at a time, half of the lanes
// would repeat what the other half computes: 8B gate/up 1.5 % at 20 rows, 2 % at 128.
__device__ __forceinline__ void swiglu_store(const GemmArgs& a, floatx4 first, floatx4 second, int q, int m, int n, bool live) {
    half4 hi, lo;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const float other = __shfl_xor(q < 2 ? second[x] : first[x], 32, RL_WAVE);
        f16_t h, l;
        split_f16(swiglu_act(q < 2 ? first[x] : other, q < 2 ? other : second[x]), h, l);
        hi[x] = h; lo[x] = l;
    }
    if (live && m < a.M && n < a.N) {
        f16_t* o = a.outH + (int64_t)m * a.ldc + n;
        *reinterpret_cast<half4*>(o) = hi;
        if (a.split_out) *reinterpret_cast<half4*>(o + a.N) = lo;
    }
}

template <int EPI, int MT, int CT, bool WF16>
__global__ __launch_bounds__(512, gs_lds(MT, CT) <= 80 * 1024 ? 4 : 2) void gemm_stream_kernel(GemmArgs a) {
    constexpr int WN = 8 / GS_WK, CW = (CT + WN - 1) / WN, NW = gs_nw(MT, CT), NA = gs_na(MT, CT);
    constexpr int WST = CT * 16 * GS_RB, AST = MT * 16 * GS_RB;               // bytes of a stage
    constexpr int NBW = CT * 4, NBA = MT * 4;                                 // its 1 KB requests: 4 rows x 256 B each
    constexpr int NIW = (NBW + 7) / 8, NIA = (NBA + 7) / 8;                   // per wave; odd tile counts: half of the waves one fewer
    constexpr int IB = MT * CT * GS_WK * 1024 <= gs_lds(MT, CT) ? MT : MT / 2;   // row tiles per exchange at the end
    static_assert(IB * CT * GS_WK * 1024 <= gs_lds(MT, CT), "the exchange reuses the stages");
    static_assert(MT % 2 == 0 || MT == 1, "one odd A tile");
    extern __shared__ __attribute__((aligned(1024))) char smem[];            // [NW][W tiles] [NA][A tiles]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, q = lane >> 4, wk = wave % GS_WK, wn = wave / GS_WK;
    const int t0 = blockIdx.x * CT;                            // first 16-row tile of W
    const int kbeg = blockIdx.z * a.k_per_split, kend = min(a.Kw, kbeg + a.k_per_split);
    const int nk = (kend - kbeg) / GS_KT, kt0 = kbeg / GS_KT;
    // activations as fp16 pairs: every k-tile of W meets the hi tile of A, then the lo tile, in two trips; W is requested on the first
    const int pair = a.pair, nv = nk << pair;
    const int rot = a.rotate_k ? (int)(blockIdx.x % (unsigned)nk) : 0;
    // Staging: request t of a wave fills the 1 KB block t*8 + wave = 4 rows of a W stage, or (counted from wave 4 on if W's
    // tiles are odd) of an A stage; lane -> row + lane/16, physical chunk lane%16, which holds the row's logical chunk
    // (lane%16) ^ (row%16).
    const int wa = (wave + 4 * (CT & 1)) & 7;
    const bool has_w = CT % 2 == 0 || wave < 4, has_a = MT % 2 == 0 || wa < 4;     // the last request of the wave
    unsigned w_off[NIW], a_off[NIA];
#pragma unroll
    for (int t = 0; t < NIW; ++t) {
        const int row = (t * 8 + wave) * 4 + (lane >> 4);      // rows past the end: clamped, never stored
        w_off[t] = (unsigned)min(stream_w_row<EPI>(t0 + (row >> 4), row & 15, a), a.Wrows - 1) * (unsigned)a.Kw * 2u +
                   (unsigned)((lane & 15) ^ (row & 15)) * 16u;
    }
#pragma unroll
    for (int t = 0; t < NIA; ++t) {
        const int row = (t * 8 + wa) * 4 + (lane >> 4);
        a_off[t] = (unsigned)min(row, a.M - 1) * (unsigned)a.lda * 2u + (unsigned)((lane & 15) ^ (row & 15)) * 16u;
    }
    const unsigned lds_w = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem + wave * 1024;
    const unsigned lds_a = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem + NW * WST + wa * 1024;
    const char* const Ag = reinterpret_cast<const char*>(a.A);
    const char* const Wg = reinterpret_cast<const char*>(a.W);
#define GS_TILE(kt) (kt0 + ((kt) + rot >= nk ? (kt) + rot - nk : (kt) + rot))
#define GS_REQ(lds, off, g)                                                                                     \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds), "v"(off), "s"(g) : "memory")
#define GS_REQ_NT(lds, off, g)                                                                                  \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" :: "s"(lds), "v"(off), "s"(g) : "memory")
#define GS_ISSUE_W(stage, kt)                                                                                   \
    {                                                                                                           \
        const char* g_ = Wg + (size_t)GS_TILE(kt) * GS_RB;                                                      \
        if (a.stream_w) {                                                                                       \
            _Pragma("unroll") for (int t = 0; t < NIW; ++t)                                                     \
                if (t < NIW - 1 || has_w) { const unsigned l_ = lds_w + (stage) * WST + t * 8192; GS_REQ_NT(l_, w_off[t], g_); } \
        } else {                                                                                                \
            _Pragma("unroll") for (int t = 0; t < NIW; ++t)                                                     \
                if (t < NIW - 1 || has_w) { const unsigned l_ = lds_w + (stage) * WST + t * 8192; GS_REQ(l_, w_off[t], g_); } \
        }                                                                                                       \
    }
#define GS_ISSUE_A(stage, v)                                                                                    \
    {                                                                                                           \
        const int v_ = (v);                                                                                     \
        const char* g_ = Ag + (size_t)GS_TILE(v_ >> pair) * GS_RB + (v_ & pair ? a.Kw * 2 : 0);                 \
        _Pragma("unroll") for (int t = 0; t < NIA; ++t)                                                         \
            if (t < NIA - 1 || has_a) { const unsigned l_ = lds_a + (stage) * AST + t * 8192; GS_REQ(l_, a_off[t], g_); } \
    }
    floatx4 acc[MT][CW];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < CW; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int frag = r * GS_RB + (((wk * 4 + q) ^ r) * 16);    // this lane's 16 bytes of a 16-row tile
    // in the order of the loop's requests, so that its counts hold from the first k-tile on
#pragma unroll
    for (int s = 0; s < NW - 1; ++s) {
        if (s >= NW - NA && s - (NW - NA) < nv) GS_ISSUE_A(s - (NW - NA), s - (NW - NA))
        if (s < nk) GS_ISSUE_W(s, s)
    }
    int w_st = 0, a_st = 0, w_fill = NW - 1, a_fill = NA - 1;
    // at most w tiles of W and at most `as` of A on their way; waves with one request fewer than others count theirs
    auto wait = [&](auto wc, auto ac) {
        constexpr int w = decltype(wc)::value, as = decltype(ac)::value, all = NIW * w + NIA * as;
        if (CT % 2 != 0 && MT % 2 != 0) __builtin_amdgcn_s_waitcnt(dma_waitcnt(all - (w > as ? w : as), 0));   // every wave lacks one of either
        else if ((w == 0 || CT % 2 == 0 || has_w) && (as == 0 || MT % 2 == 0 || has_a)) __builtin_amdgcn_s_waitcnt(dma_waitcnt(all, 0));
        else __builtin_amdgcn_s_waitcnt(dma_waitcnt(all - (CT % 2 != 0 ? w : 0) - (MT % 2 != 0 ? as : 0), 0));
    };
    constexpr std::integral_constant<int, 0> none{};
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, NW - 2> fly_w{};
    constexpr std::integral_constant<int, NA - 2> fly_a{};
    for (int v = 0; v < nv; ++v) {
        // the trip's tiles landed, own fragment reads of the trip before done.  What may still be on its way is younger than the
        // trip's A tile: A of the next NA - 2 trips and as many tiles of W (one with two stages of A); nothing behind the last ones.
        // Pairs ask for W on every other trip, so that one is young at most (fewer are waited for than could be on some trips),
        // none near the end, nor with two stages of A on even trips
        if (v + 1 == nv) wait(none, none);
        else if (!pair) {
            if (NW == 4 && v + 2 == nv) wait(one, one);
            else wait(fly_w, fly_a);
        } else if (NA == 4) {
            if (v + 2 == nv) wait(none, one);
            else if (v + 6 > nv) wait(none, fly_a);
            else wait(one, fly_a);
        } else if (v + 3 >= nv || (NA == 2 && (v & 1) == 0)) wait(none, fly_a);
        else wait(one, fly_a);
        __syncthreads();
        // every wave is done with the trip before: its stages are filled again
        if (v + NA - 1 < nv) GS_ISSUE_A(a_fill, v + NA - 1)
        if (!(v & pair)) {
            if ((v >> pair) + NW - 1 < nk) GS_ISSUE_W(w_fill, (v >> pair) + NW - 1)
            w_fill = w_fill + 1 == NW ? 0 : w_fill + 1;
        }
        a_fill = a_fill + 1 == NA ? 0 : a_fill + 1;
        const char* sw = smem + w_st * WST + frag;
        const char* sa = smem + NW * WST + a_st * AST + frag;
        if ((v & pair) == pair) w_st = w_st + 1 == NW ? 0 : w_st + 1;
        a_st = a_st + 1 == NA ? 0 : a_st + 1;
        u32x4_t w[CW];
        half8 af[MT];
#pragma unroll
        for (int j = 0; j < CW; ++j)
            if (CT % WN == 0 || wn * CW + j < CT) w[j] = *reinterpret_cast<const u32x4_t*>(sw + (wn * CW + j) * 16 * GS_RB);
#pragma unroll
        for (int i = 0; i < MT; ++i) af[i] = *reinterpret_cast<const half8*>(sa + i * 16 * GS_RB);
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            if (CT % WN == 0 || wn * CW + j < CT) {
                const half8 wf = WF16 ? __builtin_bit_cast(half8, w[j]) : bf16x8_to_half8(w[j]);
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    acc[i][j] = EPI == MG_SWIGLU ? __builtin_amdgcn_mfma_f32_16x16x32_f16(wf, af[i], acc[i][j], 0, 0, 0)
                                                 : __builtin_amdgcn_mfma_f32_16x16x32_f16(af[i], wf, acc[i][j], 0, 0, 0);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(dma_waitcnt(0, 0));             // fragment reads done; nothing is on its way to LDS
#undef GS_ISSUE_A
#undef GS_ISSUE_W
#undef GS_TILE
    // the four waves along k meet in LDS, IB row tiles at a time; tile (i, j) of lane (r, q): column r, rows 4 q .. 4 q + 3
    // (gate/up: row r, columns 4 q .. 4 q + 3)
    floatx4* const red = reinterpret_cast<floatx4*>(smem);
#pragma unroll
    for (int i0 = 0; i0 < MT; i0 += IB) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
            for (int j = 0; j < CW; ++j)
                if (CT % WN == 0 || wn * CW + j < CT) red[((i * CT + wn * CW + j) * GS_WK + wk) * 64 + lane] = acc[i0 + i][j];
        __syncthreads();
        auto sum = [&](int i, int j) {
            const floatx4* p = red + (i * CT + j) * GS_WK * 64 + lane;
            floatx4 v = p[0];
#pragma unroll
            for (int w = 1; w < GS_WK; ++w) {
                const floatx4 o = p[w * 64];
#pragma unroll
                for (int x = 0; x < 4; ++x) v[x] += o[x];
            }
            return v;
        };
        if constexpr (EPI == MG_SAMPLE) {
            // statistics of 32-column blocks = two tiles; ties of the maximum go to the lowest column
            const int nblk = a.N / 32;
            for (int t = wave; t < IB * CT / 2; t += 8) {
                const int i = t / (CT / 2), jp = t % (CT / 2), blk = blockIdx.x * (CT / 2) + jp;
                const floatx4 v0 = sum(i, 2 * jp), v1 = sum(i, 2 * jp + 1);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    float mx = fmaxf(v0[x], v1[x]);
                    mx = fmaxf(mx, dpp_move<0xB1>(mx));    // quad_perm [1,0,3,2]
                    mx = fmaxf(mx, dpp_move<0x4E>(mx));    // quad_perm [2,3,0,1]
                    mx = fmaxf(mx, dpp_move<0x141>(mx));   // row_half_mirror
                    mx = fmaxf(mx, dpp_move<0x140>(mx));   // row_mirror
                    const unsigned h0 = (unsigned)(__ballot(v0[x] == mx) >> (16 * q)) & 0xffffu;
                    const unsigned h1 = (unsigned)(__ballot(v1[x] == mx) >> (16 * q)) & 0xffffu;
                    const int mi = __ffs(h0 | h1 << 16) - 1;
                    float e1 = __expf(v0[x] - mx) + __expf(v1[x] - mx);
                    float eT = __expf((v0[x] - mx) * a.inv_temp) + __expf((v1[x] - mx) * a.inv_temp);
                    e1 += dpp_move<0xB1>(e1); eT += dpp_move<0xB1>(eT);
                    e1 += dpp_move<0x4E>(e1); eT += dpp_move<0x4E>(eT);
                    e1 += dpp_move<0x141>(e1); eT += dpp_move<0x141>(eT);
                    e1 += dpp_move<0x140>(e1); eT += dpp_move<0x140>(eT);
                    const int m = (i0 + i) * 16 + q * 4 + x;
                    if (r == 0 && m < a.M && blk < nblk) a.samp_part[(int64_t)m * nblk + blk] = make_float4(mx, eT, e1, __int_as_float(mi));
                }
            }
        } else if constexpr (EPI == MG_SWIGLU) {
            constexpr int RT = IB > 1 ? 2 : 1;                 // row tiles at a time
            for (int t = wave; t < IB / RT * CT; t += 8) {
                const int i = t / CT * RT, j = t % CT;
                const floatx4 v = sum(i, j);
                swiglu_store(a, v, RT == 2 ? sum(i + RT - 1, j) : v, q, (i0 + i + (q >> 1)) * 16 + r, (t0 + j) * 8 + (q & 1) * 4, RT == 2 || q < 2);
            }
        } else {
            for (int t = wave; t < IB * CT; t += 8) {
                const int i = t / CT, j = t % CT;
                const floatx4 v = sum(i, j);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int m = (i0 + i) * 16 + q * 4 + x, n = (t0 + j) * 16 + r;
                    if (m < a.M && n < a.N) a.outF[(int64_t)blockIdx.z * a.split_stride + (int64_t)m * a.ldc + n] = v[x];
                }
            }
        }
    }
}

// GEMMs whose weights are more than one round of workgroups (LM heads, gate/up of the 70B width), on tiles of up to 128 rows x 256
// columns, the whole K each.  What a CU has on its way at once is about 64 KB, of W and A together, so A's bytes cost what W's
// do: 256 columns read A half as often as 128.  One round of wide tiles also pays once for what a workgroup does alone,
// its first loads and its epilogue.  Eight waves: two along the k-step of 64 (32 k each), four along the columns, each wave
// all rows; every W fragment is read, and on bf16 weights converted, by one wave.  As many stages as LDS holds, of which all but
// one are on their way; no request past the last k-step.  A pair layer's stage holds A's hi and lo rows: W is read once.  Chunks
// of the 128-byte rows are XOR-swizzled on the source side as above.  At the end the two waves along k each finish half of the
// row tiles and hand the other half over; a logit's fp32 sum is two chains over k instead of the stream kernel's four.  The MFMAs take W first: a lane holds four consecutive columns of a row.
// Against gemm_stream_kernel (fp16 weights; bf16 within 3 % of it), 3, 32, 64, 128 rows: LM head of the 8B shape 161, 170, 179, 218
// -> 161, 159, 164, 176 us; of 65536 x 4096 84, 88, 93, 109 -> 85, 84, 85, 87; 70B gate/up 148, 151, 152, 183 -> 144, 143,
// 145, 153; in a pair layer 147, 160, 186, 282 -> 145, 145, 151, 225.  Where stream_kernel's tiles are one round already it has the same or
// better times (8B gate/up at 128 rows takes 1.36 times as long on these, which leave half of the CUs idle; on a 56 x 128 form as long): wide_tiles.
static constexpr int GW_KT = 64, GW_RB = 128, GW_CT = 16;                // k-step, its bytes per row, column tiles
static constexpr int gw_stage(int MT, bool PAIR) { return (GW_CT + MT * (PAIR ? 2 : 1)) * 16 * GW_RB; }
static constexpr int gw_stages(int MT, bool PAIR) { return 160 * 1024 / gw_stage(MT, PAIR); }     // 2 .. 4

template <int EPI, int MT, bool WF16, bool PAIR>
__global__ __launch_bounds__(512, 2) void gemm_wide_kernel(GemmArgs a) {
    constexpr int CT = GW_CT, CW = CT / 4, S = gw_stages(MT, PAIR), ST = gw_stage(MT, PAIR);
    constexpr int NB = ST / 1024, NI = (NB + 7) / 8;           // 1 KB requests of a stage, 8 rows each; per wave
    constexpr int KEEP = MT > 1 ? MT / 2 : 1;                  // row tiles a wave finishes
    static_assert(8 * KEEP * CW * 1024 <= S * ST, "the exchange reuses the stages");
    extern __shared__ __attribute__((aligned(1024))) char smem[];            // [S][W tiles | A tiles | A tiles, lo]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, q = lane >> 4, kh = wave & 1, wn = wave >> 1;
    const int t0 = blockIdx.x * CT;                            // first 16-row tile of W
    const int nk = a.Kw / GW_KT;
    const int rot = a.rotate_k ? (int)((blockIdx.x * 2) % (unsigned)nk) : 0;
    // request t of a wave fills the 1 KB block t * 8 + wave of a stage; lane -> row + lane / 8, physical chunk lane % 8, which holds
    // the row's logical chunk (lane % 8) ^ (row / 2 % 8)
    const bool has_last = NB % 8 == 0 || wave < NB % 8;
    unsigned off[NI];
#pragma unroll
    for (int t = 0; t < NI; ++t) {
        const int row = (t * 8 + wave) * 8 + (lane >> 3);      // rows past the end: clamped, never stored
        const unsigned ch = (unsigned)((lane & 7) ^ ((row >> 1) & 7)) * 16u;
        if (t * 8 + wave < CT * 2) off[t] = (unsigned)min(stream_w_row<EPI>(t0 + (row >> 4), row & 15, a), a.Wrows - 1) * (unsigned)a.Kw * 2u + ch;
        else {
            const int ra = row - CT * 16, m = ra < MT * 16 ? ra : ra - MT * 16;
            off[t] = (unsigned)min(m, a.M - 1) * (unsigned)a.lda * 2u + (ra < MT * 16 ? 0u : (unsigned)a.Kw * 2u) + ch;
        }
    }
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem + wave * 1024;
    const char* const Ag = reinterpret_cast<const char*>(a.A);
    const char* const Wg = reinterpret_cast<const char*>(a.W);
#define GW_ISSUE(stage, k)                                                                                      \
    {                                                                                                           \
        const int k_ = (k) + rot;                                                                               \
        const size_t o_ = (size_t)(k_ >= nk ? k_ - nk : k_) * GW_RB;                                    \
        _Pragma("unroll") for (int t = 0; t < NI; ++t) {                                                        \
            const unsigned l_ = lds0 + (stage) * ST + t * 8192;                                                 \
            if (t < NI - 1 || has_last) {                                                                       \
                if (t * 8 + wave < CT * 2) {                                                                    \
                    const char* g_ = Wg + o_;                                                                   \
                    if (a.stream_w) GS_REQ_NT(l_, off[t], g_);                                                  \
                    else GS_REQ(l_, off[t], g_);                                                                \
                } else {                                                                                        \
                    const char* g_ = Ag + o_;                                                                   \
                    GS_REQ(l_, off[t], g_);                                                                     \
                }                                                                                               \
            }                                                                                                   \
        }                                                                                                       \
    }
    floatx4 acc[MT][CW];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < CW; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
        if (s < nk) GW_ISSUE(s, s)
    const int frag = r * GW_RB + (((kh * 4 + q) ^ ((r >> 1) & 7)) * 16);     // this lane's 16 bytes of a 16-row tile
    int st = 0, fill = S - 1;
    static_assert(S >= 2 && S <= 4, "waits written out below");
    auto landed = [&](int left, auto uc) __attribute__((always_inline)) {
        constexpr int u = decltype(uc)::value;
        if (u > S - 2 || (u == S - 2 ? left < u : left != u)) return;
        if (has_last) __builtin_amdgcn_s_waitcnt(dma_waitcnt(NI * u, 0));
        else __builtin_amdgcn_s_waitcnt(dma_waitcnt((NI - 1) * u, 0));
    };
    for (int j = 0; j < nk; ++j) {
        // stage j landed, own fragment reads of the step before done; the steps requested behind it, at most S - 2, may be on their way
        const int left = nk - 1 - j;
        landed(left, std::integral_constant<int, 2>{});
        landed(left, std::integral_constant<int, 1>{});
        landed(left, std::integral_constant<int, 0>{});
        __syncthreads();
        // every wave is done with the step before: its stage is filled again
        if (left >= S - 1) GW_ISSUE(fill, j + S - 1)
        fill = fill + 1 == S ? 0 : fill + 1;
        const char* sw = smem + st * ST + frag;
        const char* sa = sw + CT * 16 * GW_RB;
        st = st + 1 == S ? 0 : st + 1;
        u32x4_t w[CW];
        half8 af[MT];
#pragma unroll
        for (int c = 0; c < CW; ++c)
            w[c] = *reinterpret_cast<const u32x4_t*>(sw + (wn * CW + c) * 16 * GW_RB);
#pragma unroll
        for (int p = 0; p < (PAIR ? 2 : 1); ++p) {
#pragma unroll
            for (int i = 0; i < MT; ++i) af[i] = *reinterpret_cast<const half8*>(sa + (p * MT + i) * 16 * GW_RB);
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const half8 wf = WF16 ? __builtin_bit_cast(half8, w[c]) : bf16x8_to_half8(w[c]);
#pragma unroll
                for (int i = 0; i < MT; ++i) acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf, af[i], acc[i][c], 0, 0, 0);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(dma_waitcnt(0, 0));             // fragment reads done; nothing is on its way to LDS
#undef GW_ISSUE
    // The two waves along k: each finishes half of the row tiles and hands the other half over
    floatx4* const red = reinterpret_cast<floatx4*>(smem);
    __syncthreads();
    if (MT > 1 || kh == 1) {
#pragma unroll
        for (int i = 0; i < KEEP; ++i)
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const floatx4 first = acc[i][c], second = acc[MT > 1 ? KEEP + i : 0][c];
                red[((wave * KEEP + i) * CW + c) * 64 + lane] = MT == 1 || kh ? first : second;
            }
    }
    __syncthreads();
    if (MT == 1 && kh == 1) return;
    const int m0 = kh * KEEP * 16;
    floatx4 v[KEEP][CW];
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const floatx4 first = acc[i][c], second = acc[MT > 1 ? KEEP + i : 0][c], own = MT > 1 && kh ? second : first;
            const floatx4 o = red[(((wave ^ 1) * KEEP + i) * CW + c) * 64 + lane];
#pragma unroll
            for (int x = 0; x < 4; ++x) v[i][c][x] = own[x] + o[x];
        }
    // lane (r, q): row r of a row tile, columns 4 q .. 4 q + 3 of a column tile
#pragma unroll
    for (int i = 0; i < KEEP; ++i) {
        const int m = m0 + i * 16 + r;
        if constexpr (EPI == MG_SAMPLE) {
            // statistics of 32-column blocks = two tiles; ties of the maximum go to the lowest column
            const int nblk = a.N / 32;
#pragma unroll
            for (int c = 0; c < CW; c += 2) {
                const int blk = (t0 + wn * CW + c) / 2;
                const floatx4 v0 = v[i][c], v1 = v[i][c + 1];
                float mx = fmaxf(fmaxf(fmaxf(v0[0], v0[1]), fmaxf(v0[2], v0[3])), fmaxf(fmaxf(v1[0], v1[1]), fmaxf(v1[2], v1[3])));
                mx = fmaxf(mx, __shfl_xor(mx, 16, RL_WAVE));
                mx = fmaxf(mx, __shfl_xor(mx, 32, RL_WAVE));
                int mi = 32;
                float e1 = 0.f, eT = 0.f;
#pragma unroll
                for (int x = 3; x >= 0; --x) mi = v1[x] == mx ? 16 + q * 4 + x : mi;
#pragma unroll
                for (int x = 3; x >= 0; --x) mi = v0[x] == mx ? q * 4 + x : mi;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    e1 += __expf(v0[x] - mx) + __expf(v1[x] - mx);
                    eT += __expf((v0[x] - mx) * a.inv_temp) + __expf((v1[x] - mx) * a.inv_temp);
                }
                mi = min(mi, __shfl_xor(mi, 16, RL_WAVE));
                e1 += __shfl_xor(e1, 16, RL_WAVE);
                eT += __shfl_xor(eT, 16, RL_WAVE);
                mi = min(mi, __shfl_xor(mi, 32, RL_WAVE));
                e1 += __shfl_xor(e1, 32, RL_WAVE);
                eT += __shfl_xor(eT, 32, RL_WAVE);
                if (q == 0 && m < a.M && blk < nblk)
                    a.samp_part[(int64_t)m * nblk + blk] = make_float4(mx, eT, e1, __int_as_float(mi < 32 ? mi : -1));
            }
        } else {
#pragma unroll
            for (int c = 0; c < CW; c += 2)
                swiglu_store(a, v[i][c], v[i][c + 1], q, m, (t0 + wn * CW + c + (q >> 1)) * 8 + (q & 1) * 4, true);
        }
    }
}
#undef GS_REQ
#undef GS_REQ_NT

// Tiles per workgroup and splits over K.  A workgroup's time goes with its k-tiles x (CT + what its rows of A cost), times
// the rounds of 256 workgroups; each split costs its consumer a pass over the partial sums.  Both costs are those of the
// context's limit (64 rows or 128).  Of the measured candidates the rule takes the fastest or one within 3 %: up to 64 rows 8B QKV
// 3 x 2 splits, O and down 4 x 4, gate/up 7, 1B O 2 x 4, down 4 x 8, gate/up 4, 70B QKV 5 x 2, O and down 8 x 4, gate/up 7, LM
// heads 8; up to 128 rows 8B QKV 6 x 4 (17.2 us; 3 x 2: 20), O 4 x 4 (13.2; 8 x 8: 15.2), down 8 x 8 (31.6; 4 x 4: 35), gate/up 7.
// A pair layer's rows of A count twice; its choices are within 3 % of the best of those measured at 3 to 128 rows.
// The rule must not look at the rows of a call: a row's bits would depend on its batch-mates.  z: in, the number of splits, 0
// for the best; out, theirs.
static void stream_plan(int epi, int N, int K, int Kw, int max_rows, int& ct, int& z) {
    const int tiles = (epi == MG_SWIGLU ? 2 * N : N) / 16, units = Kw / GS_KT;
    const int zmin = z > 0 ? z : 1, zmax = z > 0 ? z : (units < 8 ? units : 8);
    const float rows = (max_rows <= 64 ? 1.f : 4.f) * (float)(K / Kw), split = max_rows <= 64 ? 1.8f : 5.f;
    float best = 0.f;
    ct = 0;
    for (int zz = zmin; zz <= zmax; ++zz) {
        const int per = (units + zz - 1) / zz;
        if ((units + per - 1) / per != zz) continue;
        for (int c = 1; c <= 8; ++c) {
            if (epi == MG_SAMPLE && c % 2 != 0) continue;
            const int wgs = (tiles + c - 1) / c * zz;
            const float cost = (float)((wgs + 255) / 256) * (float)per * ((float)c + rows) + split * (float)zz * (float)N / 2048.f;
            if (ct == 0 || cost < best) { best = cost; ct = c; z = zz; }
        }
    }
}

// Whether a GEMM without splits takes gemm_wide_kernel: rounds of 256 workgroups times what one draws per k-step (its columns and
// rows in 16s; A of a context of more than 64 rows counts 4, as above) and 2 for what it does alone.  Measured at 3 to
// 128 rows on 4 LM heads and 4 gate/up widths, plain and pair, fp16 and bf16 (tiles of 16 columns: 1024 to 9496): the faster one, or within
// 2 % at 3 rows and 5 % above.  As the plan, it must not look at the rows of a call.
static bool wide_tiles(int tiles, int ct, int pair, int max_rows) {
    const int rows = (max_rows <= 64 ? 1 : 4) << pair;
    auto rounds = [&](int c) { return ((tiles + c - 1) / c + 255) / 256; };
    return rounds(GW_CT) * (GW_CT + 2 + rows) <= rounds(ct) * (ct + 2 + rows);
}

bool k_gemm_decode_supported(int epi, int N, int K, int Kw) {
    if (epi != MG_STORE_F32 && epi != MG_SWIGLU && epi != MG_SAMPLE) return false;
    const int rows = epi == MG_SWIGLU ? 2 * N : N;
    return K > 0 && (K == Kw || K == 2 * Kw) && Kw % GS_KT == 0 && rows % 32 == 0 && (uint64_t)rows * Kw * 2 < (1ull << 32);
}

int k_gemm_decode_splits(int N, int K, int Kw, int max_rows) {
    int ct, z = 0;
    stream_plan(MG_STORE_F32, N, K, Kw, max_rows, ct, z);
    return z;
}

template <int EPI, int MT, int CT, bool WF16>
static void launch_stream_t(const GemmArgs& a, int tiles, int z, hipStream_t s) {
    constexpr int lds = gs_lds(MT, CT);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void*)gemm_stream_kernel<EPI, MT, CT, WF16>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    gemm_stream_kernel<EPI, MT, CT, WF16><<<dim3((tiles + CT - 1) / CT, 1, z), 512, lds, s>>>(a);
}
template <int EPI, int CT>
static void launch_stream_ct(const GemmArgs& a, int tiles, int z, hipStream_t s) {
    if constexpr (EPI != MG_SAMPLE || CT % 2 == 0) {
        if (a.w_f16) {
            if (a.M <= 16) launch_stream_t<EPI, 1, CT, true>(a, tiles, z, s);
            else if (a.M <= 32) launch_stream_t<EPI, 2, CT, true>(a, tiles, z, s);
            else if (a.M <= 64) launch_stream_t<EPI, 4, CT, true>(a, tiles, z, s);
            else launch_stream_t<EPI, 8, CT, true>(a, tiles, z, s);
        } else {
            if (a.M <= 16) launch_stream_t<EPI, 1, CT, false>(a, tiles, z, s);
            else if (a.M <= 32) launch_stream_t<EPI, 2, CT, false>(a, tiles, z, s);
            else if (a.M <= 64) launch_stream_t<EPI, 4, CT, false>(a, tiles, z, s);
            else launch_stream_t<EPI, 8, CT, false>(a, tiles, z, s);
        }
    }
}
template <int EPI, int MT, bool WF16, bool PAIR>
static void launch_wide_t(const GemmArgs& a, int tiles, hipStream_t s) {
    constexpr int lds = gw_stages(MT, PAIR) * gw_stage(MT, PAIR);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void*)gemm_wide_kernel<EPI, MT, WF16, PAIR>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    gemm_wide_kernel<EPI, MT, WF16, PAIR><<<(tiles + GW_CT - 1) / GW_CT, 512, lds, s>>>(a);
}
template <int EPI, bool WF16, bool PAIR>
static void launch_wide_m(const GemmArgs& a, int tiles, hipStream_t s) {
    if (a.M <= 16) launch_wide_t<EPI, 1, WF16, PAIR>(a, tiles, s);
    else if (a.M <= 32) launch_wide_t<EPI, 2, WF16, PAIR>(a, tiles, s);
    else if (a.M <= 64) launch_wide_t<EPI, 4, WF16, PAIR>(a, tiles, s);
    else launch_wide_t<EPI, 8, WF16, PAIR>(a, tiles, s);
}
template <int EPI>
static void launch_wide(const GemmArgs& a, int tiles, hipStream_t s) {
    if (a.w_f16) {
        if (a.pair) launch_wide_m<EPI, true, true>(a, tiles, s);
        else launch_wide_m<EPI, true, false>(a, tiles, s);
    } else {
        if (a.pair) launch_wide_m<EPI, false, true>(a, tiles, s);
        else launch_wide_m<EPI, false, false>(a, tiles, s);
    }
}
template <int EPI>
static void launch_stream(const GemmArgs& a, int tiles, int ct, int z, hipStream_t s) {
    switch (ct) {
        case 1: launch_stream_ct<EPI, 1>(a, tiles, z, s); break;
        case 2: launch_stream_ct<EPI, 2>(a, tiles, z, s); break;
        case 3: launch_stream_ct<EPI, 3>(a, tiles, z, s); break;
        case 4: launch_stream_ct<EPI, 4>(a, tiles, z, s); break;
        case 5: launch_stream_ct<EPI, 5>(a, tiles, z, s); break;
        case 6: launch_stream_ct<EPI, 6>(a, tiles, z, s); break;
        case 7: launch_stream_ct<EPI, 7>(a, tiles, z, s); break;
        default: launch_stream_ct<EPI, 8>(a, tiles, z, s); break;
    }
}

static int g_decode_tile_above = -1;   // measurement switch: rows above which the 128 x 128 tile kernel runs; < 0: never
void k_gemm_decode_tile_above(int rows) { g_decode_tile_above = rows; }

void k_gemm_decode(int epi, GemmArgs a, int splits, int max_rows, hipStream_t s) {
    if (a.Kw <= 0) a.Kw = a.K;
    if (a.M <= 0 || a.M > 128 || !k_gemm_decode_supported(epi, a.N, a.K, a.Kw)) return;   // callers check first
    int ct, z = epi == MG_STORE_F32 && splits > 1 ? splits : 1;
    stream_plan(epi, a.N, a.K, a.Kw, max_rows, ct, z);
    if (ct == 0) return;                                       // a split count that is not one of this K's
    a.Wrows = epi == MG_SWIGLU ? a.up_offset + a.N : a.N;
    if (g_decode_tile_above >= 0 && a.M > g_decode_tile_above && epi != MG_SAMPLE && (epi == MG_SWIGLU ? 2 * a.N : a.N) % 128 == 0) {
        a.k_per_split = (a.K / GS_KT + z - 1) / z * GS_KT;     // as many splits, of hi and lo one behind the other
        k_gemm_tile_decode(epi, a, z, s);
        return;
    }
    a.pair = a.K == 2 * a.Kw;
    // Weights pass through the caches once; those that are well beyond the eight L2s together (32 MB) are read as non-temporal. Alone: 8B
    // gate/up 41.7 -> 37.5 us at 32 rows, 51.5 -> 48.6 at 128, down 23.4 -> 21.5 at 32, LM head 177 -> 159 (183 -> 162 at 3 rows), 70B gate/up
    // 162 -> 142 at 64, 1B gate/up (67 MB) 14.4 -> 13.4 at 32; at 128 rows that one is longer alone, 21.2 -> 21.9, and a generation
    // 0.7 % shorter.  In a step 70B down 89 -> 78, QKV 33.4 -> 31.2 at 64 rows.  Below that they are slower: 8B QKV (50 MB) at 128 rows
    // in a step 18.8 -> 21.2, O (34 MB) 13.3 -> 14.0.
    a.stream_w = (int64_t)a.Wrows * a.Kw * 2 > ((int64_t)60 << 20);
    a.k_per_split = (a.Kw / GS_KT + z - 1) / z * GS_KT;
    a.rotate_k = (a.Kw & (a.Kw - 1)) == 0 && a.k_per_split >= 16 * GS_KT;
    const int tiles = (epi == MG_SWIGLU ? 2 * a.N : a.N) / 16;
    if (epi != MG_STORE_F32 && wide_tiles(tiles, ct, a.pair, max_rows)) {
        if (epi == MG_SWIGLU) launch_wide<MG_SWIGLU>(a, tiles, s);
        else launch_wide<MG_SAMPLE>(a, tiles, s);
        return;
    }
    if (epi == MG_STORE_F32) launch_stream<MG_STORE_F32>(a, tiles, ct, z, s);
    else if (epi == MG_SWIGLU) launch_stream<MG_SWIGLU>(a, tiles, ct, z, s);
    else launch_stream<MG_SAMPLE>(a, tiles, ct, z, s);
}
