// Plain reference kernels for every step of the rollout path (any dtype) plus the
// small bookkeeping kernels (packing, paging, sampling, log-sum-exp, KL).
// The formulas are the standard Llama-style decoder ones; the paper (Sections 3.1-3.2)
// only names the stages.
#include <type_traits>

#include "rl_common.h"

// ---------------------------------------------------------------- fills / tables
__global__ void fill_i32_kernel(int* p, int v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
__global__ void fill_f32_kernel(float* p, float v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
void k_fill_i32(int* p, int v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    fill_i32_kernel<<<dim3((unsigned)((n + 255) / 256)), 256, 0, s>>>(p, v, n);
}
void k_fill_f32(float* p, float v, int64_t n, hipStream_t s) {
    if (n <= 0) return;
    fill_f32_kernel<<<dim3((unsigned)((n + 255) / 256)), 256, 0, s>>>(p, v, n);
}

// cos/sin of pos * base^(-2j/hd), evaluated in fp64 and rounded once to fp32.
__global__ void rope_table_kernel(float2* tab, int max_seq, int half, double log_base, int hd) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= max_seq * half) return;
    int pos = i / half, j = i % half;
    double theta = exp(-2.0 * (double)j / (double)hd * log_base);
    double ang = (double)pos * theta;
    tab[i] = make_float2((float)cos(ang), (float)sin(ang));
}
void k_rope_table(float2* tab, int max_seq, int hd, float base, hipStream_t s) {
    int n = max_seq * (hd / 2);
    rope_table_kernel<<<(n + 255) / 256, 256, 0, s>>>(tab, max_seq, hd / 2, log((double)base), hd);
}

// block_table[slot][idx] = page for up to 64 (slot, idx, page) triples passed by value.
struct PageTriples { int v[192]; };
__global__ void set_pages_kernel(int* bt, int mpps, PageTriples t, int n) {
    int i = threadIdx.x;
    if (i < n) bt[(int64_t)t.v[3 * i] * mpps + t.v[3 * i + 1]] = t.v[3 * i + 2];
}
void k_set_pages(int* block_table, int mpps, const int* triples_host, int n_triples, hipStream_t s) {
    for (int o = 0; o < n_triples; o += 64) {
        PageTriples t;
        int n = n_triples - o < 64 ? n_triples - o : 64;
        for (int i = 0; i < 3 * n; ++i) t.v[i] = triples_host[3 * o + i];
        set_pages_kernel<<<1, 64, 0, s>>>(block_table, mpps, t, n);
    }
}

// ---------------------------------------------------------------- token bookkeeping
// Row descriptors of a chunk -- batch row, cache slot, first packed row, length of up to 240 rows -- reach the device as
// kernel arguments: nothing is copied from host memory that would have to outlive the call, so the call need not wait.
struct RowDescs { int v[4 * 240]; };
__global__ void put_rows_kernel(RowDescs r, int n, int first, int* seq_first, int* row_slot, int* row_start, int* row_len) {
    const int i = threadIdx.x;
    if (i >= n) return;
    seq_first[first + i] = r.v[4 * i];
    row_slot[first + i] = r.v[4 * i + 1];
    row_start[first + i] = r.v[4 * i + 2];
    row_len[first + i] = r.v[4 * i + 3];
}
void k_put_rows(const int* seq_first_h, const int* row_slot_h, const int* row_start_h, const int* row_len_h, int n,
                int* seq_first, int* row_slot, int* row_start, int* row_len, hipStream_t s) {
    for (int o = 0; o < n; o += 240) {
        RowDescs r;
        const int m = n - o < 240 ? n - o : 240;
        for (int i = 0; i < m; ++i) {
            r.v[4 * i] = seq_first_h[o + i];
            r.v[4 * i + 1] = row_slot_h[o + i];
            r.v[4 * i + 2] = row_start_h[o + i];
            r.v[4 * i + 3] = row_len_h[o + i];
        }
        put_rows_kernel<<<1, 256, 0, s>>>(r, m, o, seq_first, row_slot, row_start, row_len);
    }
}
// List of the rows first[i] .. first[i] + count[i] - 1 of every sequence i, from at[i] on.
__global__ void list_rows_kernel(const int* at, const int* first, const int* count, int* rows) {
    const int i = blockIdx.x;
    for (int j = threadIdx.x; j < count[i]; j += blockDim.x) rows[at[i] + j] = first[i] + j;
}
void k_list_rows(const int* at, const int* first, const int* count, int n, int* rows, hipStream_t s) {
    if (n > 0) list_rows_kernel<<<n, 256, 0, s>>>(at, first, count, rows);
}
// One block per row, 16 bytes per access.
__global__ __launch_bounds__(256) void gather_rows_kernel(const f16_t* src_a, f16_t* dst_a, int wa, const float* src_x, float* dst_x,
                                                          int d, const int* rows) {
    const int64_t i = blockIdx.x, r = rows[i];
    const float4* sa = reinterpret_cast<const float4*>(src_a + r * wa);
    const float4* sx = reinterpret_cast<const float4*>(src_x + r * d);
    float4* da = reinterpret_cast<float4*>(dst_a + i * wa);
    float4* dx = reinterpret_cast<float4*>(dst_x + i * d);
    for (int j = threadIdx.x; j < wa / 8; j += 256) da[j] = sa[j];
    for (int j = threadIdx.x; j < d / 4; j += 256) dx[j] = sx[j];
}
void k_gather_rows(const f16_t* src_a, f16_t* dst_a, int wa, const float* src_x, float* dst_x, int d, const int* rows, int n,
                   hipStream_t s) {
    if (n > 0) gather_rows_kernel<<<n, 256, 0, s>>>(src_a, dst_a, wa, src_x, dst_x, d, rows);
}
// Pack rows of a padded [*, ld_ids] id matrix into a flat token list.
// Row r of the chunk is batch row seq_first[r]; its row_len[r] tokens go to
// [row_start[r], row_start[r] + row_len[r]).  tok_tgt (optional) = next token id of the
// same row, or -1 when there is none.
// With align > 1 every row is padded to a multiple of align tokens; padding entries carry
// token id 0, position -1 and no target.
// blocks (optional): the prefill attention's work list, one entry (first row, length, query block) per block of qrows queries,
// late (long) blocks first so that the tail of the grid is short work, rows in order within a block index: an entry's
// place is the number of entries with a later block, plus the earlier rows that have this one.
__global__ void pack_tokens_kernel(const int* ids, int ld_ids, const int* seq_first, const int* row_slot,
                                   const int* row_start, const int* row_len, int align, int* tok_ids, int* tok_pos,
                                   int* tok_slot, int* tok_tgt, int4* blocks, int qrows) {
    int r = blockIdx.x;
    int b = seq_first[r], st = row_start[r], len = row_len[r];
    const int slot = row_slot[r];
    const int alen = (len + align - 1) / align * align;
    const int* src = ids + (int64_t)b * ld_ids;
    for (int t = threadIdx.x; t < alen; t += blockDim.x) {
        const bool real = t < len;
        tok_ids[st + t] = real ? src[t] : 0;
        tok_pos[st + t] = real ? t : -1;
        tok_slot[st + t] = slot;
        if (tok_tgt) tok_tgt[st + t] = (real && t + 1 < len) ? src[t + 1] : -1;
    }
    if (!blocks) return;
    for (int qb = threadIdx.x; qb < (len + qrows - 1) / qrows; qb += blockDim.x) {
        int at = 0;
        for (int i = 0; i < (int)gridDim.x; ++i) {
            const int nbi = (row_len[i] + qrows - 1) / qrows;
            at += max(0, nbi - (qb + 1)) + (i < r && nbi > qb ? 1 : 0);
        }
        blocks[at] = make_int4(st, len, qb, 0);
    }
}
void k_pack_tokens(const int* ids, int ld_ids, const int* seq_first, const int* row_slot, const int* row_start,
                   const int* row_len, int align, int* tok_ids, int* tok_pos, int* tok_slot, int* tok_tgt, int4* blocks,
                   int qrows, int nrows, hipStream_t s) {
    if (nrows <= 0) return;
    pack_tokens_kernel<<<nrows, 256, 0, s>>>(ids, ld_ids, seq_first, row_slot, row_start, row_len, align, tok_ids, tok_pos,
                                             tok_slot, tok_tgt, blocks, qrows);
}

// After prefill of the first P-1 prompt tokens: remember the last prompt token, lengths, counters.
__global__ void prefill_state_kernel(const int* ids, int ld_ids, const int* prompt_len, int* last_tok, int* seq_len,
                                     int* gen_count, int* finished, int* step_count, int B) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    int P = prompt_len[b];
    last_tok[b] = ids[(int64_t)b * ld_ids + P - 1];
    seq_len[b] = P - 1;
    gen_count[b] = 0;
    finished[b] = 0;
    step_count[b] = 0;
}
void k_prefill_state(const int* ids, int ld_ids, const int* row_len, int* last_tok, int* seq_len, int* gen_count,
                     int* finished, int* step_count, int B, hipStream_t s) {
    prefill_state_kernel<<<(B + 255) / 256, 256, 0, s>>>(ids, ld_ids, row_len, last_tok, seq_len, gen_count,
                                                         finished, step_count, B);
}

__global__ void prefill_state_slots_kernel(const int* ids, int ld_ids, int n, const int* seq_first, const int* row_slot,
                                           const int* row_len, const int* limit, int* last_tok, int* seq_len,
                                           int* gen_count, int* finished, int* step_count, int* out_row, int* seq_id,
                                           int* gen_limit) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int row = seq_first[i], b = row_slot[i], P = row_len[i];
    last_tok[b] = ids[(int64_t)row * ld_ids + P - 1];
    seq_len[b] = P - 1;
    gen_count[b] = 0;
    finished[b] = 0;
    step_count[b] = 0;
    out_row[b] = row;
    seq_id[b] = row;
    gen_limit[b] = limit[i];
}
void k_prefill_state_slots(const int* ids, int ld_ids, int n, const int* seq_first, const int* row_slot,
                           const int* row_len, const int* limit, int* last_tok, int* seq_len, int* gen_count,
                           int* finished, int* step_count, int* out_row, int* seq_id, int* gen_limit, hipStream_t s) {
    if (n <= 0) return;
    prefill_state_slots_kernel<<<(n + 255) / 256, 256, 0, s>>>(ids, ld_ids, n, seq_first, row_slot, row_len, limit,
                                                               last_tok, seq_len, gen_count, finished, step_count,
                                                               out_row, seq_id, gen_limit);
}

__global__ void out_len_kernel(const int* gen_count, int* out_len, int B) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) out_len[b] = gen_count[b];
}
void k_out_len(const int* gen_count, int* out_len, int B, hipStream_t s) {
    out_len_kernel<<<(B + 255) / 256, 256, 0, s>>>(gen_count, out_len, B);
}

typedef float floatx4 __attribute__((ext_vector_type(4)));
// four consecutive values (4-element aligned) as floats
template <typename T>
__device__ __forceinline__ floatx4 load4(const T* p) {
    typedef T T4 __attribute__((ext_vector_type(4)));
    const T4 v = *reinterpret_cast<const T4*>(p);
    return floatx4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}

// ---------------------------------------------------------------- embedding gather
template <typename T>
__global__ void embed_kernel(const int* ids, const T* E, int d, int V, float* x, int* errflag, const T* E2, int n1) {
    int n = blockIdx.x;
    int id = ids[n];
    if (id < 0 || id >= V) {
        if (threadIdx.x == 0) atomicOr(errflag, 1);
        id = id < 0 ? 0 : V - 1;
    }
    const T* row = (E2 && n >= n1 ? E2 : E) + (int64_t)id * d;
    float* xo = x + (int64_t)n * d;
    for (int j = threadIdx.x; j < d; j += blockDim.x) xo[j] = to_f(row[j]);
}
void k_embed(int dtype, const int* ids, int n, const void* E, int d, int V, float* x, int* errflag, hipStream_t s,
             const void* E2, int n1) {
    if (n <= 0) return;
    if (dtype == 0) embed_kernel<float><<<n, 256, 0, s>>>(ids, (const float*)E, d, V, x, errflag, (const float*)E2, n1);
    else embed_kernel<bf16_t><<<n, 256, 0, s>>>(ids, (const bf16_t*)E, d, V, x, errflag, (const bf16_t*)E2, n1);
}

// Store v as T at o[0]; with split also what the rounding left over, as T, at o[lo_off]: the pair hi + lo
// carries about 22 significant bits when T is fp16.
template <typename T>
__device__ __forceinline__ void put_pair(T* o, int64_t lo_off, float v, int split) {
    const T hi = from_f<T>(v);
    o[0] = hi;
    if (split) o[lo_off] = from_f<T>(v - to_f(hi));
}
// Four consecutive gains, fetched as they are stored.
template <typename TW> struct Gain4 {
    typedef typename std::conditional<sizeof(TW) == 2, uint2, float4>::type raw_t;
    raw_t raw;
    __device__ __forceinline__ void load(const TW* g) { raw = *reinterpret_cast<const raw_t*>(g); }
    __device__ __forceinline__ void get(float (&gf)[4]) const {
        if constexpr (sizeof(TW) == 2) {                                  // bf16
            gf[0] = __uint_as_float(raw.x << 16); gf[1] = __uint_as_float(raw.x & 0xffff0000u);
            gf[2] = __uint_as_float(raw.y << 16); gf[3] = __uint_as_float(raw.y & 0xffff0000u);
        } else {
            gf[0] = raw.x; gf[1] = raw.y; gf[2] = raw.z; gf[3] = raw.w;
        }
    }
};
// Four consecutive values (o 4-element aligned) scaled by four consecutive gains: one store per plane.
template <typename T, typename TW>
__device__ __forceinline__ void put_pair4(T* o, int64_t lo_off, float4 v, float rs, const Gain4<TW>& g, int split) {
    float gf[4];
    g.get(gf);
    const float w[4] = {v.x * rs * gf[0], v.y * rs * gf[1], v.z * rs * gf[2], v.w * rs * gf[3]};
    if constexpr (sizeof(T) == 2) {
        typedef T T4 __attribute__((ext_vector_type(4)));
        T4 hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            hi[e] = from_f<T>(w[e]);
            lo[e] = from_f<T>(w[e] - to_f(hi[e]));
        }
        *reinterpret_cast<T4*>(o) = hi;
        if (split) *reinterpret_cast<T4*>(o + lo_off) = lo;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) put_pair(o + e, lo_off, w[e], split);
    }
}
template <typename T, typename TW>
__device__ __forceinline__ void put_pair4(T* o, int64_t lo_off, float4 v, float rs, const TW* g, int split) {
    Gain4<TW> gain;
    gain.load(g);
    put_pair4(o, lo_off, v, rs, gain, split);
}

// ---------------------------------------------------------------- RMSNorm: out = x * rsqrt(mean(x^2) + eps) * g
// split: the output row is twice as wide, [d values rounded to T | d remainders] (fp16 pairs).
// rows (optional): output row n is the norm of row rows[n].  g2 (optional): the gains of rows n1 and later.
template <typename T, typename TW>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* x, const TW* g, T* out, int d, float eps, int split,
                                                      const int* rows, const TW* g2, int n1) {
    __shared__ float red[16];
    int n = blockIdx.x;
    if (g2 && n >= n1) g = g2;
    const float* xr = x + (int64_t)(rows ? rows[n] : n) * d;
    T* o = out + (int64_t)n * d * (split ? 2 : 1);
    if (d % 4 == 0 && d <= 8192) {
        // the row is read once, 16 bytes per lane, and kept in registers between the two passes
        float4 keep[8];
        float ss = 0.f;
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int j = (it * 256 + threadIdx.x) * 4;
            if (j < d) {
                keep[it] = *reinterpret_cast<const float4*>(xr + j);
                ss += keep[it].x * keep[it].x + keep[it].y * keep[it].y + keep[it].z * keep[it].z + keep[it].w * keep[it].w;
            }
        }
        ss = block_sum(ss, red);
        const float rs = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int j = (it * 256 + threadIdx.x) * 4;
            if (j < d) put_pair4(o + j, d, keep[it], rs, g + j, split);
        }
        return;
    }
    float ss = 0.f;
    for (int j = threadIdx.x; j < d; j += 256) { float v = xr[j]; ss += v * v; }
    ss = block_sum(ss, red);
    float rs = 1.0f / sqrtf(ss / (float)d + eps);
    for (int j = threadIdx.x; j < d; j += 256) put_pair(o + j, d, xr[j] * rs * to_f(g[j]), split);
}
void k_rmsnorm(int dtype, const float* x, const void* g, void* out, int n, int d, float eps, hipStream_t s, int split,
               const int* rows, const void* g2, int n1) {
    if (n <= 0) return;
    if (dtype == 0)
        rmsnorm_kernel<float, float><<<n, 256, 0, s>>>(x, (const float*)g, (float*)out, d, eps, 0, rows, (const float*)g2, n1);
    else
        rmsnorm_kernel<f16_t, bf16_t><<<n, 256, 0, s>>>(x, (const bf16_t*)g, (f16_t*)out, d, eps, split, rows,
                                                        (const bf16_t*)g2, n1);
}

// ---------------------------------------------------------------- start of a decode step
// One block per row: the row's position and cache slot, its embedding into the residual stream, and -- norm_gain given
// -- the first layer's RMSNorm of it (split: as fp16 pairs).  One launch of about 5 us where there were three.
// A finished sequence is parked: position -1, which every consumer reads as "no cache slot, no
// attention, zeros" (the padding-row rule of the packed token lists), so it stops growing its cache.
template <typename T, typename TW>
__global__ __launch_bounds__(256) void step_start_kernel(const int* tok_in, const int* last_tok, const int* seq_len,
                                                         const int* finished, int* tok_pos, int* tok_slot, const TW* E, int d,
                                                         int V, float* x, int* errflag, const TW* norm_gain, T* h, float eps,
                                                         int split) {
    __shared__ float red[16];
    const int b = blockIdx.x;
    int id = tok_in ? tok_in[b] : last_tok[b];
    if (threadIdx.x == 0) {
        tok_pos[b] = finished[b] ? -1 : seq_len[b];
        tok_slot[b] = b;
        if (id < 0 || id >= V) atomicOr(errflag, 1);
    }
    id = min(max(id, 0), V - 1);
    const TW* row = E + (int64_t)id * d;
    float* xo = x + (int64_t)b * d;
    // d is a multiple of 64
    float ss = 0.f;
    for (int j = threadIdx.x * 4; j < d; j += 1024) {
        const floatx4 v = load4(row + j);
        *reinterpret_cast<floatx4*>(xo + j) = v;
        ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    }
    if (!norm_gain) return;
    ss = block_sum(ss, red);
    const float rs = 1.0f / sqrtf(ss / (float)d + eps);
    T* o = h + (int64_t)b * d * (split ? 2 : 1);
    for (int j = threadIdx.x * 4; j < d; j += 1024) {
        const floatx4 v = load4(row + j);
        put_pair4(o + j, d, make_float4(v[0], v[1], v[2], v[3]), rs, norm_gain + j, split);
    }
}
void k_step_start(int dtype, const int* tok_in, const int* last_tok, const int* seq_len, const int* finished, int* tok_pos,
                  int* tok_slot, const void* E, int d, int V, float* x, int* errflag, const void* norm_gain, void* h,
                  float eps, int split, int B, hipStream_t s) {
    if (B <= 0) return;
    if (dtype == 0)
        step_start_kernel<float, float><<<B, 256, 0, s>>>(tok_in, last_tok, seq_len, finished, tok_pos, tok_slot, (const float*)E,
                                                          d, V, x, errflag, (const float*)norm_gain, (float*)h, eps, split);
    else
        step_start_kernel<f16_t, bf16_t><<<B, 256, 0, s>>>(tok_in, last_tok, seq_len, finished, tok_pos, tok_slot,
                                                           (const bf16_t*)E, d, V, x, errflag, (const bf16_t*)norm_gain,
                                                           (f16_t*)h, eps, split);
}

// ---------------------------------------------------------------- sums and maxima over lanes by data-parallel-primitive moves
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// sum over 16 lanes, sum and maximum over the wave, every lane with the result
__device__ __forceinline__ float sum16(float v) {
    v = dpp_add<0xB1>(v);        // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);        // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);       // row_half_mirror
    return dpp_add<0x140>(v);    // row_mirror
}
__device__ __forceinline__ float sum64(float v) {
    v = sum16(v);
    v += __shfl_xor(v, 16, RL_WAVE);
    return v + __shfl_xor(v, 32, RL_WAVE);
}
template <int CTRL>
__device__ __forceinline__ int dpp_int(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false); }
template <int CTRL>
__device__ __forceinline__ float dpp_max(float v) { return fmaxf(v, __int_as_float(dpp_int<CTRL>(__float_as_int(v)))); }
__device__ __forceinline__ float max64(float v) {
    v = dpp_max<0xB1>(v);
    v = dpp_max<0x4E>(v);
    v = dpp_max<0x141>(v);
    v = dpp_max<0x140>(v);
    v = fmaxf(v, __shfl_xor(v, 16, RL_WAVE));
    return fmaxf(v, __shfl_xor(v, 32, RL_WAVE));
}

// ---------------------------------------------------------------- plain GEMM  C = A[M,K] * W[N,K]^T
// fp32 multiply-adds on the matrix cores (v_mfma_f32_16x16x4_f32), whatever the operand types.  A workgroup owns
// MT x NT tiles of 16 x 16 outputs; its eight waves split K between them -- wave w takes the 16-wide k chunks
// w, w + 8, ... -- and their sums are added in wave order through LDS.  The shapes this path serves are small (the fp32
// configuration's matrices are 0.25 - 4 MB, decode has a handful of rows): what bounds them is the latency of the
// loads and the number of waves in flight, not arithmetic, hence the K split inside the workgroup and tiles that
// shrink with the grid (k_gemm_simple).  A lane fetches four consecutive k of its row at once: as A and W use the
// same assignment of k to MFMA steps, any assignment gives the same contraction.  The order of the sums depends on K
// alone, so a row's bits do not depend on how many rows run beside it.
// Measured on the fp32 configuration (d 256, ffn 1024, vocab 4096; 4 rows, decode): 31 us (QKV, LM head), 39 us (gate /
// up) and 75 us (O, down) per GEMM with 64 x 64 tiles on plain multiply-adds (4 - 64 workgroups of one k loop), 3.7, 4.5
// and 4.8 us now, of which about 2 are the launch.
// NORM: A is the fp32 residual stream and its RMSNorm is part of the GEMM: with r = 1 / rms of the row,
// sum_k (x r g) W = r sum_k (x g) W, and the sum of squares comes from the values the lanes hold anyway.
struct PlainGemmArgs {
    const void *A, *W, *W2;
    int lda, M, N, K;
    float* outF;
    void* outT;
    int ldc;
    const void* gain;   // NORM
    float eps;
};
template <typename T, typename TW, int EPI, int MT, int NT, bool NORM>
__global__ __launch_bounds__(512) void gemm_plain_kernel(PlainGemmArgs a) {
    constexpr int NW = EPI == EPI_SWIGLU ? 2 : 1;        // weight matrices
    constexpr int U = MT * NT * NW == 1 ? 8 : MT * NT * NW == 2 ? 4 : 1;   // chunks requested at a time
    __shared__ float red[8][NW * NT * 256];
    __shared__ float ssq[8][MT * 16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, q4 = lane >> 4;
    const int m0 = blockIdx.y * (16 * MT), n0 = blockIdx.x * (16 * NT);
    const T* Ap[MT];
    const TW* Wp[NW][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i) Ap[i] = (const T*)a.A + (int64_t)min(m0 + i * 16 + r16, a.M - 1) * a.lda + q4 * 4;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int64_t o = (int64_t)min(n0 + j * 16 + r16, a.N - 1) * a.K + q4 * 4;
        Wp[0][j] = (const TW*)a.W + o;
        if (NW == 2) Wp[NW - 1][j] = (const TW*)a.W2 + o;
    }
    floatx4 acc[NW][MT][NT];
    float ss[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        ss[i] = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[w][i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    // the element this thread adds to, requested with the operands (one tile: a thread has at most one)
    float old = 0.f;
    if (EPI == EPI_RESID && MT * NT == 1 && threadIdx.x < 256) {
        const int l = threadIdx.x >> 2, m = m0 + 4 * (l >> 4) + (threadIdx.x & 3), n = n0 + (l & 15);
        old = a.outF[(int64_t)min(m, a.M - 1) * a.ldc + min(n, a.N - 1)];
    }
    const int nc = a.K / 16;                              // K is a multiple of 64
    for (int c0 = wave; c0 < nc; c0 += 8 * U) {
        floatx4 af[U][MT], wf[U][NW][NT], gf[NORM ? U : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(c0 + 8 * u, nc - 1) * 16;   // past the end: the last chunk again, not used
#pragma unroll
            for (int i = 0; i < MT; ++i) af[u][i] = load4(Ap[i] + k);
            if (NORM) gf[NORM ? u : 0] = load4((const TW*)a.gain + k + q4 * 4);
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int j = 0; j < NT; ++j) wf[u][w][j] = load4(Wp[w][j] + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c0 + 8 * u >= nc) break;                  // wave-uniform
            if (NORM) {
#pragma unroll
                for (int i = 0; i < MT; ++i) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) ss[i] += af[u][i][e] * af[u][i][e];
                    af[u][i] *= gf[NORM ? u : 0];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int w = 0; w < NW; ++w)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < NT; ++j)
                            acc[w][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[u][i][e], wf[u][w][j][e], acc[w][i][j], 0, 0, 0);
        }
    }
    if (NORM) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            float s = ss[i];                              // this lane's share of row i * 16 + r16
            s += __shfl_xor(s, 16, RL_WAVE);
            s += __shfl_xor(s, 32, RL_WAVE);
            if (q4 == 0) ssq[wave][i * 16 + r16] = s;
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        if (i > 0) __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int j = 0; j < NT; ++j) *reinterpret_cast<floatx4*>(&red[wave][(w * NT + j) * 256 + lane * 4]) = acc[w][i][j];
        __syncthreads();
        for (int e = threadIdx.x; e < NT * 256; e += 512) {
            const int l = (e & 255) >> 2, row = i * 16 + 4 * (l >> 4) + (e & 3), m = m0 + row, n = n0 + (e >> 8) * 16 + (l & 15);
            if (m >= a.M || n >= a.N) continue;
            float v = 0.f, u = 0.f, s = 0.f;
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                v += red[w][e];
                if (NW == 2) u += red[w][(NW - 1) * NT * 256 + e];
                if (NORM) s += ssq[w][row];
            }
            if (NORM) {
                const float rs = 1.0f / sqrtf(s / (float)a.K + a.eps);
                v *= rs;
                u *= rs;
            }
            const int64_t o = (int64_t)m * a.ldc + n;
            if (EPI == EPI_STORE_F32) a.outF[o] = v;
            else if (EPI == EPI_RESID) a.outF[o] = (MT * NT == 1 ? old : a.outF[o]) + v;
            else ((T*)a.outT)[o] = from_f<T>(v / (1.0f + __expf(-v)) * u);
        }
    }
}
template <typename T, typename TW, int EPI, bool NORM>
static void gemm_plain_t(const PlainGemmArgs& a, hipStream_t s) {
    // The largest tile that still gives the 256 compute units two workgroups each: a bigger tile reads its operands
    // fewer times, but a grid that leaves units idle costs more than that.
    auto wgs = [&](int mt, int nt) { return (int64_t)((a.M + 16 * mt - 1) / (16 * mt)) * ((a.N + 16 * nt - 1) / (16 * nt)); };
    if (wgs(4, 4) >= 512) gemm_plain_kernel<T, TW, EPI, 4, 4, NORM><<<dim3((a.N + 63) / 64, (a.M + 63) / 64), 512, 0, s>>>(a);
    else if (wgs(2, 2) >= 512) gemm_plain_kernel<T, TW, EPI, 2, 2, NORM><<<dim3((a.N + 31) / 32, (a.M + 31) / 32), 512, 0, s>>>(a);
    else gemm_plain_kernel<T, TW, EPI, 1, 1, NORM><<<dim3((a.N + 15) / 16, (a.M + 15) / 16), 512, 0, s>>>(a);
}
template <typename T, typename TW>
static void gemm_simple_t(int epi, const PlainGemmArgs& a, hipStream_t s) {
    switch (epi) {
        case EPI_STORE_F32: gemm_plain_t<T, TW, EPI_STORE_F32, false>(a, s); break;
        case EPI_RESID: gemm_plain_t<T, TW, EPI_RESID, false>(a, s); break;
        default: gemm_plain_t<T, TW, EPI_SWIGLU, false>(a, s); break;
    }
}
void k_gemm_simple(int dtype, int epi, const void* A, int lda, const void* W, const void* W2, int M, int N, int K,
                   float* outF, void* outT, int ldc, hipStream_t s) {
    if (M <= 0 || N <= 0) return;
    const PlainGemmArgs a{A, W, W2, lda, M, N, K, outF, outT, ldc, nullptr, 0.f};
    if (dtype == 0) gemm_simple_t<float, float>(epi, a, s);
    else gemm_simple_t<f16_t, bf16_t>(epi, a, s);
}
void k_gemm_norm_f32(int epi, const float* x, const float* gain, float eps, const float* W, const float* W2, int M, int N,
                     int K, float* out, int ldc, hipStream_t s) {
    if (M <= 0 || N <= 0) return;
    const PlainGemmArgs a{x, W, W2, K, M, N, K, out, out, ldc, gain, eps};
    if (epi == EPI_SWIGLU) gemm_plain_t<float, float, EPI_SWIGLU, true>(a, s);
    else gemm_plain_t<float, float, EPI_STORE_F32, true>(a, s);
}

// outF += A W^T for at most 8 rows, fp32 (the down projection of a decode step of few rows).  The tiles above give it one
// workgroup per 16 columns, whose eight waves share four SIMDs and multiply padding rows; here four columns have a workgroup
// and its four waves share K, so that every operand is requested at once from four times as many CUs.  16 lanes per column,
// lane l taking k = 64 j + 4 l .. + 3.  Rows are independent: the rows of a call do not change a row's sums.
// 256 columns, K = 1024, in a graph of such launches: 4 rows 4.3 -> 2.7 us, 8 rows 4.7 -> 3.5.
template <int NM>
__global__ __launch_bounds__(256) void gemm_rows_kernel(PlainGemmArgs a) {
    constexpr int U = NM == 4 ? 4 : 2;                               // chunks of 64 k at a time
    __shared__ float red[4][NM][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, q4 = lane >> 4;
    const int n = min((int)blockIdx.x * 4 + q4, a.N - 1);            // N is a multiple of 4
    const float* const A = (const float*)a.A + l16 * 4;
    const float* const W = (const float*)a.W + (int64_t)n * a.K + l16 * 4;
    // lane l16 = row m of the first wave puts out column n; what it adds to is requested with the operands
    float* const o = a.outF + (int64_t)min(l16, a.M - 1) * a.ldc + n;
    const float old = *o;
    float acc[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[m] = 0.f;
    const int nc = a.K / 64, per = (nc + 3) / 4, cend = min(nc, (wave + 1) * per);         // K is a multiple of 64
    for (int c0 = wave * per; c0 < cend; c0 += U) {
        floatx4 xf[U][NM], wf[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(c0 + u, cend - 1) * 64;                // past the end: the last chunk again, not used
            wf[u] = load4(W + k);
#pragma unroll
            for (int m = 0; m < NM; ++m) xf[u][m] = load4(A + (int64_t)min(m, a.M - 1) * a.lda + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c0 + u >= cend) break;                               // wave-uniform
#pragma unroll
            for (int m = 0; m < NM; ++m)
                acc[m] += xf[u][m][0] * wf[u][0] + xf[u][m][1] * wf[u][1] + xf[u][m][2] * wf[u][2] + xf[u][m][3] * wf[u][3];
        }
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        const float t = sum16(acc[m]);
        if (l16 == m) red[wave][m][q4] = t;
    }
    __syncthreads();
    if (wave == 0 && l16 < a.M) *o = old + (((red[0][l16][q4] + red[1][l16][q4]) + red[2][l16][q4]) + red[3][l16][q4]);
}
// From the context's limit of rows, never from the rows of a call.  One round of loads (K up to 256) is as fast on the tiles; on
// wide matrices the rows, read again by every four columns, weigh more than the weights.  8 rows, K = N = 512 / 1024 / 2048 /
// 4096: tiles 3.3 / 4.8 / 8.8 / 16 us, this 2.9 / 3.8 / 6.5 / 21; 4 rows 3.1 / 4.3 / 8.7 / 16 and 2.4 / 2.9 / 4.5 / 12.
bool k_gemm_rows_supported(int N, int K, int max_batch) { return max_batch <= 8 && K > 256 && N <= 2048 && N % 4 == 0; }
void k_gemm_rows_f32(const float* A, int lda, const float* W, int M, int N, int K, float* out, int ldc, hipStream_t s) {
    if (M <= 0 || M > 8 || N <= 0) return;                           // callers check first
    const PlainGemmArgs a{A, W, nullptr, lda, M, N, K, out, nullptr, ldc, nullptr, 0.f};
    if (M <= 4) gemm_rows_kernel<4><<<N / 4, 256, 0, s>>>(a);
    else gemm_rows_kernel<8><<<N / 4, 256, 0, s>>>(a);
}

// ---------------------------------------------------------------- RoPE + split + KV append
// Plain path, whole sequences: qkv fp32 [n, (Hq+2Hkv) hd] -> rotated q (T) [n, Hq hd]; rotated k and plain v to the
// contiguous buffers and to the page slot of (slot, pos) (optional).
template <typename T>
__global__ __launch_bounds__(256) void rope_append_kernel(const float* qkv, const int* tok_pos, const int* tok_slot,
                                                          const float2* rope, T* q_out, T* k_out, T* v_out, T* pool,
                                                          int layer, KvGeom geo, const int* bt, int mpps, int Hq) {
    const int n = blockIdx.x, hd = geo.hd, half = hd / 2, Hkv = geo.Hkv;
    const int pos = tok_pos[n];
    const float* row = qkv + (int64_t)n * (Hq + 2 * Hkv) * hd;
    if (pos < 0) {   // padding row: zero query, no key or value
        for (int i = threadIdx.x; i < Hq * hd; i += 256) q_out[(int64_t)n * Hq * hd + i] = from_f<T>(0.f);
        for (int i = threadIdx.x; i < Hkv * hd; i += 256) k_out[(int64_t)n * Hkv * hd + i] = from_f<T>(0.f);
        for (int i = threadIdx.x; i < Hkv * hd; i += 256) v_out[(int64_t)n * Hkv * hd + i] = from_f<T>(0.f);
        return;
    }
    const float2* rt = rope + (int64_t)pos * half;
    int64_t page = 0;
    int slot_tok = 0;
    if (pool) {
        page = bt[(int64_t)tok_slot[n] * mpps + pos / geo.PT];
        slot_tok = pos % geo.PT;
    }
    // q heads
    for (int i = threadIdx.x; i < Hq * half; i += 256) {
        int h = i / half, j = i % half;
        float a = row[h * hd + j], b = row[h * hd + j + half];
        float2 cs = rt[j];
        T* o = q_out + (int64_t)n * Hq * hd + h * hd;
        o[j] = from_f<T>(a * cs.x - b * cs.y);
        o[j + half] = from_f<T>(b * cs.x + a * cs.y);
    }
    // k heads
    const float* krow = row + Hq * hd;
    for (int i = threadIdx.x; i < Hkv * half; i += 256) {
        int g = i / half, j = i % half;
        float a = krow[g * hd + j], b = krow[g * hd + j + half];
        float2 cs = rt[j];
        T r0 = from_f<T>(a * cs.x - b * cs.y), r1 = from_f<T>(b * cs.x + a * cs.y);
        T* o = k_out + (int64_t)n * Hkv * hd + g * hd;
        o[j] = r0; o[j + half] = r1;
        if (pool) {
            pool[geo.k_off(layer, page, g, slot_tok, j)] = r0;
            pool[geo.k_off(layer, page, g, slot_tok, j + half)] = r1;
        }
    }
    // v heads
    const float* vrow = row + (Hq + Hkv) * hd;
    for (int i = threadIdx.x; i < Hkv * hd; i += 256) {
        int g = i / hd, dd = i % hd;
        T v = from_f<T>(vrow[i]);
        v_out[(int64_t)n * Hkv * hd + i] = v;
        if (pool) pool[geo.v_off(layer, page, g, slot_tok, dd)] = v;
    }
}
void k_rope_append(int dtype, const float* qkv, int n, const int* tok_pos, const int* tok_slot, const float2* rope,
                   void* q_out, void* k_out, void* v_out, void* pool, int layer, KvGeom geo, const int* block_table,
                   int mpps, int Hq, hipStream_t s) {
    if (n <= 0) return;
    if (dtype == 0)
        rope_append_kernel<float><<<n, 256, 0, s>>>(qkv, tok_pos, tok_slot, rope, (float*)q_out, (float*)k_out, (float*)v_out,
                                                    (float*)pool, layer, geo, block_table, mpps, Hq);
    else
        rope_append_kernel<f16_t><<<n, 256, 0, s>>>(qkv, tok_pos, tok_slot, rope, (f16_t*)q_out, (f16_t*)k_out, (f16_t*)v_out,
                                                    (f16_t*)pool, layer, geo, block_table, mpps, Hq);
}

#define RL_MAX_SPLITS 16
// Decode variant: the qkv row arrives as nsplit split-K partial rows.  One block of 1024 threads
// per token; a thread owns (column j, column j + hd/2) pairs and requests every partial of a pair
// before summing them in split order.  Writes rotated q, and k / v into the page slot.
template <typename T>
__global__ __launch_bounds__(1024) void rope_append_split_kernel(const float* part, int nsplit, int64_t split_stride,
                                                                 const int* tok_pos, const int* tok_slot,
                                                                 const float2* rope, T* q_out, T* pool, int layer,
                                                                 KvGeom geo, const int* bt, int mpps, int Hq,
                                                                 int split, int layer_lo) {
    const int n = blockIdx.x, hd = geo.hd, half = hd / 2, Hkv = geo.Hkv;
    const int pos = tok_pos[n];
    const int width = (Hq + 2 * Hkv) * hd;
    const float* row = part + (int64_t)n * width;
    // split: q rows are fp16 pairs [Hq hd hi | Hq hd lo]; the lo planes of k and v go to layer_lo of the pool
    const int qw = (split ? 2 : 1) * Hq * hd;
    const int64_t lo_off = split ? (int64_t)(layer_lo - layer) * geo.layer_elems() : 0;
    if (pos < 0) {   // parked row: zero query, nothing appended to the cache
        for (int i = threadIdx.x; i < qw; i += 1024) q_out[(int64_t)n * qw + i] = from_f<T>(0.f);
        return;
    }
    const float2* rt = rope + (int64_t)pos * half;
    const int64_t page = bt[(int64_t)tok_slot[n] * mpps + pos / geo.PT];
    const int st = pos % geo.PT;
    // a thread owns four consecutive pairs (j .. j+3, and their partners j + hd/2 ..): 16-byte loads of every
    // split's partials, all requested before the first add
    const int nquads = (Hq + 2 * Hkv) * half / 4;
    for (int i = threadIdx.x; i < nquads; i += 1024) {
        const int head = i / (half / 4), j = (i % (half / 4)) * 4;
        const int c0 = head * hd + j;
        float a[4] = {0.f, 0.f, 0.f, 0.f}, b[4] = {0.f, 0.f, 0.f, 0.f};
        // eight splits at a time (their loads all in flight together), summed in split order
        for (int s0 = 0; s0 < nsplit; s0 += 8) {
            float4 p0[8], p1[8];
#pragma unroll
            for (int sp = 0; sp < 8; ++sp)
                if (s0 + sp < nsplit) {
                    p0[sp] = *reinterpret_cast<const float4*>(row + (s0 + sp) * split_stride + c0);
                    p1[sp] = *reinterpret_cast<const float4*>(row + (s0 + sp) * split_stride + c0 + half);
                }
#pragma unroll
            for (int sp = 0; sp < 8; ++sp)
                if (s0 + sp < nsplit) {
                    a[0] += p0[sp].x; a[1] += p0[sp].y; a[2] += p0[sp].z; a[3] += p0[sp].w;
                    b[0] += p1[sp].x; b[1] += p1[sp].y; b[2] += p1[sp].z; b[3] += p1[sp].w;
                }
        }
        if (head < Hq + Hkv) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float2 cs = rt[j + t];
                const float r0 = a[t] * cs.x - b[t] * cs.y, r1 = b[t] * cs.x + a[t] * cs.y;
                a[t] = r0; b[t] = r1;
            }
        }
        if (head < Hq) {
            T* o = q_out + (int64_t)n * qw + head * hd + j;
#pragma unroll
            for (int t = 0; t < 4; ++t) { put_pair(o + t, Hq * hd, a[t], split); put_pair(o + half + t, Hq * hd, b[t], split); }
        } else if (head < Hq + Hkv) {
            const int g = head - Hq;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                put_pair(pool + geo.k_off(layer, page, g, st, j + t), lo_off, a[t], split);
                put_pair(pool + geo.k_off(layer, page, g, st, j + t + half), lo_off, b[t], split);
            }
        } else {
            const int g = head - Hq - Hkv;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                put_pair(pool + geo.v_off(layer, page, g, st, j + t), lo_off, a[t], split);
                put_pair(pool + geo.v_off(layer, page, g, st, j + t + half), lo_off, b[t], split);
            }
        }
    }
}
void k_rope_append_split(int dtype, const float* part, int nsplit, int64_t split_stride, int n, const int* tok_pos,
                         const int* tok_slot, const float2* rope, void* q_out, void* pool, int layer, KvGeom geo,
                         const int* block_table, int mpps, int Hq, hipStream_t s, int split, int layer_lo) {
    if (n <= 0) return;
    if (dtype == 0)
        rope_append_split_kernel<float><<<n, 1024, 0, s>>>(part, nsplit, split_stride, tok_pos, tok_slot, rope,
                                                           (float*)q_out, (float*)pool, layer, geo, block_table, mpps, Hq, 0, layer);
    else
        rope_append_split_kernel<f16_t><<<n, 1024, 0, s>>>(part, nsplit, split_stride, tok_pos, tok_slot, rope,
                                                           (f16_t*)q_out, (f16_t*)pool, layer, geo, block_table, mpps, Hq,
                                                           split, layer_lo);
}

// ---------------------------------------------------------------- split-K reduce + residual add + RMSNorm
// x[n,:] += sum_s part[s][n,:] (split order);  out[n,:] = RMSNorm(x[n,:]; g).  One block per row, as many threads as the
// row has groups of four columns (at most 1024).  A chain of one memory round trip, one reduction and one store around
// which a launch is built (an empty one takes 1.7 us): the row, every split's partial and the gains are requested at once,
// without branches (a split past the last re-reads the last), and 16 lanes reduce by data-parallel-primitive moves.  Behind
// a GEMM it adds 3.4 us to a step (32 rows of 2048, 4 or 8 splits).  Against 1024 threads for every row and a branch per
// split: 200 steps of the 1B shape, 32 rows, 197.6 -> 196.1 ms.
template <typename T, typename TW, int NSP, int PER>
__global__ __launch_bounds__(1024) void resid_norm_kernel(float* x, const float* part, int nsplit, int64_t split_stride,
                                                          const TW* g, T* out, int d, float eps, int split) {
    __shared__ float red[16];
    const int n = blockIdx.x;
    float* xr = x + (int64_t)n * d;
    const float* pr = part + (int64_t)n * d;
    float4 v[PER], p[PER][NSP];
    Gain4<TW> gain[PER];
#pragma unroll
    for (int it = 0; it < PER; ++it) {
        const int j = min((int)(it * blockDim.x + threadIdx.x) * 4, d - 4);
        v[it] = *reinterpret_cast<const float4*>(xr + j);
#pragma unroll
        for (int sp = 0; sp < NSP; ++sp) p[it][sp] = *reinterpret_cast<const float4*>(pr + min(sp, nsplit - 1) * split_stride + j);
        gain[it].load(g + j);
    }
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < PER; ++it) {
        const int j = (it * blockDim.x + threadIdx.x) * 4;
#pragma unroll
        for (int sp = 0; sp < NSP; ++sp)
            if (sp < nsplit) { v[it].x += p[it][sp].x; v[it].y += p[it][sp].y; v[it].z += p[it][sp].z; v[it].w += p[it][sp].w; }
        if (j < d) {
            *reinterpret_cast<float4*>(xr + j) = v[it];
            ss += v[it].x * v[it].x + v[it].y * v[it].y + v[it].z * v[it].z + v[it].w * v[it].w;
        }
    }
    ss = sum64(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float t = 0.f;
    for (int w = 0; w < (int)blockDim.x / 64; ++w) t += red[w];
    const float rs = 1.0f / sqrtf(t / (float)d + eps);
    T* o = out + (int64_t)n * d * (split ? 2 : 1);   // split: [d values rounded to T | d remainders]
#pragma unroll
    for (int it = 0; it < PER; ++it) {
        const int j = (it * blockDim.x + threadIdx.x) * 4;
        if (j < d) put_pair4(o + j, d, v[it], rs, gain[it], split);
    }
}
template <typename T, typename TW, int NSP>
static void launch_resid_norm(float* x, const float* part, int nsplit, int64_t split_stride, const TW* g, T* out, int n, int d,
                              float eps, hipStream_t s, int split) {
    const int threads = d >= 4096 ? 1024 : (d / 4 + 63) / 64 * 64;
    if (d <= 4096) resid_norm_kernel<T, TW, NSP, 1><<<n, threads, 0, s>>>(x, part, nsplit, split_stride, g, out, d, eps, split);
    else resid_norm_kernel<T, TW, NSP, 2><<<n, threads, 0, s>>>(x, part, nsplit, split_stride, g, out, d, eps, split);
}
// d must be a multiple of 4 and at most 8192; 1 <= nsplit <= RL_MAX_SPLITS.
void k_resid_norm(float* x, const float* part, int nsplit, int64_t split_stride, const void* g, void* out, int n, int d,
                  float eps, hipStream_t s, int split) {
    if (n <= 0) return;
    const bf16_t* gw = (const bf16_t*)g;
    f16_t* o = (f16_t*)out;
    if (nsplit <= 4) launch_resid_norm<f16_t, bf16_t, 4>(x, part, nsplit, split_stride, gw, o, n, d, eps, s, split);
    else if (nsplit <= 8) launch_resid_norm<f16_t, bf16_t, 8>(x, part, nsplit, split_stride, gw, o, n, d, eps, s, split);
    else launch_resid_norm<f16_t, bf16_t, RL_MAX_SPLITS>(x, part, nsplit, split_stride, gw, o, n, d, eps, s, split);
}

// ---------------------------------------------------------------- plain attention
// One block per (query token, query head).  Keys 0..pos of the query's own sequence,
// read either from contiguous [tokens, Hkv, hd] buffers (the sequence's tokens are
// consecutive, so key m sits at row n - pos + m) or from the paged pool.
// DEC (decode, paged, one row per cache slot): q, k and v of the new token come straight from the QKV projection's
// fp32 row.  The block rotates its own query head and its kv head's new key, rounds all three to T, and uses the new
// key and value from LDS; the group's first head appends them to the page.  One launch instead of two per layer: at
// the sizes this path serves each of them is little more than its launch (4.7 + 8.5 us before, 7.4 us now; 4 rows, 48 keys).
template <typename T, bool DEC>
__global__ __launch_bounds__(256) void attn_simple_kernel(const T* q, const float* qkv, const float2* rope, const T* kc,
                                                          const T* vc, T* pool, int layer, KvGeom geo, const int* bt,
                                                          int mpps, const int* tok_pos, const int* tok_slot, T* out, int Hq) {
    extern __shared__ __attribute__((aligned(16))) float sm[];
    const int hd = geo.hd, Hkv = geo.Hkv, half = hd / 2, G = Hq / Hkv;
    const int n = blockIdx.x, h = blockIdx.y, g = h / G;
    const int pos = tok_pos[n], ctx = pos + 1;
    if (ctx <= 0) {            // parked row (position -1): no keys, zeros
        if (threadIdx.x < hd) out[((int64_t)n * Hq + h) * hd + threadIdx.x] = from_f<T>(0.f);
        return;
    }
    float* qs = sm;            // [hd]
    float* red = sm + hd;      // [16]
    float* part = red + 16;    // [256]
    float* sc = part + 256;    // [ctx]
    float* kn = part;          // [hd] DEC: the new token's key and value, as the cache will hold them (2 hd <= 256; the
    float* vn = part + hd;     // [hd] partial sums come after their last use)
    const int* btr = DEC ? bt + (int64_t)tok_slot[n] * mpps : nullptr;
    if (DEC) {
        const float* row = qkv + (int64_t)n * (Hq + 2 * Hkv) * hd;
        if (threadIdx.x < 2 * half) {                       // first the query's pairs, then the key's
            const int j = threadIdx.x % half;
            const float* r = row + (threadIdx.x < half ? h : Hq + g) * hd;
            float* o = threadIdx.x < half ? qs : kn;
            const float2 cs = rope[(int64_t)pos * half + j];
            o[j] = to_f(from_f<T>(r[j] * cs.x - r[j + half] * cs.y));
            o[j + half] = to_f(from_f<T>(r[j + half] * cs.x + r[j] * cs.y));
        }
        if (threadIdx.x < hd) vn[threadIdx.x] = to_f(from_f<T>(row[(Hq + Hkv + g) * hd + threadIdx.x]));
    } else {
        for (int j = threadIdx.x; j < hd; j += 256) qs[j] = to_f(q[((int64_t)n * Hq + h) * hd + j]);
    }
    __syncthreads();
    const int dd = threadIdx.x % hd, grp = threadIdx.x / hd, ngrp = 256 / hd;
    const float k_new = DEC ? kn[dd] : 0.f, v_new = DEC ? vn[dd] : 0.f;
    const float scale = 1.0f / sqrtf((float)hd);
    float lmax = -INFINITY;
    // four threads per key: a context of a few dozen keys would otherwise leave most of the block idle behind one
    // thread's chain of loads
    const int sub = threadIdx.x & 3;
    for (int m = threadIdx.x >> 2; m < ctx; m += 64) {
        const T* kr = DEC ? pool + geo.k_off(layer, btr[m / geo.PT], g, m % geo.PT, 0)
                          : kc + ((int64_t)(n - pos + m) * Hkv + g) * hd;
        const bool fresh = DEC && m == pos;                 // its page slot may not be written yet: LDS holds it
        float dot = 0.f;
#pragma unroll 4
        for (int j = sub * 4; j < hd; j += 16) {
            const floatx4 kv = fresh ? *reinterpret_cast<const floatx4*>(kn + j) : load4(kr + j);
            const floatx4 qv = *reinterpret_cast<const floatx4*>(qs + j);
            dot += qv[0] * kv[0] + qv[1] * kv[1] + qv[2] * kv[2] + qv[3] * kv[3];
        }
        dot += __shfl_xor(dot, 1, RL_WAVE);
        dot += __shfl_xor(dot, 2, RL_WAVE);
        dot *= scale;
        if (sub == 0) sc[m] = dot;
        lmax = fmaxf(lmax, dot);
    }
    float mx = block_max(lmax, red);
    float ls = 0.f;
    for (int m = threadIdx.x; m < ctx; m += 256) { float e = __expf(sc[m] - mx); sc[m] = e; ls += e; }
    float tot = block_sum(ls, red);   // has barriers: sc[] visible afterwards
    float acc = 0.f;
    if (DEC) {
        // V pages are dim-major: four tokens of a dimension are one load
        for (int m = grp * 4; m < pos; m += ngrp * 4) {
            const T* vp = pool + geo.v_off(layer, btr[m / geo.PT], g, m % geo.PT, dd);
            if (m + 4 <= pos) {
                const floatx4 v = load4(vp);
                acc += sc[m] * v[0] + sc[m + 1] * v[1] + sc[m + 2] * v[2] + sc[m + 3] * v[3];
            } else {
                for (int i = 0; m + i < pos; ++i) acc += sc[m + i] * to_f(vp[i]);
            }
        }
        if (grp == 0) acc += sc[pos] * v_new;
    } else {
        for (int m = grp; m < ctx; m += ngrp) acc += sc[m] * to_f(vc[((int64_t)(n - pos + m) * Hkv + g) * hd + dd]);
    }
    part[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < hd) {
        float o = 0.f;
        for (int i = 0; i < ngrp; ++i) o += part[i * hd + threadIdx.x];
        out[((int64_t)n * Hq + h) * hd + threadIdx.x] = from_f<T>(o / tot);
        if (DEC && h == g * G) {
            pool[geo.k_off(layer, btr[pos / geo.PT], g, pos % geo.PT, threadIdx.x)] = from_f<T>(k_new);
            pool[geo.v_off(layer, btr[pos / geo.PT], g, pos % geo.PT, threadIdx.x)] = from_f<T>(v_new);
        }
    }
}
size_t k_attn_simple_lds(int hd, int max_ctx) { return (size_t)(hd + 16 + 256 + max_ctx) * sizeof(float); }
void k_attn_simple(int dtype, const void* q, const void* kc, const void* vc, const int* tok_pos, void* out, int n, int Hq,
                   int Hkv, int hd, int max_ctx, hipStream_t s) {
    if (n <= 0) return;
    const size_t lds = k_attn_simple_lds(hd, max_ctx);
    const KvGeom geo{Hkv, hd, 16, 0};
    dim3 grid(n, Hq);
    if (dtype == 0)
        attn_simple_kernel<float, false><<<grid, 256, lds, s>>>((const float*)q, nullptr, nullptr, (const float*)kc,
                                                                (const float*)vc, nullptr, 0, geo, nullptr, 0, tok_pos,
                                                                nullptr, (float*)out, Hq);
    else
        attn_simple_kernel<f16_t, false><<<grid, 256, lds, s>>>((const f16_t*)q, nullptr, nullptr, (const f16_t*)kc,
                                                                (const f16_t*)vc, nullptr, 0, geo, nullptr, 0, tok_pos,
                                                                nullptr, (f16_t*)out, Hq);
}
void k_attn_simple_decode(int dtype, const float* qkv, const float2* rope, void* pool, int layer, KvGeom geo,
                          const int* block_table, int mpps, const int* tok_pos, const int* tok_slot, void* out, int n,
                          int Hq, int max_ctx, hipStream_t s) {
    if (n <= 0) return;
    const size_t lds = k_attn_simple_lds(geo.hd, max_ctx);
    dim3 grid(n, Hq);
    if (dtype == 0)
        attn_simple_kernel<float, true><<<grid, 256, lds, s>>>(nullptr, qkv, rope, nullptr, nullptr, (float*)pool, layer, geo,
                                                               block_table, mpps, tok_pos, tok_slot, (float*)out, Hq);
    else
        attn_simple_kernel<f16_t, true><<<grid, 256, lds, s>>>(nullptr, qkv, rope, nullptr, nullptr, (f16_t*)pool, layer, geo,
                                                               block_table, mpps, tok_pos, tok_slot, (f16_t*)out, Hq);
}

// Everything of a plain fp32 decode layer up to the attention's output in one launch: RMSNorm, the QKV projection of this row
// and kv head, rotation, append and attention; in the first layer also the start of the step (position, embedding).  One block
// of 16 waves per (row, kv head).  At the sizes this path serves a launch costs as much as what it does (an empty one takes
// 1.6 us behind another), so the projection is repeated per row, a dot product of 16-byte pieces per wave and column, and the
// pages' first keys and values are requested before it: they wait for the position and a page number, not for the query.
// 4 rows, 48 keys, d 256, in a step's trace: 3.8 + 7.4 us for the two kernels before (and 2.2 for the step's start), 7.4 now.
// A row's sums depend on the shape and its own length only.
struct PlainFrontArgs {
    const float *x, *gain, *W;
    float eps;
    int d;
    const float2* rope;
    float* pool;
    int layer;
    KvGeom geo;
    const int *bt, *tok_pos;
    int mpps, Hq, ctx_cap;
    float* out;
    PlainStart start;             // .E: first layer
};
template <int HD, int G>
__global__ __launch_bounds__(1024) void plain_front_kernel(PlainFrontArgs a) {
    constexpr int HALF = HD / 2, NC = (G + 2) * HD;
    constexpr int CG = NC / 64, CB = CG % 3 == 0 ? 3 : 2;              // groups of four columns per wave: of all, at a time
    constexpr int TPK = HD / 4, KPP = 1024 / TPK, PARTS = 1024 / HD;   // threads per key, keys per pass; groups of 4 tokens per pass
    static_assert(KPP == PARTS * 4 && CG % CB == 0, "keys and values advance together");
    extern __shared__ __attribute__((aligned(16))) float sm[];
    float* const qkv = sm;                          // [G + 2][HD]: queries, key, value
    float* const part = qkv + NC;                   // [G][PARTS][HD]
    float* const sm_l = part + G * 1024;            // [4]
    float* const sc = sm_l + 4;                     // [G][ctx_cap]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = blockIdx.x, g = blockIdx.y, Hkv = a.geo.Hkv, d = a.d;
    const int l16 = lane & 15, q4 = lane >> 4;
    const int km = tid / TPK, sub = tid % TPK, dd = tid % HD, pt = tid / HD;
    const int* const bt = a.bt + (int64_t)b * a.mpps;
    // entries past the last page are never used
    const int page_k = bt[min(km / 16, a.mpps - 1)], page_v = bt[min(pt / 4, a.mpps - 1)];
    // Projection: 16 lanes per column, lane l16 taking k = 64 j + 4 l16 .. + 3; four columns per wave and step, 256 k at a
    // time.  The first weights are requested before anything that is waited for.
    const float* wrow[CG];
#pragma unroll
    for (int i = 0; i < CG; ++i) {
        const int c = (wave * CG + i) * 4 + q4, hh = c / HD;
        wrow[i] = a.W + (int64_t)((hh < G ? g * G + hh : hh == G ? a.Hq + g : a.Hq + Hkv + g) * HD + c % HD) * d + l16 * 4;
    }
    floatx4 w[CB][4];
    auto request = [&](int k0, int c0) {
#pragma unroll
        for (int i = 0; i < CB; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) w[i][j] = load4(wrow[c0 + i] + min(k0 + j * 64, d - 64));
    };
    request(0, 0);
    int pos;
    const float* x;
    if (a.start.E) {
        pos = a.start.finished[b] ? -1 : a.start.seq_len[b];
        const int id = a.start.tok_in ? a.start.tok_in[b] : a.start.last_tok[b];
        x = a.start.E + (int64_t)min(max(id, 0), a.start.V - 1) * d;
        if (g == 0) {
            if (tid == 0) {
                a.start.pos_out[b] = pos;
                a.start.slot_out[b] = b;
                if (id < 0 || id >= a.start.V) atomicOr(a.start.errflag, 1);
            }
            for (int j = tid; j < d; j += 1024) a.start.x_out[(int64_t)b * d + j] = x[j];
        }
    } else {
        pos = a.tok_pos[b];
        x = a.x + (int64_t)b * d;
    }
    floatx4 xv[4], gv[4];
    auto request_x = [&](int kb) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = min(kb + j * 64, d - 64) + l16 * 4;
            xv[j] = load4(x + k);
            gv[j] = load4(a.gain + k);
        }
    };
    request_x(0);
    const int ctx = pos + 1;
    float* const out = a.out + ((int64_t)b * a.Hq + g * G) * HD;
    if (ctx <= 0) {                                 // parked row: no keys, zeros
        if (tid < G * HD) out[tid] = 0.f;
        return;
    }
    floatx4 k0 = {0.f, 0.f, 0.f, 0.f}, v0 = {0.f, 0.f, 0.f, 0.f};
    if (km < pos) k0 = load4(a.pool + a.geo.k_off(a.layer, page_k, g, km % 16, sub * 4));
    if (pt * 4 < pos) v0 = load4(a.pool + a.geo.v_off(a.layer, page_v, g, pt * 4 % 16, dd));
    const float2 cs = a.rope[(int64_t)pos * HALF + tid % HALF];
    const int page_new = bt[pos / 16];
    float acc[CG], ss = 0.f;
#pragma unroll
    for (int i = 0; i < CG; ++i) acc[i] = 0.f;
    for (int kb = 0; kb < d; kb += 256) {
        if (kb > 0) request_x(kb);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (kb + j * 64 >= d) xv[j] = floatx4{0.f, 0.f, 0.f, 0.f};
            ss += xv[j][0] * xv[j][0] + xv[j][1] * xv[j][1] + xv[j][2] * xv[j][2] + xv[j][3] * xv[j][3];
            xv[j] *= gv[j];
        }
#pragma unroll
        for (int c0 = 0; c0 < CG; c0 += CB) {
            if (kb > 0 || c0 > 0) request(kb, c0);
#pragma unroll
            for (int i = 0; i < CB; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[c0 + i] += xv[j][0] * w[i][j][0] + xv[j][1] * w[i][j][1] + xv[j][2] * w[i][j][2] + xv[j][3] * w[i][j][3];
        }
    }
    const float rs = 1.0f / sqrtf(sum16(ss) / (float)d + a.eps);
#pragma unroll
    for (int i = 0; i < CG; ++i) {
        const float v = sum16(acc[i]) * rs;
        if (l16 == 0) qkv[(wave * CG + i) * 4 + q4] = v;
    }
    __syncthreads();
    if (tid < (G + 1) * HALF) {                     // queries and the key
        float* const p = qkv + tid / HALF * HD + tid % HALF;
        const float p0 = p[0], p1 = p[HALF];
        p[0] = p0 * cs.x - p1 * cs.y;
        p[HALF] = p1 * cs.x + p0 * cs.y;
    }
    __syncthreads();
    const float* const k_new = qkv + G * HD;
    const float* const v_new = qkv + (G + 1) * HD;
    if (tid < HD) {
        a.pool[a.geo.k_off(a.layer, page_new, g, pos % 16, tid)] = k_new[tid];
        a.pool[a.geo.v_off(a.layer, page_new, g, pos % 16, tid)] = v_new[tid];
    }
    const float scale = 1.0f / sqrtf((float)HD);
    for (int m0 = 0; m0 < ctx; m0 += KPP) {
        const int m = m0 + km;
        floatx4 kv = k0;
        if (m0 > 0 && m < pos) kv = load4(a.pool + a.geo.k_off(a.layer, bt[m / 16], g, m % 16, sub * 4));
        if (m == pos) kv = *reinterpret_cast<const floatx4*>(k_new + sub * 4);
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const floatx4 q = *reinterpret_cast<const floatx4*>(qkv + h * HD + sub * 4);
            float s = sum16(q[0] * kv[0] + q[1] * kv[1] + q[2] * kv[2] + q[3] * kv[3]);
            if (TPK == 32) s += __shfl_xor(s, 16, RL_WAVE);
            if (sub == 0 && m < ctx) sc[h * a.ctx_cap + m] = s * scale;
        }
    }
    __syncthreads();
    float mx[G];                                    // every wave forms the maximum and the sum itself
#pragma unroll
    for (int h = 0; h < G; ++h) {
        mx[h] = -INFINITY;
        float l = 0.f;
        for (int m = lane; m < ctx; m += 64) mx[h] = fmaxf(mx[h], sc[h * a.ctx_cap + m]);
        mx[h] = max64(mx[h]);
        if (wave == h) {
            for (int m = lane; m < ctx; m += 64) l += __expf(sc[h * a.ctx_cap + m] - mx[h]);
            l = sum64(l);
            if (lane == 0) sm_l[h] = l;
        }
    }
    float o[G];
#pragma unroll
    for (int h = 0; h < G; ++h) o[h] = pt == 0 ? __expf(sc[h * a.ctx_cap + pos] - mx[h]) * v_new[dd] : 0.f;
    for (int m0 = 0; m0 < pos; m0 += KPP) {
        const int m = m0 + pt * 4;
        if (m >= pos) continue;
        floatx4 v = v0;
        if (m0 > 0) v = load4(a.pool + a.geo.v_off(a.layer, bt[m / 16], g, m % 16, dd));
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i)             // slots past the last key hold anything
                if (m + i < pos) o[h] += __expf(sc[h * a.ctx_cap + m + i] - mx[h]) * v[i];
    }
#pragma unroll
    for (int h = 0; h < G; ++h) part[(h * PARTS + pt) * HD + dd] = o[h];
    __syncthreads();
    if (tid < G * HD) {
        const int h = tid / HD;
        float r = 0.f;
#pragma unroll
        for (int i = 0; i < PARTS; ++i) r += part[(h * PARTS + i) * HD + dd];
        out[tid] = r / sm_l[h];
    }
}
static size_t plain_front_lds(int G, int hd, int ctx) { return (size_t)((G + 2) * hd + G * 1024 + 4 + G * ctx) * sizeof(float); }
// A block reads its columns' weights by itself, 256 k of them at a time, each a memory latency.  Whole generations of 48 tokens, 6 layers,
// 4 to 256 blocks, contexts of 12 to 60 keys, time of this over the two kernels': one query head per kv head, head_dim 64, d 640 (480 KB a
// block) 0.94 - 0.95; 128, d 320 (480 KB) 0.97 - 1.00; two heads, 64, d 384 and 512 (384, 512 KB) 0.94 - 0.97; 128, d 64 to 256 (128
// to 512 KB) 0.91 - 1.00; four heads, 64, d 64 (96 KB) 0.92 - 1.02, 192 0.92 - 0.99, 256 (384 KB) 0.92 - 1.03, 320 (480 KB) 1.00 - 1.09.  Longer
// contexts gain more: alone, 400 to 14000 keys, 0.55 - 0.95.  Blocks beyond one per CU would wait for a second round.
bool k_plain_front_supported(int Hq, int Hkv, int hd, int d, int max_batch, int max_seq) {
    const int G = Hq / Hkv;
    if (!(G == 1 || G == 2 || (G == 4 && hd == 64))) return false;
    return (int64_t)(G + 2) * hd * d * 4 <= (G == 4 ? 384 : 512) * 1024 && (int64_t)max_batch * Hkv <= 256 &&
           plain_front_lds(G, hd, max_seq) <= 65536;
}
void k_plain_front(const float* x, const float* gain, float eps, const float* W, int d, const float2* rope, float* pool, int layer,
                   KvGeom geo, const int* block_table, int mpps, const int* tok_pos, float* out, int n, int Hq, int max_ctx,
                   const PlainStart& start, hipStream_t s) {
    if (n <= 0) return;
    const PlainFrontArgs a{x, gain, W, eps, d, rope, pool, layer, geo, block_table, tok_pos, mpps, Hq, max_ctx, out, start};
    const int G = Hq / geo.Hkv;
    const dim3 grid(n, geo.Hkv);
    const size_t lds = plain_front_lds(G, geo.hd, max_ctx);
    if (geo.hd == 64) {
        if (G == 1) plain_front_kernel<64, 1><<<grid, 1024, lds, s>>>(a);
        else if (G == 2) plain_front_kernel<64, 2><<<grid, 1024, lds, s>>>(a);
        else plain_front_kernel<64, 4><<<grid, 1024, lds, s>>>(a);
    } else {
        if (G == 1) plain_front_kernel<128, 1><<<grid, 1024, lds, s>>>(a);
        else plain_front_kernel<128, 2><<<grid, 1024, lds, s>>>(a);
    }
}

// ---------------------------------------------------------------- sampling
// Counter-based uniform: two rounds of the splitmix64 output function over
// (seed, sequence id, step); top 24 bits -> [0,1).  Integer-only, so the CPU
// checker reproduces it bit for bit.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__device__ __forceinline__ float hash_uniform(uint64_t seed, uint64_t seq, uint64_t step) {
    const uint64_t G = 0x9E3779B97F4A7C15ull;
    uint64_t h = mix64(seed + G * (seq + 1));
    h = mix64(h + G * (step + 1));
    return (float)(h >> 40) * (1.0f / 16777216.0f);
}

// Row statistics shared by sampling and scoring: max, arg-max (lowest index on ties).
struct ArgMax { float v; int i; };
__device__ __forceinline__ ArgMax argmax_combine(ArgMax a, ArgMax b) {
    if (b.v > a.v || (b.v == a.v && b.i < a.i)) return b;
    return a;
}
template <int CTRL>
__device__ __forceinline__ ArgMax argmax_dpp(ArgMax a) {
    return argmax_combine(a, ArgMax{__int_as_float(dpp_int<CTRL>(__float_as_int(a.v))), dpp_int<CTRL>(a.i)});
}
// over a block, every thread with the result; red holds one element per wave and is used for nothing else
__device__ __forceinline__ ArgMax block_argmax(ArgMax a, ArgMax* red) {
    a = argmax_dpp<0xB1>(a);     // quad_perm [1,0,3,2]
    a = argmax_dpp<0x4E>(a);     // quad_perm [2,3,0,1]
    a = argmax_dpp<0x141>(a);    // row_half_mirror
    a = argmax_dpp<0x140>(a);    // row_mirror
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) a = argmax_combine(a, ArgMax{__shfl_xor(a.v, o, RL_WAVE), __shfl_xor(a.i, o, RL_WAVE)});
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) red[w] = a;
    __syncthreads();
    ArgMax r = red[0];
    for (int i = 1; i < nw; ++i) r = argmax_combine(r, red[i]);
    return r;
}

// One block of 1024 threads per sequence.  Wave w owns the contiguous vocabulary
// segment [w*seg, (w+1)*seg); sums are formed lane-column-wise then reduced, in a
// fixed order, so results are reproducible run to run.  A chain of loads, reductions and barriers: everything the row needs is
// requested first, lanes reduce by data-parallel-primitive moves, greedy leaves out the tempered sums (4 rows of 4096, in a
// graph of such launches: 4.7 -> 4.0 us).
// out_ids / out_logp (optional) are [B, out_stride]; the column is the sequence's decode-step
// counter, kept on the device so that a captured step can be replayed unchanged.
__global__ __launch_bounds__(1024) void sample_kernel(const float* logits, int ldz, int V, SampleArgs a, int* last_tok,
                                                      int* seq_len, int* gen_count, int* finished, int* step_count,
                                                      int* tok_out, float* logp_out, int* out_ids, float* out_logp,
                                                      int out_stride) {
    __shared__ ArgMax ared[16];
    __shared__ float ws1[16], wsT[16];
    __shared__ int s_tok;
    const int b = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const float* z = logits + (int64_t)b * ldz;
    const bool greedy = !(a.temperature > 0.f);
    const float invT = greedy ? 1.0f : 1.0f / a.temperature;
    int seg = (V + 15) / 16;
    seg = (seg + 255) / 256 * 256;
    const int s0 = w * seg, s1 = min(V, s0 + seg);
    const bool vec = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(z) & 15) == 0;
    const float4* const z4 = reinterpret_cast<const float4*>(z);
    // the first 16 bytes of every lane (all of a vocabulary of 4096) stay in registers; the row's counters travel with them
    float4 first = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    if (vec && s0 / 4 + lane < s1 / 4) first = z4[s0 / 4 + lane];
    const int64_t orow = a.out_row ? a.out_row[b] : b;
    const int n_gen = gen_count[b], st = step_count[b], len = seq_len[b], limit = a.gen_limit ? a.gen_limit[b] : 0;
    const int64_t seq = a.seq_base + (a.seq_id ? a.seq_id[b] : b);
    if (finished[b] != 0) {
        // a finished sequence keeps emitting eos_id with log-prob 0 and no longer advances
        if (threadIdx.x == 0) {
            last_tok[b] = a.eos_id >= 0 ? a.eos_id : 0;   // a parked row still feeds a valid id through the GEMMs
            if (tok_out) tok_out[b] = a.eos_id;
            if (logp_out) logp_out[b] = 0.f;
            step_count[b] = st + 1;
            if (st < out_stride) {
                if (out_ids) out_ids[orow * out_stride + st] = a.eos_id;
                if (out_logp) out_logp[orow * out_stride + st] = 0.f;
            }
        }
        return;
    }
    ArgMax am{-INFINITY, 0x7fffffff};
    if (vec) {
        for (int i = s0 / 4 + lane; i < s1 / 4; i += 64) {
            const float4 q = i == s0 / 4 + lane ? first : z4[i];   // increasing index: "first greater" keeps the lowest of equals
            if (q.x > am.v) { am.v = q.x; am.i = 4 * i; }
            if (q.y > am.v) { am.v = q.y; am.i = 4 * i + 1; }
            if (q.z > am.v) { am.v = q.z; am.i = 4 * i + 2; }
            if (q.w > am.v) { am.v = q.w; am.i = 4 * i + 3; }
        }
    } else {
        for (int i = s0 + lane; i < s1; i += 64)
            if (z[i] > am.v) { am.v = z[i]; am.i = i; }
    }
    am = block_argmax(am, ared);
    const float mx = am.v;
    float c1 = 0.f, cT = 0.f;
    if (vec) {
        for (int i = s0 / 4 + lane; i < s1 / 4; i += 64) {
            const float4 q = i == s0 / 4 + lane ? first : z4[i];
            const float d0 = q.x - mx, d1 = q.y - mx, d2 = q.z - mx, d3 = q.w - mx;
            c1 += (__expf(d0) + __expf(d1)) + (__expf(d2) + __expf(d3));
            if (!greedy) cT += (__expf(d0 * invT) + __expf(d1 * invT)) + (__expf(d2 * invT) + __expf(d3 * invT));
        }
    } else {
        for (int i = s0 + lane; i < s1; i += 64) {
            float dz = z[i] - mx;
            c1 += __expf(dz);
            if (!greedy) cT += __expf(dz * invT);
        }
    }
    c1 = sum64(c1);
    if (!greedy) cT = sum64(cT);
    if (lane == 0) { ws1[w] = c1; wsT[w] = cT; }
    if (threadIdx.x == 0) s_tok = V - 1;
    __syncthreads();
    float tot1 = 0.f, totT = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) { tot1 += ws1[i]; totT += wsT[i]; }
    int tok = am.i;
    if (!greedy) {
        float u = hash_uniform(a.seed, (uint64_t)seq, (uint64_t)n_gen);
        float target = u * totT;
        float cum = 0.f;
        int wsel = -1;
        float before = 0.f;
        for (int i = 0; i < 16; ++i) {
            float nc = cum + wsT[i];
            if (wsel < 0 && nc > target) { wsel = i; before = cum; }
            cum = nc;
        }
        if (w == wsel) {
            float run = before;
            int found = -1;
            for (int r0 = s0; r0 < s1 && found < 0; r0 += 64) {
                int i = r0 + lane;
                float e = (i < s1) ? __expf((z[i] - mx) * invT) : 0.f;
                float rowsum = wave_sum(e);
                if (run + rowsum > target) {
                    float pe = e;   // inclusive prefix over lanes
#pragma unroll
                    for (int o = 1; o < 64; o <<= 1) {
                        float t = __shfl_up(pe, o, RL_WAVE);
                        if (lane >= o) pe += t;
                    }
                    unsigned long long m = __ballot((run + pe > target) && (i < s1));
                    if (m) found = r0 + __ffsll((long long)m) - 1;
                    else run += rowsum;
                } else {
                    run += rowsum;
                }
            }
            if (found < 0) found = s1 - 1;   // crossing falls on the segment end within rounding
            if (lane == 0) s_tok = found;
        }
        __syncthreads();
        tok = s_tok;
    }
    if (threadIdx.x == 0) {
        const float lp = (greedy ? mx : z[tok]) - mx - logf(tot1);
        gen_count[b] = n_gen + 1;
        if ((a.eos_id >= 0 && tok == a.eos_id) || (a.gen_limit && n_gen + 1 >= limit)) {
            finished[b] = 1;
            if (a.out_len) a.out_len[orow] = n_gen + 1;
        }
        last_tok[b] = tok;
        seq_len[b] = len + 1;
        if (tok_out) tok_out[b] = tok;
        if (logp_out) logp_out[b] = lp;
        step_count[b] = st + 1;
        if (st < out_stride) {
            if (out_ids) out_ids[orow * out_stride + st] = tok;
            if (out_logp) out_logp[orow * out_stride + st] = lp;
        }
    }
}
void k_sample(const float* logits, int ldz, int V, int B, SampleArgs a, int* last_tok, int* seq_len, int* gen_count,
              int* finished, int* step_count, int* tok_out, float* logp_out, int* out_ids, float* out_logp,
              int out_stride, hipStream_t s) {
    if (B <= 0) return;
    sample_kernel<<<B, 1024, 0, s>>>(logits, ldz, V, a, last_tok, seq_len, gen_count, finished, step_count, tok_out,
                                     logp_out, out_ids, out_logp, out_stride);
}

// The same draw from per-block statistics instead of logits (the LM-head GEMM's MG_SAMPLE epilogue: per row and
// 32-column block the maximum, its column, and the sums of exp((z - max) / T) and exp(z - max)): the logits of a decode
// step never reach memory.  One block of 1024 threads per sequence; thread t owns the contiguous run of blocks
// [t * per, (t + 1) * per), sums are formed in block order and scanned in thread order, so results are
// reproducible run to run.  Greedy: the first block holding the global maximum, and its column.  Otherwise the
// block in which the cumulative sum passes u * total is found from the statistics, and only that block's 32
// logits are recomputed (h . W rows, fp32 accumulation) to place the token inside it; if rounding differences between
// those 32 values and the block's own sum keep the cumulative sum from passing the target inside the block, the
// block's last column is taken (the crossing then lies on the block's end within rounding).
__global__ __launch_bounds__(1024) void sample_blocks_kernel(const float4* stats, int nblk, const f16_t* h, int ldh,
                                                             const bf16_t* W, int d, SampleArgs a, int* last_tok,
                                                             int* seq_len, int* gen_count, int* finished,
                                                             int* step_count, int* tok_out, float* logp_out,
                                                             int* out_ids, float* out_logp, int out_stride) {
    __shared__ ArgMax ared[16];
    __shared__ float red1[16], redT[16], zs[32];
    __shared__ int s_first, s_blk, s_tok;
    __shared__ float s_before, s_ztok;
    const int b = blockIdx.x;
    const int64_t orow = a.out_row ? a.out_row[b] : b;
    if (finished[b] != 0) {
        // a finished sequence keeps emitting eos_id with log-prob 0 and no longer advances
        if (threadIdx.x == 0) {
            last_tok[b] = a.eos_id >= 0 ? a.eos_id : 0;   // a parked row still feeds a valid id through the GEMMs
            if (tok_out) tok_out[b] = a.eos_id;
            if (logp_out) logp_out[b] = 0.f;
            const int st = step_count[b];
            step_count[b] = st + 1;
            if (st < out_stride) {
                if (out_ids) out_ids[orow * out_stride + st] = a.eos_id;
                if (out_logp) out_logp[orow * out_stride + st] = 0.f;
            }
        }
        return;
    }
    const float4* st4 = stats + (int64_t)b * nblk;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int per = (nblk + 1023) / 1024;
    const int b0 = min(nblk, t * per), b1 = min(nblk, b0 + per);
    const bool greedy = !(a.temperature > 0.f);
    const float invT = greedy ? 1.0f : 1.0f / a.temperature;
    // global maximum and the first block that holds it
    ArgMax am{-INFINITY, 0x7fffffff};
    for (int i = b0; i < b1; ++i) {
        const float v = st4[i].x;
        if (v > am.v) { am.v = v; am.i = i; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        ArgMax o2{__shfl_xor(am.v, o, RL_WAVE), __shfl_xor(am.i, o, RL_WAVE)};
        am = argmax_combine(am, o2);
    }
    if (lane == 0) ared[w] = am;
    if (t == 0) { s_first = 0x7fffffff; s_blk = nblk - 1; s_before = 0.f; }
    __syncthreads();
    am = ared[0];
    for (int i = 1; i < 16; ++i) am = argmax_combine(am, ared[i]);
    const float mx = am.v;
    // this thread's share of both sums, then an inclusive scan of the temperature sum over the threads
    float l1 = 0.f, lT = 0.f;
    for (int i = b0; i < b1; ++i) {
        const float4 q = st4[i];
        l1 += q.z * __expf(q.x - mx);
        lT += q.y * __expf((q.x - mx) * invT);
    }
    float pT = lT;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float u_ = __shfl_up(pT, o, RL_WAVE);
        if (lane >= o) pT += u_;
    }
    const float w1 = wave_sum(l1);
    if (lane == 63) redT[w] = pT;
    if (lane == 0) red1[w] = w1;
    __syncthreads();
    float tot1 = 0.f, totT = 0.f, baseT = 0.f;
    for (int i = 0; i < 16; ++i) {
        if (i == w) baseT = totT;
        tot1 += red1[i];
        totT += redT[i];
    }
    const float up1 = __shfl_up(pT, 1, RL_WAVE);
    const float incl = baseT + pT, excl = baseT + (lane > 0 ? up1 : 0.f);   // excl of thread t == incl of thread t - 1, bit for bit
    const int n_gen = gen_count[b];
    float target = 0.f;
    if (!greedy) {
        const float u = hash_uniform(a.seed, (uint64_t)(a.seq_base + (a.seq_id ? a.seq_id[b] : b)), (uint64_t)n_gen);
        target = u * totT;
        if (b0 < b1 && incl > target) atomicMin(&s_first, t);
        __syncthreads();
        if (t == s_first) {
            // the scan says this thread's run of blocks holds the crossing; summed block by block it may fall just
            // short of it within rounding: then the run's last block takes it
            float cum = excl;
            int sel = b1 - 1;
            for (int i = b0; i < b1; ++i) {
                const float4 q = st4[i];
                const float nc = cum + q.y * __expf((q.x - mx) * invT);
                if (nc > target || i == b1 - 1) { sel = i; break; }
                cum = nc;
            }
            s_blk = sel;
            s_before = cum;
        }
        __syncthreads();
        // the 32 logits of the chosen block: column t / 32, 32 threads per column over 16-byte pieces of k
        const int blk = s_blk;
        const float4 top = st4[blk];
        const int col = t >> 5, part = t & 31;
        const bf16_t* wrow = W + ((int64_t)blk * 32 + col) * d;
        const f16_t* hrow = h + (int64_t)b * ldh;
        float acc = 0.f;
        for (int k = part * 8; k < d; k += 256) {
            typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
            typedef unsigned short us8_t __attribute__((ext_vector_type(8)));
            const half8_t hv = *reinterpret_cast<const half8_t*>(hrow + k);
            const us8_t wv = *reinterpret_cast<const us8_t*>(wrow + k);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc += (float)hv[e] * __uint_as_float((unsigned)wv[e] << 16);
        }
#pragma unroll
        for (int o = 1; o < 32; o <<= 1) acc += __shfl_xor(acc, o, RL_WAVE);
        if (part == 0) zs[col] = acc;
        __syncthreads();
        if (t < 64) {
            const float e = t < 32 ? __expf((zs[t & 31] - mx) * invT) : 0.f;
            float pe = e;
#pragma unroll
            for (int o = 1; o < 32; o <<= 1) {
                const float u_ = __shfl_up(pe, o, RL_WAVE);
                if (lane >= o) pe += u_;
            }
            const unsigned long long hit = __ballot(t < 32 && s_before + pe > target);
            if (t == 0) {
                const int c = hit ? __ffsll((long long)hit) - 1 : 31;
                s_tok = blk * 32 + c;
                // the block's largest logit as the LM head has it: of the row's largest, which most draws take, nothing but the
                // sum of exponentials is left then, and not the rounding of two sums over d in different order
                s_ztok = c == __float_as_int(top.w) ? top.x : zs[c];
            }
        }
    } else if (t == 0) {
        s_tok = am.i * 32 + __float_as_int(st4[am.i].w);
        s_ztok = mx;
    }
    __syncthreads();
    if (t == 0) {
        const int tok = s_tok;
        const float lp = s_ztok - mx - logf(tot1);
        gen_count[b] = n_gen + 1;
        if ((a.eos_id >= 0 && tok == a.eos_id) || (a.gen_limit && n_gen + 1 >= a.gen_limit[b])) {
            finished[b] = 1;
            if (a.out_len) a.out_len[orow] = n_gen + 1;
        }
        last_tok[b] = tok;
        seq_len[b] = seq_len[b] + 1;
        if (tok_out) tok_out[b] = tok;
        if (logp_out) logp_out[b] = lp;
        const int st = step_count[b];
        step_count[b] = st + 1;
        if (st < out_stride) {
            if (out_ids) out_ids[orow * out_stride + st] = tok;
            if (out_logp) out_logp[orow * out_stride + st] = lp;
        }
    }
}
void k_sample_blocks(const float4* stats, int V, const void* h, int ldh, const void* W, int d, int B, SampleArgs a,
                     int* last_tok, int* seq_len, int* gen_count, int* finished, int* step_count, int* tok_out,
                     float* logp_out, int* out_ids, float* out_logp, int out_stride, hipStream_t s) {
    if (B <= 0) return;
    sample_blocks_kernel<<<B, 1024, 0, s>>>(stats, V / 32, (const f16_t*)h, ldh, (const bf16_t*)W, d, a, last_tok, seq_len,
                                            gen_count, finished, step_count, tok_out, logp_out, out_ids, out_logp,
                                            out_stride);
}

// ---------------------------------------------------------------- log-sum-exp + gather over materialised logits
// logp_out[slot, pos + 1] = z[target] - log sum_v exp(z_v) for rows with a target.
__global__ __launch_bounds__(1024) void lse_gather_kernel(const float* logits, int ldz, int V, const int* tok_tgt,
                                                          const int* tok_slot, const int* tok_pos, float* logp_out,
                                                          int ld_out) {
    __shared__ float red[16];
    const int r = blockIdx.x;
    const int tgt = tok_tgt[r];
    if (tgt < 0) return;
    const float* z = logits + (int64_t)r * ldz;
    float m = -INFINITY;
    for (int i = threadIdx.x; i < V; i += 1024) m = fmaxf(m, z[i]);
    m = block_max(m, red);
    float su = 0.f;
    for (int i = threadIdx.x; i < V; i += 1024) su += __expf(z[i] - m);
    su = block_sum(su, red);
    if (threadIdx.x == 0) {
        int t = min(max(tgt, 0), V - 1);
        logp_out[(int64_t)tok_slot[r] * ld_out + tok_pos[r] + 1] = z[t] - m - logf(su);
    }
}
void k_lse_gather(const float* logits, int ldz, int V, int nrows, const int* tok_tgt, const int* tok_slot,
                  const int* tok_pos, float* logp_out, int ld_out, hipStream_t s) {
    if (nrows <= 0) return;
    lse_gather_kernel<<<nrows, 1024, 0, s>>>(logits, ldz, V, tok_tgt, tok_slot, tok_pos, logp_out, ld_out);
}

// ---------------------------------------------------------------- KL term on response positions
__global__ void kl_kernel(const float* lp, const float* lr, const int* seq_len, const int* prompt_len, int Lmax,
                          float coef, float* kl, float* pen) {
    int b = blockIdx.y;
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= Lmax) return;
    int64_t o = (int64_t)b * Lmax + t;
    int lo = max(prompt_len[b], 1);
    float v = (t >= lo && t < seq_len[b]) ? lp[o] - lr[o] : 0.f;
    if (kl) kl[o] = v;
    if (pen) pen[o] = coef * v;
}
void k_kl(const float* lp, const float* lr, const int* seq_len, const int* prompt_len, int B, int Lmax, float coef,
          float* kl, float* pen, hipStream_t s) {
    if (B <= 0 || Lmax <= 0) return;
    dim3 grid((Lmax + 255) / 256, B);
    kl_kernel<<<grid, 256, 0, s>>>(lp, lr, seq_len, prompt_len, Lmax, coef, kl, pen);
}

// ---------------------------------------------------------------- value head of a critic / reward model
// v[slot, pos] = head . RMSNorm(x_row; g) for every packed row with pos >= 0: the final norm and the
// [d] -> 1 head in one pass over the fp32 residual stream (nothing is rounded to fp16 on the way).
template <typename TW>
__global__ __launch_bounds__(256) void value_head_kernel(const float* x, const TW* g, const TW* head, int d, float eps,
                                                         const int* tok_slot, const int* tok_pos, float* out,
                                                         int ld_out) {
    __shared__ float red[16];
    const int n = blockIdx.x;
    const int pos = tok_pos[n];
    if (pos < 0) return;
    const float* xr = x + (int64_t)n * d;
    float ss = 0.f, dot = 0.f;
    for (int j = threadIdx.x; j < d; j += 256) {
        const float v = xr[j];
        ss += v * v;
        dot += v * to_f(g[j]) * to_f(head[j]);
    }
    ss = block_sum(ss, red);
    dot = block_sum(dot, red);
    if (threadIdx.x == 0) out[(int64_t)tok_slot[n] * ld_out + pos] = dot / sqrtf(ss / (float)d + eps);
}
void k_value_head(int dtype, const float* x, const void* g, const void* head, int n, int d, float eps,
                  const int* tok_slot, const int* tok_pos, float* out, int ld_out, hipStream_t s) {
    if (n <= 0) return;
    if (dtype == 0)
        value_head_kernel<float><<<n, 256, 0, s>>>(x, (const float*)g, (const float*)head, d, eps, tok_slot, tok_pos, out, ld_out);
    else
        value_head_kernel<bf16_t><<<n, 256, 0, s>>>(x, (const bf16_t*)g, (const bf16_t*)head, d, eps, tok_slot, tok_pos, out, ld_out);
}

// ---------------------------------------------------------------- PPO reward per token
// r[b,t] = -coef * kl[b,t] on response positions [prompt_len, L), plus seq_reward[b] at t = L-1; 0 elsewhere.
__global__ void ppo_reward_kernel(const float* kl, const float* seq_reward, const int* seq_len, const int* prompt_len,
                                  int Lmax, float coef, float* out) {
    int b = blockIdx.y;
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= Lmax) return;
    const int64_t o = (int64_t)b * Lmax + t;
    const int L = seq_len[b], P = prompt_len[b];
    float r = 0.f;
    if (t >= P && t < L) {
        r = -coef * kl[o];
        if (t == L - 1) r += seq_reward[b];
    }
    out[o] = r;
}
// dst[first + i] = v[i] for i < n <= 192: small host arrays reach the device as kernel arguments (no copy engine,
// no pinned staging), 192 values per launch.
struct IntChunk { int v[192]; };
__global__ void put_i32_kernel(int* dst, IntChunk c, int n) {
    if ((int)threadIdx.x < n) dst[threadIdx.x] = c.v[threadIdx.x];
}
void k_put_i32(int* dst, const int* src_host, int n, hipStream_t s) {
    for (int o = 0; o < n; o += 192) {
        IntChunk c;
        const int m = n - o < 192 ? n - o : 192;
        for (int i = 0; i < m; ++i) c.v[i] = src_host[o + i];
        put_i32_kernel<<<1, 192, 0, s>>>(dst + o, c, m);
    }
}

void k_ppo_reward(const float* kl, const float* seq_reward, const int* seq_len, const int* prompt_len, int B, int Lmax,
                  float coef, float* out, hipStream_t s) {
    if (B <= 0 || Lmax <= 0) return;
    dim3 grid((Lmax + 255) / 256, B);
    ppo_reward_kernel<<<grid, 256, 0, s>>>(kl, seq_reward, seq_len, prompt_len, Lmax, coef, out);
}

// ---------------------------------------------------------------- exact KL from per-group partials
// One wave per row: combine the nparts quintuples (m_p, S_p, T, m_r, S_r) written by the dual LM-head GEMM
// into KL(pi_policy || pi_ref) = T/S_p - lse_p + lse_r and write it at [slot, pos + 1] on response
// positions (pos + 1 >= max(prompt_len, 1)); rows without a next token inside their sequence are skipped.
__global__ __launch_bounds__(64) void kl_full_reduce_kernel(const float* part, int nparts, const int* tok_tgt,
                                                            const int* tok_slot, const int* tok_pos,
                                                            const int* prompt_len, const int* rows, float* out, int ld_out) {
    const int r = rows[blockIdx.x];                 // row of the packed token list behind the compacted row blockIdx.x
    if (tok_tgt[r] < 0) return;
    const int slot = tok_slot[r], t = tok_pos[r] + 1;
    if (t < max(prompt_len[slot], 1)) return;
    const float* p = part + (int64_t)blockIdx.x * nparts * 5;
    float mp = -INFINITY, sp = 0.f, tt = 0.f, mr = -INFINITY, sr = 0.f;
    for (int i = threadIdx.x; i < nparts; i += 64) {
        const float m1 = p[i * 5], s1 = p[i * 5 + 1], t1 = p[i * 5 + 2], m2 = p[i * 5 + 3], s2 = p[i * 5 + 4];
        const float mn = fmaxf(mp, m1), a0 = __expf(mp - mn), a1 = __expf(m1 - mn);
        sp = sp * a0 + s1 * a1;
        tt = tt * a0 + t1 * a1;
        mp = mn;
        const float mq = fmaxf(mr, m2);
        sr = sr * __expf(mr - mq) + s2 * __expf(m2 - mq);
        mr = mq;
    }
    const float Mp = wave_max(mp), Mr = wave_max(mr);
    const float wp = __expf(mp - Mp);
    sp = wave_sum(sp * wp);
    tt = wave_sum(tt * wp);
    sr = wave_sum(sr * __expf(mr - Mr));
    if (threadIdx.x == 0) out[(int64_t)slot * ld_out + t] = tt / sp - (Mp + logf(sp)) + (Mr + logf(sr));
}
void k_kl_full_reduce(const float* part, int nparts, int nrows, const int* tok_tgt, const int* tok_slot,
                      const int* tok_pos, const int* prompt_len, const int* rows, float* out, int ld_out, hipStream_t s) {
    if (nrows <= 0) return;
    kl_full_reduce_kernel<<<nrows, 64, 0, s>>>(part, nparts, tok_tgt, tok_slot, tok_pos, prompt_len, rows, out, ld_out);
}

// The same from two materialised logit rows (plain path): one block per row.
__global__ __launch_bounds__(1024) void kl_full_rows_kernel(const float* zp, const float* zr, int ldz, int V,
                                                            const int* tok_tgt, const int* tok_slot,
                                                            const int* tok_pos, const int* prompt_len, const int* rows, float* out,
                                                            int ld_out) {
    __shared__ float red[16];
    const int r = rows[blockIdx.x];
    if (tok_tgt[r] < 0) return;
    const int slot = tok_slot[r], t = tok_pos[r] + 1;
    if (t < max(prompt_len[slot], 1)) return;
    const float* a = zp + (int64_t)blockIdx.x * ldz;
    const float* b = zr + (int64_t)blockIdx.x * ldz;
    float mp = -INFINITY, mr = -INFINITY;
    for (int i = threadIdx.x; i < V; i += 1024) { mp = fmaxf(mp, a[i]); mr = fmaxf(mr, b[i]); }
    mp = block_max(mp, red);
    mr = block_max(mr, red);
    float sp = 0.f, tt = 0.f, sr = 0.f;
    for (int i = threadIdx.x; i < V; i += 1024) {
        const float e = __expf(a[i] - mp);
        sp += e;
        tt += e * (a[i] - b[i]);
        sr += __expf(b[i] - mr);
    }
    sp = block_sum(sp, red);
    tt = block_sum(tt, red);
    sr = block_sum(sr, red);
    if (threadIdx.x == 0) out[(int64_t)slot * ld_out + t] = tt / sp - (mp + logf(sp)) + (mr + logf(sr));
}
void k_kl_full_rows(const float* zp, const float* zr, int ldz, int V, int nrows, const int* tok_tgt,
                    const int* tok_slot, const int* tok_pos, const int* prompt_len, const int* rows, float* out, int ld_out,
                    hipStream_t s) {
    if (nrows <= 0) return;
    kl_full_rows_kernel<<<nrows, 1024, 0, s>>>(zp, zr, ldz, V, tok_tgt, tok_slot, tok_pos, prompt_len, rows, out, ld_out);
}

// ---------------------------------------------------------------- log-prob from per-group (max, sum-exp) partials
// One wave per row: combine the nparts pairs written by the LM-head GEMM epilogue into
// log sum_v exp(z_v) and write logp = z_target - lse at [slot, pos + 1].
__global__ __launch_bounds__(64) void lse_reduce_kernel(const float2* part, int nparts, const float* z_tgt,
                                                        const int* tok_tgt, const int* tok_slot, const int* tok_pos,
                                                        float* logp_out, int ld_out) {
    const int r = blockIdx.x;
    if (tok_tgt[r] < 0) return;
    const float2* p = part + (int64_t)r * nparts;
    float m = -INFINITY, s = 0.f;
    for (int i = threadIdx.x; i < nparts; i += 64) {
        float2 v = p[i];
        float mn = fmaxf(m, v.x);
        s = s * __expf(m - mn) + v.y * __expf(v.x - mn);
        m = mn;
    }
    float mt = wave_max(m);
    s = wave_sum(s * __expf(m - mt));
    if (threadIdx.x == 0) logp_out[(int64_t)tok_slot[r] * ld_out + tok_pos[r] + 1] = z_tgt[r] - mt - logf(s);
}
void k_lse_reduce(const float2* part, int nparts, const float* z_tgt, int nrows, const int* tok_tgt,
                  const int* tok_slot, const int* tok_pos, float* logp_out, int ld_out, hipStream_t s) {
    if (nrows <= 0) return;
    lse_reduce_kernel<<<nrows, 64, 0, s>>>(part, nparts, z_tgt, tok_tgt, tok_slot, tok_pos, logp_out, ld_out);
}

// ---------------------------------------------------------------- instrument: sustained rate of the matrix cores
// Nothing but v_mfma_f32_16x16x32_f16 -- the shape the large-M GEMMs run -- on operands held in registers (64
// independent accumulator tiles per wave, four waves per CU, no memory traffic inside the loop): what the matrix cores
// sustain under the chip's power management on operands of the given kind.  Random operands (uniform in [-1, 1)) draw
// far more power than zeros, and the clock follows.  The accumulators are written out once at the end so that the loop
// cannot be removed.
__global__ __launch_bounds__(256, 1) void mfma_rate_kernel(const f16_t* in, float* out, int iters) {
    typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
    typedef float floatx4_t __attribute__((ext_vector_type(4)));
    const int l = threadIdx.x;
    half8_t a[8], b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = *reinterpret_cast<const half8_t*>(in + (size_t)(l + 256 * i) * 8);
        b[i] = *reinterpret_cast<const half8_t*>(in + (size_t)(l + 256 * (8 + i)) * 8);
    }
    floatx4_t acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[i], b[j], acc[i][j], 0, 0, 0);
        asm volatile("" : "+v"(a[0]), "+v"(b[0]));
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) s += acc[i][j][1] + acc[i][j][2];
    out[blockIdx.x * 256 + l] = s;
}
__global__ void mfma_rate_fill_kernel(f16_t* p, int n, int random) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    unsigned h = (unsigned)i * 2654435761u + 12345u;
    h ^= h >> 13; h *= 0x5bd1e995u; h ^= h >> 15;
    p[i] = random ? (f16_t)(((h & 0xffff) / 65536.0f) * 2.f - 1.f) : (f16_t)0.f;
}
// scratch: at least 64 KB + n_wg * 1 KB of device memory.  One launch of n_wg workgroups x iters x 64 MFMAs per wave.
void k_mfma_rate(void* scratch, int n_wg, int iters, int random, hipStream_t s) {
    f16_t* in = reinterpret_cast<f16_t*>(scratch);
    float* out = reinterpret_cast<float*>(reinterpret_cast<char*>(scratch) + 65536);
    mfma_rate_fill_kernel<<<(16 * 256 * 8 + 255) / 256, 256, 0, s>>>(in, 16 * 256 * 8, random);
    mfma_rate_kernel<<<n_wg, 256, 0, s>>>(in, out, iters);
}
