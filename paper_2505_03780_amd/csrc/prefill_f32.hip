// fp32 attention on the fp32 matrix instructions (exact fp32 products, fp32 accumulation).
//
// Same operation as the bf16 MFMA kernels (tiled online-softmax attention, the
// FlashAttention-2 formulation the paper's kernel follows, section "Method and
// Investigated Kernels"), kept in true fp32 for inputs that are fp32.  It serves
// small calls, so what bounds it is latency: the chain launch - lengths - K and V - two products - merge - store.
//
// A workgroup owns 16 query rows of one KV head (HPW heads of its group x 16 / HPW tokens: rows that share keys); its
// eight wavefronts split the keys, each taking every eighth 16-key chunk with a softmax state of its own, merged
// through LDS at the end, so that 128 keys are one chunk per wavefront.  Scores are computed transposed
// (S^T = K Q^T, v_mfma_f32_16x16x4_f32: lane holds four keys of one query row) and are, as they stand, the B operand of
// O^T += V^T P^T.  The contraction order is free as long as both operands agree: a lane's K load is 16 bytes of
// one key (dims 16j + 4g ..), a V load 16 bytes of one key's channels (the matrix instruction of index e takes channels
// 4i + e), so K and V come straight from memory in whole vectors without LDS.
// One wavefront per (token, head) with a lane per key, the kernel before, read K with 64 rows per load and V key after
// key: 128 tokens, 4 heads, D = 64 9.4 -> 6.1 us; 4 x 512 tokens, 8 heads 191 -> 23.7 us (D = 64) and 431 -> 46.7 us
// (D = 128, 46 TFLOP/s of visible pairs); the error against 64 bits is a tenth smaller.
#include "kernel_params.hpp"

#include <type_traits>

namespace attn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
// fp32 tensors need no more than their own alignment (the entry point asks for none): 16 bytes from any dword
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kRows = 16;
constexpr int kChunk = 16;
constexpr int kWaves = 8;

template <int HD>
struct F32Cfg {
    static constexpr int kRedPitch = HD + 4;  // floats per row and wavefront in the merge
    static constexpr size_t kLdsBytes = (size_t)kWaves * kRows * (kRedPitch + 2) * 4;
};

// query heads of one KV head in a workgroup: the largest power of two that divides the group, at most 16
__host__ __device__ inline int f32_heads(int group)
{
    const int h = group & -group;
    return h < kRows ? h : kRows;
}

// HD is 64 or 128.
template <int HD>
__global__ __launch_bounds__(kWaves * 64) void prefill_f32_kernel(const KParams p)
{
    using C = F32Cfg<HD>;
    constexpr int KJ = HD / 16;  // 16-byte K loads of a lane per chunk
    constexpr int VJ = HD / 64;  // 16-byte V loads of a lane per key
    extern __shared__ __attribute__((aligned(16))) float red[];  // [wave][row][HD + 4], then (max, sum) of every wave and row

    touch_args(p);
    const int hpw = f32_heads(p.group);
    const int log_hpw = __builtin_ctz(hpw);
    const int tok = kRows >> log_hpw;
    const QuotRem by_kvh = divmod_uniform(blockIdx.x, p.num_kv_heads);
    const QuotRem by_hsub = divmod_uniform(by_kvh.quot, p.group >> log_hpw);
    const QuotRem by_seq = divmod_uniform(by_hsub.quot, p.num_seqs);
    const int kvh = by_kvh.rem, hsub = by_hsub.rem, s = by_seq.rem;
    const int q_tiles = (p.max_q_len + tok - 1) >> (__builtin_ctz(kRows) - log_hpw);
    const int t0 = (q_tiles - 1 - by_seq.quot) * tok;  // costly (late) tiles first
    int q0 = load_uniform(p.query_start_loc, s), q1 = load_uniform(p.query_start_loc, s + 1), n_kv = load_uniform(p.seq_lens, s), kv0 = 0;
    if (!p.block_table) kv0 = load_uniform(p.kv_start_loc, s);
    asm volatile("" : "+s"(q0), "+s"(q1), "+s"(n_kv), "+s"(kv0));  // one round trip, ahead of the branch
    const int n_q = q1 - q0;
    if (t0 >= n_q) return;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15;  // query row; key of a K load; channel block of a V load
    const int g = lane >> 4;
    const int head0 = kvh * p.group + (hsub << log_hpw);

    // ---- this lane's query row, its dims 16j + 4g .. + 3 ----
    int t = t0 + (i >> log_hpw);
    t = t < n_q ? t : n_q - 1;
    const float *qrow = (const float *)p.q + (int64_t)(q0 + t) * p.q_stride_tok + (int64_t)(head0 + (i & (hpw - 1))) * p.q_stride_head + 4 * g;
    f32x4 qf[KJ];
#pragma unroll
    for (int j = 0; j < KJ; ++j) qf[j] = *(const f32x4u *)(qrow + 16 * j);
    // keys that the row sees, that any row of the tile sees, and that every row sees
    int limit = n_kv, kv_end = n_kv, open_end = n_kv;
    if (p.causal) {
        const int off = n_kv - n_q, last_tok = t0 + tok < n_q ? t0 + tok : n_q;
        limit = off + t + 1 < n_kv ? off + t + 1 : n_kv;
        kv_end = off + last_tok < n_kv ? off + last_tok : n_kv;
        open_end = off + t0 + 1 < n_kv ? off + t0 + 1 : n_kv;
    }

    const float *kbase = (const float *)p.k + (int64_t)kvh * p.kv_stride_head + 4 * g;
    const float *vbase = (const float *)p.v + (int64_t)kvh * p.kv_stride_head + 4 * i;
    const int32_t *bt_row = p.block_table ? p.block_table + (int64_t)s * p.block_table_stride : nullptr;

    f32x4 kf[KJ], vf[4][VJ];
    // element offset of the chunk of keys at c0 < n_kv (a multiple of 16: one cache block)
    auto chunk_base = [&](int c0) -> int64_t {
        if (!bt_row) return (int64_t)(kv0 + c0) * p.kv_stride_tok;
        return (int64_t)load_uniform(bt_row, c0 >> p.block_shift) * p.kv_stride_block + (int64_t)(c0 & (p.block_size - 1)) * p.kv_stride_tok;
    };
    // rows past the end re-read the last key
    auto load_k = [&](int c0, int64_t base) {
        const int last = n_kv - 1 - c0;
        const float *kr = kbase + base + (int64_t)(i < last ? i : last) * p.kv_stride_tok;
#pragma unroll
        for (int j = 0; j < KJ; ++j) kf[j] = *(const f32x4u *)(kr + 16 * j);
    };
    auto load_v = [&](int c0, int64_t base) {
        const int last = n_kv - 1 - c0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float *vr = vbase + base + (int64_t)(4 * g + v < last ? 4 * g + v : last) * p.kv_stride_tok;
#pragma unroll
            for (int j = 0; j < VJ; ++j) vf[v][j] = *(const f32x4u *)(vr + 64 * j);
        }
    };

    f32x4 oacc[VJ][4];  // [j][e]: lane holds channels 64j + 16g + 4v + e of its row
#pragma unroll
    for (int j = 0; j < VJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) oacc[j][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;  // l: this lane's keys only

    // A chunk with keys that some row does not see (or past the end): the products below multiply those by a weight of
    // zero, which turns an infinity or NaN in V into NaN.  Non-finite values are therefore taken out of the operand and
    // added, key by key, to the rows that see them.  Rare: a test per value of such a chunk is all that finite inputs pay.
    auto keep_apart = [&](int c0, const float (&w)[4]) {
        auto finite = [](float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; };
        float probe[4] = {0.f, 0.f, 0.f, 0.f};  // NaN once a value is not finite
#pragma unroll
        for (int j = 0; j < VJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int v = 0; v < 4; ++v) probe[v] = __builtin_fmaf(vf[v][j][e], 0.f, probe[v]);
        if (__builtin_amdgcn_ballot_w64(!finite((probe[0] + probe[1]) + (probe[2] + probe[3]))) == 0) return;
#pragma unroll 1
        for (int kg = 0; kg < 4; ++kg) {
#pragma unroll
            for (int kv = 0; kv < 4; ++kv) {  // key c0 + 4 kg + kv: its weights and values lie in the lanes of group kg
                const float wk = __shfl(w[kv], 16 * kg + i);
                const bool sees = c0 + 4 * kg + kv < limit;
#pragma unroll
                for (int j = 0; j < VJ; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float x = __shfl(vf[kv][j][e], 16 * kg + 4 * g + v);
                            if (sees && !finite(x)) oacc[j][e][v] += wk * x;
                        }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < VJ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) vf[v][j][e] = finite(vf[v][j][e]) ? vf[v][j][e] : 0.f;
    };

    // one chunk; MORE: the registers of K, then of V, take the wave's next chunk as soon as they are free
    constexpr int kStep = kWaves * kChunk;
    int64_t next_base = 0;
    auto step = [&](int c0, auto more_tag) {
        constexpr bool MORE = decltype(more_tag)::value;
        f32x4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) sacc = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][e], qf[j][e], sacc, 0, 0, 0);
        if (MORE) load_k(c0 + kStep, next_base);
        __builtin_amdgcn_sched_barrier(0);
        float x[4], mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            x[v] = c0 + 4 * g + v < limit ? sacc[v] * p.scale : -INFINITY;
            mx = fmaxf(mx, x[v]);
        }
        mx = max_over_groups(mx);
        const float m_new = fmaxf(m, mx);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;  // (no visible key so far: all weights are zero)
        const float alpha = expf(m - m_use);
        m = m_new;
        float w[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) w[v] = expf(x[v] - m_use);
        l = l * alpha + ((w[0] + w[1]) + (w[2] + w[3]));
#pragma unroll
        for (int j = 0; j < VJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) oacc[j][e] *= alpha;
        if (c0 + kChunk > open_end) keep_apart(c0, w);
#pragma unroll
        for (int j = 0; j < VJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
#pragma unroll
                for (int v = 0; v < 4; ++v) oacc[j][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v][j][e], w[v], oacc[j][e], 0, 0, 0);
            }
        if (MORE) {
            load_v(c0 + kStep, next_base);
            next_base = chunk_base(c0 + 2 * kStep < kv_end ? c0 + 2 * kStep : c0);
        }
    };
    int c0 = wave * kChunk;
    if (c0 < kv_end) {
        const int64_t base = chunk_base(c0);
        load_k(c0, base);
        load_v(c0, base);
        next_base = chunk_base(c0 + kStep < kv_end ? c0 + kStep : c0);
        for (; c0 + kStep < kv_end; c0 += kStep) step(c0, std::integral_constant<bool, true>{});
        step(c0, std::integral_constant<bool, false>{});
    }

    // ---- merge the wavefronts ----
    l = sum_over_groups(l);
    float *state = red + kWaves * kRows * C::kRedPitch;
    float *mine = red + (wave * kRows + i) * C::kRedPitch + 16 * g;
#pragma unroll
    for (int j = 0; j < VJ; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) *(f32x4 *)(mine + 64 * j + 4 * v) = f32x4{oacc[j][0][v], oacc[j][1][v], oacc[j][2][v], oacc[j][3][v]};
    if (g == 0) *(float2 *)(state + 2 * (wave * kRows + i)) = float2{m, l};
    __syncthreads();
    for (int idx = tid; idx < kRows * (HD / 4); idx += kWaves * 64) {
        const int row = idx / (HD / 4), ch = 4 * (idx % (HD / 4));
        const int tr = t0 + (row >> log_hpw);
        if (tr >= n_q) continue;
        float2 ml[kWaves];
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            ml[w] = *(const float2 *)(state + 2 * (w * kRows + row));
            M = fmaxf(M, ml[w].x);
        }
        const float m_use = M == -INFINITY ? 0.f : M;
        float L = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float sc = expf(ml[w].x - m_use);  // 0 for a wavefront without keys
            L += ml[w].y * sc;
            o += *(const f32x4 *)(red + (w * kRows + row) * C::kRedPitch + ch) * sc;
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;  // (a query without a visible key gets zeros)
        *(f32x4u *)((float *)p.out + (int64_t)(q0 + tr) * p.o_stride_tok + (int64_t)(head0 + (row & (hpw - 1))) * p.o_stride_head + ch) = o * inv;
    }
}

template <int HD>
hipError_t f32_launch(const KParams &p, hipStream_t stream, unsigned blocks)
{
    auto kern = prefill_f32_kernel<HD>;
    static std::atomic<uint64_t> granted{0};
    const hipError_t allowed = allow_dynamic_lds((const void *)kern, F32Cfg<HD>::kLdsBytes, granted);
    if (allowed != hipSuccess) return allowed;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kWaves * 64), F32Cfg<HD>::kLdsBytes, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_f32(const KParams &p, hipStream_t stream)
{
    const int hpw = f32_heads(p.group), tok = kRows / hpw;
    const int64_t blocks = (int64_t)((p.max_q_len + tok - 1) / tok) * p.num_seqs * (p.num_q_heads / hpw);
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    if (p.head_dim == 64) return f32_launch<64>(p, stream, (unsigned)blocks);
    if (p.head_dim == 128) return f32_launch<128>(p, stream, (unsigned)blocks);
    return hipErrorInvalidValue;
}

}  // namespace attn
