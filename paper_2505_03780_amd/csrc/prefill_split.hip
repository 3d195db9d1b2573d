// Causal variable-length prefill for few query rows over many keys (gfx950): the wavefronts of a
// workgroup split the key axis.
//
// Same operation as the other prefill kernels (tiled online-softmax attention, grouped-query heads;
// the paper's section "Method and Investigated Kernels").  The ring kernel gives a workgroup 128 or 256
// query rows and lets all its wavefronts walk the keys together, one barrier per 32 keys: right when
// there are enough query tiles for every compute unit, but a chat's next turn (some dozens of new tokens
// behind a cached history of thousands) has two dozen such tiles, each a serial walk of hundreds of units
// (3 sequences of 17-70 tokens behind 5000-9000 keys, 32/8 heads: 171 us on 24 to 48 workgroups).
//
// Here a workgroup owns 32 query rows of one KV head, and each of its eight wavefronts takes every
// eighth 32-key chunk of the keys with a softmax state of its own; no barrier until the states are
// merged through LDS at the end.  That call takes 51 us.  What bounds it is the stream of K and V into one
// compute unit, because every workgroup reads all keys that its rows see, 512 bytes a key at D = 128: a
// loop of nothing but such loads reaches 100-120 GB/s per compute unit from the caches and 50 GB/s from
// HBM, however many loads are in flight; that call reads 7948 keys at 80 GB/s, start and merge included.  32 rows (not 16)
// so that half as many workgroups read the keys of a KV head; rows are HPW heads of the KV head's
// group times 32 / HPW tokens, because rows that share keys share the stream.
//  * K and V go HBM -> registers as whole head slices (1 KB per wave-wide load), then through a
//    wave-private LDS tile into MFMA operand order; the next chunk's loads are issued as soon as its
//    registers are free, so a wavefront keeps 8 to 16 KB in flight and a compute unit about 100 KB.
//  * No non-temporal hint: the workgroups of a KV head (on one XCD when Hkv is a multiple of eight) walk
//    the same keys at about the same time and share them in its L2.  (Starting the tiles of a sequence
//    at different places of the key axis, so that each fetches another part first, lost that sharing:
//    121 against 76 us for 3 sequences of 64 tokens behind 8192 keys.  Idle compute units that touched the keys
//    ahead gave 1 % on some shapes and cost as much on others.)
//  * Where even these workgroups leave compute units idle, a call that brings scratch memory has the keys of every
//    sequence cut into parts (grid dimension y): a part's workgroups leave records, which
//    prefill_split_merge_kernel merges (about 5 us with its launch).  2 x 4 tokens behind 5900 keys: 44 -> 18 us in
//    twelve parts, 2 x 9-12 behind 14000-18700 103 -> 32 us in eight; key_plan in attn_api.hip has the rule (from enough new tokens
//    for 128-row tiles on, the ring kernel in parts takes over).
//  * The reference of the exponentials moves only when a row outgrows it by 2^kSlack, as in the ring kernel (D = 128; at
//    D = 64 it is the running maximum).
#include "kernel_params.hpp"
#include "prefill_parts.hpp"

#include <type_traits>

namespace attn {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

struct SplitBf16 {
    typedef __bf16 elem;
    typedef __bf16 x8 __attribute__((ext_vector_type(8)));
    static constexpr int kDtype = kDtypeBf16;
    static __device__ __forceinline__ f32x16 mfma(x8 a, x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
struct SplitF16 {
    typedef _Float16 elem;
    typedef _Float16 x8 __attribute__((ext_vector_type(8)));
    static constexpr int kDtype = kDtypeF16;
    static __device__ __forceinline__ f32x16 mfma(x8 a, x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};

constexpr int kRows = kSplitRows;  // query rows (heads x tokens) of a workgroup
constexpr int kChunk = 32;   // keys per wavefront step
constexpr int kWaves = 8;
constexpr int kStep = kWaves * kChunk;  // keys per step of all wavefronts
// log2 of the largest weight tolerated before the reference moves, as in the ring kernel
template <int HD>
constexpr float kSlack = HD == 64 ? 0.f : 8.f;

template <int HD>
struct SplitCfg {
    static constexpr int kKPitch = HD * 2 + 16;  // bytes; consecutive rows start four banks apart (128-bit reads)
    static constexpr int kVPitch = HD * 2 + 64;  // bytes; for the transposing reads (same tile, after K)
    static constexpr int kTileBytes = kChunk * kVPitch;
    static constexpr int kRedPitch = HD + 4;     // floats per row of the final reduction
    static constexpr int kRedBytes = kWaves * kRows * kRedPitch * 4;
    static constexpr int kStateBytes = kWaves * kRows * 8;  // (reference, sum) of every wavefront and row
    static constexpr int kMainBytes = kWaves * kTileBytes > kRedBytes ? kWaves * kTileBytes : kRedBytes;
    static constexpr size_t kLdsBytes = kMainBytes + kStateBytes;
    static_assert(kKPitch <= kVPitch, "K uses the tile that V takes over");
    static_assert(kLdsBytes <= 160 * 1024, "LDS of one compute unit");
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float swap32_max(float x)
{
    const uint32_t u = __float_as_uint(x);
    const u32x2 r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float swap32_sum(float x)
{
    const uint32_t u = __float_as_uint(x);
    const u32x2 r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// What a workgroup of the unsplit grid (index w) stands for: hpw query heads of one KV head x tok tokens of one sequence.
struct SplitTile {
    int hpw, log_hpw, tok;
    int kvh, head0, s, q0, n_q, n_kv, off, t0;
    int kv0;       // packed keys: row of the sequence's first one
    int kv_end;    // keys that any row of the tile sees
    int part_len;  // keys of a part, a multiple of kStep
    int n_parts;   // parts of the tile that hold keys it sees (at least 1)
};
__device__ __forceinline__ SplitTile split_tile(const KParams &p, int w)
{
    touch_args(p);
    SplitTile t;
    t.hpw = split_heads(p.group);
    t.log_hpw = __builtin_ctz(t.hpw);
    t.tok = kRows >> t.log_hpw;
    const int q_tiles = (p.max_q_len + t.tok - 1) >> (__builtin_ctz(kRows) - t.log_hpw);
    const QuotRem by_kvh = divmod_uniform(w, p.num_kv_heads);  // KV head fastest, as in the other kernels
    const QuotRem by_hsub = divmod_uniform(by_kvh.quot, p.group >> t.log_hpw);
    const QuotRem by_seq = divmod_uniform(by_hsub.quot, p.num_seqs);
    t.kvh = by_kvh.rem;
    t.head0 = t.kvh * p.group + (by_hsub.rem << t.log_hpw);
    t.s = by_seq.rem;
    t.t0 = (q_tiles - 1 - by_seq.quot) * t.tok;  // costly (late) tiles first
    int q0 = load_uniform(p.query_start_loc, t.s), q1 = load_uniform(p.query_start_loc, t.s + 1), n_kv = load_uniform(p.seq_lens, t.s), kv0 = 0;
    if (!p.block_table) kv0 = load_uniform(p.kv_start_loc, t.s);
    asm volatile("" : "+s"(q0), "+s"(q1), "+s"(n_kv), "+s"(kv0));  // one round trip, ahead of every branch
    t.q0 = q0;
    t.n_q = q1 - q0;
    t.n_kv = n_kv;
    t.kv0 = kv0;
    t.off = t.n_kv - t.n_q;
    t.kv_end = t.n_kv;
    if (p.causal) {
        const int last_tok = t.t0 + t.tok < t.n_q ? t.t0 + t.tok : t.n_q;
        t.kv_end = t.off + last_tok < t.n_kv ? t.off + last_tok : t.n_kv;
    }
    // equal parts of the sequence (not of the tile: the tiles of a sequence then read the same keys at about the same time)
    t.part_len = t.n_kv;
    t.n_parts = 1;
    if (p.num_splits > 1) {
        t.part_len = ((t.n_kv + p.num_splits - 1) / p.num_splits + kStep - 1) & ~(kStep - 1);
        if (t.kv_end > t.part_len) t.n_parts = (t.kv_end + t.part_len - 1) / t.part_len;
    }
    return t;
}
template <typename E, int HD, bool PAGED>
__global__ __launch_bounds__(kWaves * 64) void prefill_split_kernel(const KParams p)
{
    using C = SplitCfg<HD>;
    using elem = typename E::elem;
    using x8 = typename E::x8;
    constexpr int KSTEPS = HD / 16;
    constexpr int DB = HD / 32;
    constexpr int CPR = HD / 8;              // 16-byte vectors of a row
    constexpr int RPL = 64 / CPR;            // rows covered by one wave-wide load
    constexpr int NLD = kChunk / RPL;        // loads per lane, for K and again for V
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    // ---- which part of the keys (outermost: the tiles of a sequence walk a part side by side) of which tile ----
    const int part = (int)blockIdx.y, w = (int)blockIdx.x;
    const SplitTile T = split_tile(p, w);
    const int hpw = T.hpw, log_hpw = T.log_hpw;
    const int kvh = T.kvh, head0 = T.head0, s = T.s;
    const int q0 = T.q0, n_q = T.n_q, n_kv = T.n_kv, off = T.off, t0 = T.t0;
    if (t0 >= n_q || part >= T.n_parts) return;
    const int kv_begin = part * T.part_len;
    const int kv_end = T.kv_end < kv_begin + T.part_len ? T.kv_end : kv_begin + T.part_len;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lhalf = lane >> 5;
    const int l32 = lane & 31;

    // scores are exponentiated as 2^(c*s - ref); a negative scale is moved into Q (sign flips are exact)
    const float c = fabsf(p.scale_log2e);
    const bool negate_q = p.scale_log2e < 0.f;

    // ---- Q fragments (B operand): lane holds query row l32 = (token l32 / hpw, head l32 % hpw) ----
    x8 qf[KSTEPS];
    int limit;  // last key that this lane's row sees
    {
        int t = t0 + (l32 >> log_hpw);
        t = t < n_q ? t : n_q - 1;
        const elem *src = (const elem *)p.q + (int64_t)(q0 + t) * p.q_stride_tok + (int64_t)(head0 + (l32 & (hpw - 1))) * p.q_stride_head + 8 * lhalf;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            u32x4 raw = *(const u32x4 *)(src + 16 * ks);
            if (negate_q) raw ^= 0x80008000u;
            qf[ks] = __builtin_bit_cast(x8, raw);
        }
        limit = p.causal && off + t < n_kv - 1 ? off + t : n_kv - 1;
    }

    // ---- the first key that some row of the tile does not see ----
    int open_end = n_kv;
    if (p.causal) open_end = off + t0 + 1 < n_kv ? off + t0 + 1 : n_kv;

    // ---- loads: a wave-uniform base per 16-key group plus a 32-bit offset per lane ----
    const unsigned char *kbase = (const unsigned char *)p.k + (int64_t)kvh * p.kv_stride_head * 2;
    const unsigned char *vbase = (const unsigned char *)p.v + (int64_t)kvh * p.kv_stride_head * 2;
    typedef const __attribute__((address_space(4))) int32_t *table_ptr;  // read-only, scalar loads
    const table_ptr bt_row = PAGED ? (table_ptr)(p.block_table + (int64_t)s * p.block_table_stride) : (table_ptr) nullptr;
    const int kv0 = T.kv0;
    const uint32_t tok_bytes = (uint32_t)p.kv_stride_tok * 2;
    const int ld_row = lane / CPR;
    const uint32_t ld_col = 16 * (lane % CPR);
    // byte offset of the first row of the 16-key group that holds key `key` (a multiple of 16, below n_kv)
    auto group_base = [&](int key) -> int64_t {
        if (!PAGED) return (int64_t)(kv0 + key) * tok_bytes;
        const int blk = bt_row[key >> p.block_shift];
        return (int64_t)blk * p.kv_stride_block * 2 + (int64_t)(key & (p.block_size - 1)) * tok_bytes;
    };
    struct Bases {
        int64_t g0, g1;
    };
    // the two 16-key groups of the chunk at key c0 < n_kv; rows past the end of the sequence are never read
    auto bases = [&](int c0) -> Bases {
        const int64_t g0 = group_base(c0);
        return Bases{g0, c0 + 16 < n_kv ? group_base(c0 + 16) : g0};
    };
    // Rows past the end re-read the last key (their weight is zero, the value is finite).  Straight-line code:
    // with a branch around some of the loads the compiler cannot count how many are in flight and waits for
    // the next chunk's K where it needs this chunk's V (74 instead of 52 us for 8192 keys).
    auto load_chunk = [&](u32x4 (&dst)[NLD], const unsigned char *base, const Bases &b, int c0) {
        const int last = n_kv - 1 - c0 < kChunk - 1 ? n_kv - 1 - c0 : kChunk - 1;
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int row = ld_row + RPL * i < last ? ld_row + RPL * i : last;  // (rows of one load lie in one 16-key group)
            dst[i] = *(const u32x4 *)(base + (RPL * i < 16 ? b.g0 : b.g1) + (uint32_t)((uint32_t)(row & 15) * tok_bytes + ld_col));
        }
    };

    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[db][v] = 0.f;
    float m_ref = -INFINITY, l_run = 0.f;

    unsigned char *tile = lds + wave * C::kTileBytes;
    const unsigned char *k_rd = tile + l32 * C::kKPitch + 16 * lhalf;
    // transposing V read: lane supplies row (lane%16)/4 (+4*lhalf) and 4 channels at 4*(lane%4) + 16*((lane/16)%2)
    const unsigned char *v_rd = tile + (((lane & 15) >> 2) + 4 * lhalf) * C::kVPitch + (4 * (lane & 3) + 16 * ((lane >> 4) & 1)) * 2;
    unsigned char *k_wr = tile + ld_row * C::kKPitch + ld_col;
    unsigned char *v_wr = tile + ld_row * C::kVPitch + ld_col;

    u32x4 kreg[NLD], vreg[NLD];
    // one chunk: multiply, and (MORE) request the wave's next one, whose bases are in bn
    Bases bn{0, 0};
    auto step = [&](int c0, auto more_tag) {
        constexpr bool MORE = decltype(more_tag)::value;
        // ---- K through the wave's tile into the score MFMAs; its registers take the next chunk's K ----
        // (LDS instructions of one wave execute in order: no wait is needed between the uses of the tile)
#pragma unroll
        for (int i = 0; i < NLD; ++i) *(u32x4 *)(k_wr + RPL * i * C::kKPitch) = kreg[i];
        if (MORE) load_chunk(kreg, kbase, bn, c0 + kStep);
        __builtin_amdgcn_sched_barrier(0);  // (the compiler would sink these loads to V's, behind the wait for V)
        f32x16 sacc;
#pragma unroll
        for (int v = 0; v < 16; ++v) sacc[v] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) sacc = E::mfma(*(const x8 *)(k_rd + 32 * ks), qf[ks], sacc);
#pragma unroll
        for (int i = 0; i < NLD; ++i) *(u32x4 *)(v_wr + RPL * i * C::kVPitch) = vreg[i];
        if (MORE) {
            load_chunk(vreg, vbase, bn, c0 + kStep);
            const int after = c0 + 2 * kStep;
            bn = bases(after < kv_end ? after : c0);
            __builtin_amdgcn_sched_barrier(0);
        }

        // ---- softmax: lane holds keys c0 + 8*(v/4) + v%4 + 4*lhalf of its row ----
        if (c0 + kChunk > open_end) {
            const int rel = limit - c0 - 4 * lhalf;
#pragma unroll
            for (int v = 0; v < 16; ++v) sacc[v] = (8 * (v >> 2) + (v & 3)) > rel ? -INFINITY : sacc[v] * c;
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) sacc[v] *= c;
        }
        float mx = fmaxf(fmaxf(sacc[0], sacc[1]), sacc[2]);
#pragma unroll
        for (int v = 3; v < 15; v += 2) mx = fmaxf(fmaxf(mx, sacc[v]), sacc[v + 1]);
        mx = swap32_max(fmaxf(mx, sacc[15]));
        if (__builtin_amdgcn_ballot_w64(mx > m_ref + kSlack<HD>) != 0) {
            const float m_new = fmaxf(m_ref, mx);
            // (a row that has seen no key yet keeps -inf: a later chunk may hold its first one)
            const float alpha = m_new == -INFINITY ? 0.f : fast_exp2(m_ref - m_new);
            m_ref = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) oacc[db] *= alpha;
        }
        const float ref = m_ref == -INFINITY ? 0.f : m_ref;
        x8 pf[2];
        float sum0 = 0.f, sum1 = 0.f;
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
            const float e0 = fast_exp2(sacc[v] - ref), e1 = fast_exp2(sacc[v + 1] - ref);
            sum0 += e0;
            sum1 += e1;
            pf[v >> 3][v & 7] = (elem)e0;
            pf[v >> 3][(v & 7) + 1] = (elem)e1;
        }
        l_run += sum0 + sum1;

        // ---- O^T += V^T P^T ----
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const unsigned char *a = v_rd + 16 * ks * C::kVPitch + db * 64;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)a);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(a + 8 * C::kVPitch));
                const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                oacc[db] = E::mfma(__builtin_bit_cast(x8, both), pf[ks], oacc[db]);
            }
        }
    };
    int c0 = kv_begin + wave * kChunk;
    if (c0 < kv_end) {
        const Bases b = bases(c0);
        load_chunk(kreg, kbase, b, c0);
        __builtin_amdgcn_sched_barrier(0);
        load_chunk(vreg, vbase, b, c0);
        bn = bases(c0 + kStep < kv_end ? c0 + kStep : c0);
        for (; c0 + kStep < kv_end; c0 += kStep) step(c0, std::integral_constant<bool, true>{});
        step(c0, std::integral_constant<bool, false>{});
    }

    // ---- merge the wavefronts: reference and sum of every row first, then the scaled outputs ----
    // A wavefront without a visible key for a row has sum 0 and must not raise the common reference.
    const float l_all = swap32_sum(l_run);
    float *state = (float *)(lds + C::kMainBytes);
    if (lhalf == 0) *(float2 *)(state + 2 * (wave * kRows + l32)) = float2{l_all > 0.f ? m_ref : -INFINITY, l_all};
    __syncthreads();  // also: every wavefront is done with its tile
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) m_all = fmaxf(m_all, state[2 * (w * kRows + l32)]);
    const float mine = l_all > 0.f ? fast_exp2(m_ref - m_all) : 0.f;
    {
        float *red = (float *)lds + (wave * kRows + l32) * C::kRedPitch + 4 * lhalf;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq)
                *(f32x4 *)(red + db * 32 + 8 * vq) = f32x4{oacc[db][4 * vq], oacc[db][4 * vq + 1], oacc[db][4 * vq + 2], oacc[db][4 * vq + 3]} * mine;
    }
    __syncthreads();
    // thread -> (row, eight channels)
    for (int i = tid; i < kRows * CPR; i += kWaves * 64) {
        const int row = i / CPR, ch = 8 * (i % CPR);
        const int t = t0 + (row >> log_hpw);
        if (t >= n_q) continue;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) M = fmaxf(M, state[2 * (w * kRows + row)]);
        float L = 0.f;
        f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float2 ml = *(const float2 *)(state + 2 * (w * kRows + row));
            L += ml.y > 0.f ? ml.y * fast_exp2(ml.x - M) : 0.f;
            const float *red = (const float *)lds + (w * kRows + row) * C::kRedPitch + ch;
            a += *(const f32x4 *)red;
            b += *(const f32x4 *)(red + 4);
        }
        if (T.n_parts > 1) {  // one of several parts: left for the merge
            static_assert(kRows == 32, "rows of a record");
            float *rec = p.workspace + ((int64_t)w * p.num_splits + part) * kRecordFloats<HD>;
            *(f32x4 *)(rec + row * HD + ch) = a;
            *(f32x4 *)(rec + row * HD + ch + 4) = b;
            if (ch == 0) *(float2 *)(rec + kRows * HD + 2 * row) = float2{M, L};
            continue;
        }
        const float inv = L > 0.f ? 1.f / L : 0.f;  // (a query without a visible key gets zeros)
        x8 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = (elem)(a[e] * inv);
            o[4 + e] = (elem)(b[e] * inv);
        }
        *(x8 *)((elem *)p.out + (int64_t)(q0 + t) * p.o_stride_tok + (int64_t)(head0 + (row & (hpw - 1))) * p.o_stride_head + ch) = o;
    }
}

// Merges the parts of a tile: a thread owns four channels of a row.  Bound by latency (a launch, the lengths, the records).
template <typename E, int HD>
__global__ __launch_bounds__(kMergeThreads) void prefill_split_merge_kernel(const KParams p)
{
    using elem = typename E::elem;
    typedef elem x4 __attribute__((ext_vector_type(4)));
    const int w = (int)blockIdx.x / kMergeBlocks<HD>;
    const SplitTile T = split_tile(p, w);
    const int i = (int)blockIdx.x % kMergeBlocks<HD> * kMergeThreads + (int)threadIdx.x;
    const int row = i / (HD / 4), ch = 4 * (i % (HD / 4));
    const int t = T.t0 + (row >> T.log_hpw);
    if (T.n_parts <= 1 || t >= T.n_q) return;
    const float4 o = merge_records<HD>(p.workspace + (int64_t)w * p.num_splits * kRecordFloats<HD>, T.n_parts, i, row);
    *(x4 *)((elem *)p.out + (int64_t)(T.q0 + t) * p.o_stride_tok + (int64_t)(T.head0 + (row & (T.hpw - 1))) * p.o_stride_head + ch) =
        x4{(elem)o.x, (elem)o.y, (elem)o.z, (elem)o.w};
}

template <typename E, int HD>
bool split_valid(const KParams &p)
{
    // (offsets inside a 16-key group are 32 bits)
    return p.dtype == E::kDtype && p.head_dim == HD && (uint64_t)p.kv_stride_tok * 32 < (1ull << 32);
}

template <typename E, int HD, bool PAGED>
hipError_t split_launch_impl(const KParams &p, hipStream_t stream, unsigned tiles)
{
    auto kern = prefill_split_kernel<E, HD, PAGED>;
    static std::atomic<uint64_t> granted{0};
    const hipError_t allowed = allow_dynamic_lds((const void *)kern, SplitCfg<HD>::kLdsBytes, granted);
    if (allowed != hipSuccess) return allowed;
    hipLaunchKernelGGL(kern, dim3(tiles, (unsigned)p.num_splits), dim3(kWaves * 64), SplitCfg<HD>::kLdsBytes, stream, p);
    return hipGetLastError();
}

template <typename E, int HD>
hipError_t split_launch(const KParams &p, hipStream_t stream)
{
    const int64_t tiles = split_workgroups(p);
    if (tiles <= 0) return hipSuccess;
    if (tiles > 0x7fffffff) return hipErrorInvalidConfiguration;
    const hipError_t e = p.block_table ? split_launch_impl<E, HD, true>(p, stream, (unsigned)tiles)
                                       : split_launch_impl<E, HD, false>(p, stream, (unsigned)tiles);
    if (e != hipSuccess || p.num_splits <= 1) return e;
    hipLaunchKernelGGL((prefill_split_merge_kernel<E, HD>), dim3((unsigned)(tiles * kMergeBlocks<HD>)), dim3(kMergeThreads), 0, stream, p);
    return hipGetLastError();
}

#define SPLIT_INSTANCE(E, NAME, HD)                                                                      \
    {                                                                                                    \
        NAME "_keysplit d" #HD " w8", kRows, kChunk, kWaves, 0, 2, 0, split_valid<E, HD>, split_launch<E, HD>, 0, false, true \
    }

}  // namespace

const Instance *prefill_split_instances(int *count)
{
    static const Instance table[] = {
        SPLIT_INSTANCE(SplitBf16, "prefill_bf16", 128),
        SPLIT_INSTANCE(SplitBf16, "prefill_bf16", 64),
        SPLIT_INSTANCE(SplitF16, "prefill_f16", 128),
        SPLIT_INSTANCE(SplitF16, "prefill_f16", 64),
    };
    *count = (int)(sizeof(table) / sizeof(table[0]));
    return table;
}

}  // namespace attn
