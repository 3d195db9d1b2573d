// Kernel-side view of one attention call and the launcher table shared by the
// host dispatcher, the tuner and the kernel translation units.
//
// Notation follows the problem statement of the paper's study (section "Method
// and Investigated Kernels"): Q/K/V, query heads Hq, KV heads Hkv, head size D,
// a batch of sequences of different lengths, a causal mask; the paged KV cache
// with its block table is the PagedAttention layout the paper cites.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace attn {

// element types of q, k, v, out (the values of attn_dtype in the C ABI)
constexpr int kDtypeF32 = 0, kDtypeBf16 = 1, kDtypeF16 = 2;

struct KParams {
    const void *q;
    void *out;
    const void *k;
    const void *v;
    const int32_t *block_table;  // nullptr -> contiguous K/V
    const int32_t *query_start_loc;  // nullptr in decode (one token per sequence)
    const int32_t *kv_start_loc;
    const int32_t *seq_lens;
    int64_t q_stride_tok, q_stride_head;
    int64_t o_stride_tok, o_stride_head;
    int64_t kv_stride_block, kv_stride_tok, kv_stride_head;
    int32_t dtype;  // kDtype*
    int32_t num_seqs, num_q_heads, num_kv_heads, head_dim;
    int32_t group;  // Hq / Hkv
    int32_t block_table_stride;
    int32_t block_size, block_shift;  // block_size == 1 << block_shift when block_shift >= 0
    int32_t total_q, max_q_len, max_kv_len;
    float scale;        // softmax scale
    float scale_log2e;  // scale * log2(e): scores are exponentiated with exp2
    int32_t causal;
    // split-K decode, and prefill of few query rows over many keys
    float *workspace;
    int32_t num_splits;  // parts the key axis is cut into (grid dimension)
    int32_t split_len;   // keys per part, a multiple of the kernel's key tile
    // prefill grid order: 0 = query tiles outermost (the longest tiles of all sequences start first),
    // 1 = sequences outermost (all tiles of a sequence run together and share its K/V in one L2)
    int32_t tile_order;
};

// First statement of a kernel: asks for one field of each of the four cache lines that the argument struct spans, so that they
// arrive together.  Left alone the compiler loads a field where it is first needed, and the start of a kernel is a chain of
// misses, one after the other.  With the divisions below, scalar table entries and the merge's early requests, GPU time of
// whole calls: one context of 1900 keys 8.1 -> 7.5 us, 17 of 33-271 6.8 -> 6.3, 14 of 402 at D = 64 6.4 -> 5.7, 40 of 100-400
// 12.2 -> 11.8, fp32 prefill of 2 x 7-21 tokens 4.4 -> 4.2, 8 x 400-1800 bf16 tokens 128.3 -> 127.3.
static_assert(offsetof(KParams, seq_lens) / 64 == 0 && offsetof(KParams, kv_stride_tok) / 64 == 1 && offsetof(KParams, group) / 64 == 2 &&
                  offsetof(KParams, num_splits) / 64 == 3 && sizeof(KParams) <= 256,
              "a field of every line");
__device__ __forceinline__ void touch_args(const KParams &p)
{
    asm volatile("" : : "s"(p.seq_lens), "s"(p.kv_stride_tok), "s"(p.group), "s"(p.num_splits));
}

// Block-index arithmetic at the start of a kernel: x / d and x % d of wave-uniform, non-negative values.  The divisors are head
// counts more often than not, i.e. powers of two: a shift then, instead of some thirty dependent instructions each
// (three or four of them stood in front of the first load of every kernel).
__device__ __forceinline__ int div_uniform(int x, int d)
{
    if ((d & (d - 1)) == 0) return x >> __builtin_ctz(d);
    int q = __builtin_amdgcn_readfirstlane(x / d);
    asm volatile("" : "+s"(q));  // (keeps the division in a branch of its own)
    return q;
}
struct QuotRem {
    int quot, rem;
};
__device__ __forceinline__ QuotRem divmod_uniform(int x, int d)
{
    const int q = div_uniform(x, d);
    return QuotRem{q, x - q * d};
}

// Element i of a read-only array that every lane wants (a length, an offset): through the scalar cache.  (The compiler cannot
// know that no store changes it and would take a vector load.)
__device__ __forceinline__ int32_t load_uniform(const int32_t *base, int64_t i)
{
    return ((const __attribute__((address_space(4))) int32_t *)base)[i];
}

// Values of the lanes 16 and 32 apart, through the vector pipe (__shfl_xor goes through LDS: some 120 cycles each, one after the other
// in the middle of every chunk's softmax).  A pair comes in either order, which is all that a maximum or a sum asks for.  GPU time,
// the same bits: fp32 prefill of 128 tokens 5.3 -> 5.2 us, 2 x 100-250 10.0 -> 9.8, decode of 14 x 99-495 at D = 64 7.1 -> 7.0, 23 x
// 60-304 7.7 -> 7.6; one context of 1900 level.
struct LanePair {
    float a, b;
};
__device__ __forceinline__ LanePair swap_lanes16(float x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return LanePair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ LanePair swap_lanes32(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return LanePair{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
// maximum and sum over the lanes that differ in bits 4 and 5 alone, in all of them
__device__ __forceinline__ float max_over_groups(float x)
{
    const LanePair p = swap_lanes16(x);
    const LanePair q = swap_lanes32(fmaxf(p.a, p.b));
    return fmaxf(q.a, q.b);
}
__device__ __forceinline__ float sum_over_groups(float x)
{
    const LanePair p = swap_lanes16(x);
    const LanePair q = swap_lanes32(p.a + p.b);
    return q.a + q.b;
}

// One ahead-of-time compiled template instance: the unit the autotuner sweeps
// (the paper's "kernel configuration"; its requirement list asks for a way to
// declare the parameter space together with the dependencies between
// parameters -- here `valid` is that predicate).
struct Instance {
    const char *name;
    int block_m;  // query rows (token x head) per workgroup
    int block_n;  // keys per tile
    int waves;    // wavefronts per workgroup
    int heads_per_wg;  // query heads of one KV head packed into a workgroup
    int stages;   // K/V tiles in flight (pipeline depth)
    int split_len;  // decode: keys per split-K part (0 = never split); prefill: 0
    bool (*valid)(const KParams &);
    hipError_t (*launch)(const KParams &, hipStream_t);
    int variant = 0;  // prefill: KParams::tile_order this instance launches with; decode: 0
    bool per_head = false;  // decode: fixed parts with one wavefront per KV head (otherwise all wavefronts share a KV head)
    bool key_parts = false;  // prefill: the keys may be cut into KParams::num_splits parts, whose records go to the workspace
};

const Instance *prefill_instances(int *count);         // all prefill instances, ring variants first
const Instance *prefill_ring_instances(int *count);    // LDS-ring, software-pipelined (D = 64, 128), bf16
const Instance *prefill_ring_f16_instances(int *count);  // the same kernel for fp16
const Instance *prefill_staged_instances(int *count);  // register-staged double buffer (D = 64, 128)
const Instance *prefill_staged_f16_instances(int *count);  // the same kernel for fp16
const Instance *prefill_split_instances(int *count);  // few query rows, wavefronts split the keys; bf16 and fp16
const Instance *decode_instances(int *count);       // bf16
const Instance *decode_f16_instances(int *count);   // the same kernels for fp16

hipError_t launch_prefill_f32(const KParams &, hipStream_t);
hipError_t launch_decode_combine(const KParams &, hipStream_t);
hipError_t launch_decode_combine_f16(const KParams &, hipStream_t);

// Lets `kernel` be launched with `bytes` of dynamic LDS on the current device.  HIP keeps this permission per device, so
// it is asked for on the first launch on each (bit d of `granted`, one word per kernel, stands for device d).
inline hipError_t allow_dynamic_lds(const void *kernel, size_t bytes, std::atomic<uint64_t> &granted)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
    if (granted.load(std::memory_order_relaxed) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) granted.fetch_or(bit, std::memory_order_relaxed);
    return e;
}

// Floats per (sequence, query head, split) in the split-K workspace: D partial
// outputs followed by the running max and the running sum.
inline int partial_stride(int head_dim) { return head_dim + 2; }

// The key-split prefill kernel (prefill_split.hip): rows (heads x tokens) of a workgroup, the query heads that share one
// (a power of two, at most 32, that divides the group), and the workgroups of a call whose keys are not cut into parts.
constexpr int kSplitRows = 32;
__host__ __device__ inline int split_heads(int group)
{
    const int h = group & -group;
    return h < kSplitRows ? h : kSplitRows;
}
inline int64_t split_workgroups(const KParams &p)
{
    const int heads = split_heads(p.group), tok = kSplitRows / heads;
    return (int64_t)p.num_seqs * ((p.max_q_len + tok - 1) / tok) * (p.num_q_heads / heads);
}

}  // namespace attn
