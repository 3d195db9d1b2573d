// KV-cache write: scatters the keys and values of new tokens into the paged cache by slot mapping
// (the step in front of paged attention; layout as in the PagedAttention work the paper cites).
// A copy bound by memory: each lane moves 16-byte vectors, a token row of K and of V is covered by consecutive
// lanes.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/attn.h"

namespace attn {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct KvWriteParams {
    const unsigned char *k_new, *v_new;
    unsigned char *k_cache, *v_cache;
    const int32_t *slot_mapping;
    int64_t new_tok_bytes, new_head_bytes, blk_bytes, tok_bytes, head_bytes;
    int32_t num_tokens, num_kv_heads, vec_per_head, block_size;
};

// A thread takes the same 16-byte vector of the K and V rows of TOKS consecutive tokens: 2 TOKS loads in flight, and one
// division for all of them.  Four tokens from kBulkVectors on (16 MiB: two wavefronts per SIMD are left), one below,
// where more wavefronts matter more.
//  * Four tokens whose slots are all negative are left out before their rows are read (batches padded to a captured
//    size); the rows then wait for the slots, 0.25 us of a full call of 8192 tokens.  With one token per thread the rows are
//    requested together with the slot (1024 tokens 3.3 -> 3.0 us, level where most are padding).
//  * The stores of calls from kHintVectors on carry the non-temporal hint (they need not displace what the last-level
//    cache holds of the new keys).  Below, the call that reads the keys next pays for it: a write of 64 tokens and the
//    prefill over them 11.05 us with the hint, 10.80 without, one token and a decode step over 20 keys 6.78 and 6.63; 256
//    tokens and their decode step 32.1 and 32.6, a write of 2048 tokens alone 3.7 and 4.3.  The loads carry it from
//    kStreamVectors on (96 MiB, more than a third of that cache; measured at 64 and 128 MiB).  A prefill over what a
//    bulk call wrote takes the same time within 1 %.
// Bf16, D = 128, calls on three sets of buffers in turn, against one vector of K or V per thread with 64-bit divisions,
// no hints and padding skipped:
//   tokens x heads                 4096 x 8   8192 x 8   16384 x 8
//   before                           7.8       12.1        27.4 us
//   now                              6.9       11.5        21.3
//   before, 97 % padding at the end  3.4        4.6         7.1
//   now                              3.2        3.3         3.6
constexpr int64_t kHintVectors = 1 << 15;
constexpr int64_t kBulkVectors = 1 << 20;
constexpr int64_t kStreamVectors = 6 << 20;

template <bool HINT>
__device__ __forceinline__ u32x4 load(const unsigned char *src)
{
    return HINT ? __builtin_nontemporal_load((const u32x4 *)src) : *(const u32x4 *)src;
}
template <bool HINT>
__device__ __forceinline__ void store(unsigned char *dst, u32x4 v)
{
    if (HINT)
        __builtin_nontemporal_store(v, (u32x4 *)dst);
    else
        *(u32x4 *)dst = v;
}

template <int TOKS, bool HINT_LOAD, bool HINT_STORE>
__global__ __launch_bounds__(256) void kv_cache_write_kernel(const KvWriteParams p)
{
    const uint32_t row = (uint32_t)p.num_kv_heads * p.vec_per_head;  // vectors of a token's K (and V) row
    const uint32_t groups = ((uint32_t)p.num_tokens + TOKS - 1) / TOKS;
    const uint64_t total = (uint64_t)groups * row;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < total; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t grp = total >> 32 ? (uint32_t)(i / row) : (uint32_t)i / row;
        const uint32_t r = (uint32_t)(i - (uint64_t)grp * row);
        const uint32_t h = r / (uint32_t)p.vec_per_head, c = r - h * (uint32_t)p.vec_per_head;
        const int t0 = (int)(grp * TOKS), left = p.num_tokens - t0;  // tokens from t0 on
        const int64_t src0 = (int64_t)t0 * p.new_tok_bytes + h * p.new_head_bytes + 16 * c;
        int slot[TOKS];
        u32x4 k[TOKS], v[TOKS];
        int all = -1;  // negative if every slot is
#pragma unroll
        for (int j = 0; j < TOKS; ++j) {
            slot[j] = p.slot_mapping[t0 + (j < left ? j : left - 1)];  // past the last token: its row again, not stored
            all &= slot[j];
        }
        if (TOKS > 1 && all < 0) continue;
#pragma unroll
        for (int j = 0; j < TOKS; ++j) {
            const int t = j < left ? j : left - 1;
            k[j] = load<HINT_LOAD>(p.k_new + src0 + t * p.new_tok_bytes);
            v[j] = load<HINT_LOAD>(p.v_new + src0 + t * p.new_tok_bytes);
        }
#pragma unroll
        for (int j = 0; j < TOKS; ++j) {
            if (j >= left || slot[j] < 0) continue;
            const int blk = slot[j] / p.block_size, off = slot[j] % p.block_size;
            const int64_t dst = blk * p.blk_bytes + off * p.tok_bytes + h * p.head_bytes + 16 * c;
            store<HINT_STORE>(p.k_cache + dst, k[j]);
            store<HINT_STORE>(p.v_cache + dst, v[j]);
        }
    }
}

template <int TOKS, bool HINT_LOAD, bool HINT_STORE>
void write_launch(const KvWriteParams &p, hipStream_t stream)
{
    const int64_t groups = ((int64_t)p.num_tokens + TOKS - 1) / TOKS;
    const int64_t want = (groups * p.num_kv_heads * p.vec_per_head + 255) / 256;
    const unsigned blocks = (unsigned)(want < 16384 ? want : 16384);  // grid-stride beyond that
    hipLaunchKernelGGL((kv_cache_write_kernel<TOKS, HINT_LOAD, HINT_STORE>), dim3(blocks), dim3(256), 0, stream, p);
}

}  // namespace
}  // namespace attn

extern "C" int attn_kv_cache_write(const attn_kv_write_args *a, void *hip_stream)
{
    using namespace attn;
    if (!a) return ATTN_ERR_NULL;
    if (a->struct_bytes != sizeof(attn_kv_write_args)) return ATTN_ERR_SHAPE;
    if (a->dtype != ATTN_BF16 && a->dtype != ATTN_F32 && a->dtype != ATTN_F16) return ATTN_ERR_DTYPE;
    const int esz = a->dtype == ATTN_F32 ? 4 : 2;
    if (a->num_tokens < 0 || a->num_kv_heads <= 0 || a->head_dim <= 0 || a->block_size <= 0 || a->num_blocks <= 0) return ATTN_ERR_SHAPE;
    if ((a->head_dim * esz) % 16 != 0) return ATTN_ERR_UNSUPPORTED;
    if (a->num_tokens == 0) return ATTN_OK;
    if (!a->k_new || !a->v_new || !a->k_cache || !a->v_cache || !a->slot_mapping) return ATTN_ERR_NULL;
    const int64_t strides[5] = {a->new_stride_tok, a->new_stride_head, a->kv_stride_block, a->kv_stride_tok, a->kv_stride_head};
    for (int64_t st : strides)
        if (st < a->head_dim || (st * esz) % 16 != 0) return ATTN_ERR_SHAPE;
    if (((uintptr_t)a->k_new | (uintptr_t)a->v_new | (uintptr_t)a->k_cache | (uintptr_t)a->v_cache) & 15) return ATTN_ERR_SHAPE;
    KvWriteParams p;
    p.k_new = (const unsigned char *)a->k_new;
    p.v_new = (const unsigned char *)a->v_new;
    p.k_cache = (unsigned char *)a->k_cache;
    p.v_cache = (unsigned char *)a->v_cache;
    p.slot_mapping = a->slot_mapping;
    p.new_tok_bytes = a->new_stride_tok * esz;
    p.new_head_bytes = a->new_stride_head * esz;
    p.blk_bytes = a->kv_stride_block * esz;
    p.tok_bytes = a->kv_stride_tok * esz;
    p.head_bytes = a->kv_stride_head * esz;
    p.num_tokens = a->num_tokens;
    p.num_kv_heads = a->num_kv_heads;
    p.vec_per_head = a->head_dim * esz / 16;
    p.block_size = a->block_size;
    const int64_t total = (int64_t)a->num_tokens * 2 * a->num_kv_heads * p.vec_per_head;
    if (total > ((int64_t)1 << 40)) return ATTN_ERR_SHAPE;
    const hipStream_t stream = (hipStream_t)hip_stream;
    if (total >= kStreamVectors)
        write_launch<4, true, true>(p, stream);
    else if (total >= kBulkVectors)
        write_launch<4, false, true>(p, stream);
    else if (total >= kHintVectors)
        write_launch<1, false, true>(p, stream);
    else
        write_launch<1, false, false>(p, stream);
    return hipGetLastError() == hipSuccess ? ATTN_OK : ATTN_ERR_HIP;
}
