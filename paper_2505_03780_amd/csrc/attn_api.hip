// C ABI of the attention library: argument validation, shape buckets, instance
// selection (winner cache, else heuristic), the in-library autotuner and its
// persistent cache.
//
// The tuner is the paper's thesis applied natively: instead of JIT-compiling
// configurations at first call, every configuration is a template instance
// compiled ahead of time; attn_tune times the valid ones for a shape bucket off
// the critical path and stores the winner, together with the environment it was
// measured in, in a file that later processes load (the paper's list of gaps
// towards practical autotuning: configuration spaces with parameter
// dependencies, reusable caches that record their environment, tuning moved off
// the critical path).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <mutex>
#include <sstream>
#include <string>
#include <unordered_map>
#include <vector>

#include <fcntl.h>
#include <sys/file.h>
#include <unistd.h>

#include "../../include/attn.h"
#include "kernel_params.hpp"
#include "tuner_cache.hpp"

namespace attn {
namespace {

constexpr const char *kCacheMagic = "attn-tune-cache-v1";
// Changes whenever the kernels change in a way that invalidates old timings.
// Identifies the set of compiled instances: a cache line tuned against another set must not be
// trusted (the paper asks that cached results record the environment they were measured in).
std::string build_id();
// Bounds on the split-K records of the fixed-split decode kernels: a context is cut into at most
// kMaxPartsPerSeq parts, and a batch into at most two parts per compute unit in all (more parts add
// workspace traffic and merge work, never parallelism: every part already is Hkv workgroups).
constexpr int kMaxPartsPerSeq = 64;
// The record array of attn_decode_paged_static.
constexpr size_t kScratchBytes = (size_t)16 << 20;

std::mutex g_mu;
std::unordered_map<std::string, int> g_winner[2];  // [is_decode]: bucket key -> instance id
std::unordered_map<std::string, std::string> g_named;  // other kernel kinds: bucket key -> instance name
std::atomic<int> g_forced[2] = {{-1}, {-1}};
bool g_env_cache_tried = false;
// bumped whenever the winner table may have changed (tune, load, clear): invalidates the per-thread memo
std::atomic<uint64_t> g_generation{1};

const Instance *all_decode_instances(int *count);
const Instance *instances(int is_decode, int *n) { return is_decode ? all_decode_instances(n) : prefill_instances(n); }
bool is16(int dtype) { return dtype == ATTN_BF16 || dtype == ATTN_F16; }

int ilog2_ceil(int64_t x)
{
    int r = 0;
    while (((int64_t)1 << r) < x) ++r;
    return r;
}

// ---- validation --------------------------------------------------------------------------------

int validate(const attn_args *a, int is_decode)
{
    if (!a) return ATTN_ERR_NULL;
    if (a->struct_bytes != sizeof(attn_args)) return ATTN_ERR_SHAPE;
    if (a->dtype != ATTN_F32 && !is16(a->dtype)) return ATTN_ERR_DTYPE;
    if (is_decode && !is16(a->dtype)) return ATTN_ERR_DTYPE;
    if (a->num_seqs < 0 || a->num_q_heads <= 0 || a->num_kv_heads <= 0 || a->total_q < 0 || a->max_q_len < 0 ||
        a->max_kv_len < 0)
        return ATTN_ERR_SHAPE;
    if (a->num_q_heads % a->num_kv_heads != 0) return ATTN_ERR_SHAPE;
    if (a->head_dim != 64 && a->head_dim != 128) return ATTN_ERR_UNSUPPORTED;
    if (is_decode && a->total_q != a->num_seqs) return ATTN_ERR_SHAPE;
    if (is_decode && a->max_q_len > 1) return ATTN_ERR_SHAPE;
    const int vec = is16(a->dtype) ? 8 : 1;  // elements per 16-byte vector access
    if (a->q_stride_head < a->head_dim || a->o_stride_head < a->head_dim || a->kv_stride_head < a->head_dim ||
        a->q_stride_tok <= 0 || a->o_stride_tok <= 0 || a->kv_stride_tok <= 0)
        return ATTN_ERR_SHAPE;
    if (a->q_stride_tok % vec || a->q_stride_head % vec || a->o_stride_tok % vec || a->o_stride_head % vec ||
        a->kv_stride_tok % vec || a->kv_stride_head % vec)
        return ATTN_ERR_SHAPE;
    if (a->block_table) {
        if (a->block_size < 16 || (a->block_size & (a->block_size - 1)) != 0) return ATTN_ERR_UNSUPPORTED;
        if (a->block_table_stride <= 0 || a->num_blocks <= 0 || a->kv_stride_block <= 0 || a->kv_stride_block % vec)
            return ATTN_ERR_SHAPE;
        if ((int64_t)a->block_table_stride * a->block_size < a->max_kv_len) return ATTN_ERR_SHAPE;
    } else if (is_decode) {
        return ATTN_ERR_NULL;  // decode is paged only
    }
    if (a->num_seqs == 0 || a->total_q == 0) return ATTN_OK;  // nothing to do; pointers may be NULL
    if (!a->q || !a->out || !a->seq_lens) return ATTN_ERR_NULL;
    if (a->max_kv_len > 0 && (!a->k || !a->v)) return ATTN_ERR_NULL;
    if (!is_decode && !a->query_start_loc) return ATTN_ERR_NULL;
    if (is16(a->dtype)) {
        const uintptr_t bits = (uintptr_t)a->q | (uintptr_t)a->out | (uintptr_t)a->k | (uintptr_t)a->v;
        if (bits & 15) return ATTN_ERR_SHAPE;  // 128-bit accesses
    }
    return ATTN_OK;
}

KParams to_kparams(const attn_args *a, int is_decode)
{
    KParams p{};
    p.dtype = a->dtype;
    p.q = a->q;
    p.out = a->out;
    p.k = a->k;
    p.v = a->v;
    p.block_table = a->block_table;
    p.query_start_loc = is_decode ? nullptr : a->query_start_loc;
    p.kv_start_loc = a->kv_start_loc ? a->kv_start_loc : a->query_start_loc;
    p.seq_lens = a->seq_lens;
    p.q_stride_tok = a->q_stride_tok;
    p.q_stride_head = a->q_stride_head;
    p.o_stride_tok = a->o_stride_tok;
    p.o_stride_head = a->o_stride_head;
    p.kv_stride_block = a->kv_stride_block;
    p.kv_stride_tok = a->kv_stride_tok;
    p.kv_stride_head = a->kv_stride_head;
    p.num_seqs = a->num_seqs;
    p.num_q_heads = a->num_q_heads;
    p.num_kv_heads = a->num_kv_heads;
    p.head_dim = a->head_dim;
    p.group = a->num_q_heads / a->num_kv_heads;
    p.block_table_stride = a->block_table_stride;
    p.block_size = a->block_table ? a->block_size : 0;
    p.block_shift = a->block_table ? ilog2_ceil(a->block_size) : 0;
    p.total_q = a->total_q;
    p.max_q_len = is_decode ? 1 : a->max_q_len;
    p.max_kv_len = a->max_kv_len;
    p.scale = a->scale;
    p.scale_log2e = a->scale * 1.4426950408889634f;
    p.causal = a->causal ? 1 : 0;
    p.workspace = is_decode ? (float *)a->workspace : nullptr;
    p.num_splits = 1;
    p.split_len = 0;
    return p;
}

// ---- shape buckets ------------------------------------------------------------------------------
// A bucket fixes everything a kernel instance is specialised on and rounds the three extents
// (sequences, longest query, longest context) up to powers of two.
std::string bucket_key(const KParams &p, int dtype, int is_decode)
{
    char buf[192];
    snprintf(buf, sizeof buf, "%s|%s|d%d|hq%d|hkv%d|%s|bs%d|c%d|B%d|q%d|kv%d", is_decode ? "decode" : "prefill",
             dtype == ATTN_BF16 ? "bf16" : dtype == ATTN_F16 ? "f16" : "f32", p.head_dim, p.num_q_heads, p.num_kv_heads,
             p.block_table ? "paged" : "contig", p.block_size, p.causal, ilog2_ceil(std::max(1, p.num_seqs)),
             ilog2_ceil(std::max(1, p.max_q_len)), ilog2_ceil(std::max(1, p.max_kv_len)));
    return buf;
}

// Keys of the buckets next to the one of `p`: one step up or down in each of the three extents.
std::vector<std::string> neighbour_keys(const KParams &p, int dtype, int is_decode)
{
    std::vector<std::string> out;
    for (int axis = 0; axis < 3; ++axis)
        for (int dir = -1; dir <= 1; dir += 2) {
            KParams q = p;
            int *ext = axis == 0 ? &q.num_seqs : axis == 1 ? &q.max_q_len : &q.max_kv_len;
            const int e = ilog2_ceil(std::max(1, *ext)) + dir;
            if (e < 0 || e > 30 || (axis == 1 && is_decode)) continue;
            *ext = 1 << e;
            out.push_back(bucket_key(q, dtype, is_decode));
        }
    return out;
}

constexpr int kMaxBalancedWgs = 2048;  // launch bound of the token-balanced decode

int compute_units()
{
    static std::atomic<int> cached{0};
    int cu = cached.load();
    if (cu > 0) return cu;
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 256;
    }
    cached.store(prop.multiProcessorCount);
    return prop.multiProcessorCount;
}

// Parts per sequence a fixed-split decode instance cuts the longest context into (1: no split).
int fixed_parts(const KParams &p, const Instance &inst)
{
    const int sl = inst.split_len;
    return (sl <= 0 || sl >= p.max_kv_len) ? 1 : (p.max_kv_len + sl - 1) / sl;
}

// The parameter-dependency predicate of an instance (the paper's requirement list asks for
// configuration spaces that carry the dependencies between parameters): the kernel's own conditions,
// and for a fixed-split decode instance the bound on the split-K records.
bool usable(const Instance &inst, const KParams &p, int is_decode)
{
    if (!inst.valid(p)) return false;
    if (!is_decode || inst.split_len <= 0) return true;
    const int parts = fixed_parts(p, inst);
    if (parts == 1) return true;
    return parts <= kMaxPartsPerSeq && (int64_t)p.num_seqs * parts <= std::max<int64_t>(2 * compute_units(), 2);
}

void apply_split(KParams &p, const Instance &inst)
{
    int sl = inst.split_len;
    if (sl < 0) {  // token-balanced: a fixed number of workgroups, each with an equal share of the chunks
        const int waves = inst.waves;
        const int head_blocks = (p.num_kv_heads + waves - 1) / waves;
        int wgs = compute_units() * (-sl) * (8 / waves) / head_blocks;
        wgs = std::max(1, std::min(wgs, kMaxBalancedWgs));
        p.num_splits = wgs;
        p.split_len = 0;
        return;
    }
    if (sl <= 0 || sl >= p.max_kv_len) {
        p.split_len = std::max(p.max_kv_len, 1);
        p.num_splits = 1;
    } else {
        p.split_len = sl;
        p.num_splits = (p.max_kv_len + sl - 1) / sl;
    }
}

size_t instance_workspace_bytes(const Instance &inst, const KParams &p_in);

// ---- built-in heuristic (used until a bucket has been tuned) -----------------------------------
int find_instance(int is_decode, const KParams &p, int waves, int hpw, int bn, int bm, int split_len, int variant = 0, int stages = 0,
                  bool per_head = false)
{
    int n;
    const Instance *t = instances(is_decode, &n);
    for (int i = 0; i < n; ++i) {
        if (!usable(t[i], p, is_decode)) continue;
        if (t[i].waves == waves && t[i].heads_per_wg == hpw && t[i].block_n == bn && (bm <= 0 || t[i].block_m == bm) &&
            t[i].split_len == split_len && t[i].variant == variant && (stages <= 0 || t[i].stages == stages) && t[i].per_head == per_head)
            return i;
    }
    return -1;
}

// Heads of a KV head that a ring workgroup packs: as many as divide the group, they share every K/V tile.
int ring_heads(const KParams &p) { return p.group % 4 == 0 ? 4 : p.group % 2 == 0 ? 2 : 1; }
// The ring kernel's 128-row workgroup with the tiles of a sequence side by side, whose keys can be cut into parts (-1: none).
int small_ring_instance(const KParams &p) { return find_instance(0, p, 4, ring_heads(p), 32, 128, 0, 1, 4); }

// Whether a prefill call has too few query rows to fill the chip with the ring kernel's 128- and 256-row
// workgroups, and enough keys that splitting them over the wavefronts of a 32-row workgroup pays
// (prefill_split.hip).  Measured on random shapes against the ring kernel (GPU time, 32/8, 64/8, 16/16, 16/4 and 8/2
// heads, bf16), where the lines below lie:
//  * up to one workgroup per compute unit the split is ahead from 160 keys on: at D = 128 200 keys 1.02-1.16x,
//    500 keys 1.2-1.4x (13.6 -> 10.3 us), 2000 keys 2x (31 -> 15 us), 8000-15000 keys 2.6-3.6x (322 -> 90 us), at
//    D = 64 1.15x, 1.4x (10.0 -> 7.1 us), 2x and 2.1-3.3x; below 160 keys they are level;
//  * up to two per compute unit it loses below about 1000 keys (D = 128: 24.6 against 22.0 us at 1121
//    keys, D = 64: 9.2 against 7.6 us at 252) and gains above (D = 128: 43 against 51 us at 1486 keys, 59
//    against 102 us at 4450; D = 64: 14.3 against 16.4 us at 1055, 32 against 84 us at 7700); beyond two the
//    ring is ahead but for the longest contexts.
bool few_rows_many_keys(const KParams &p)
{
    const int64_t wgs = split_workgroups(p);
    const int two_from = p.head_dim == 64 ? 1024 : 1536;
    return (p.max_kv_len >= 160 && wgs <= compute_units()) || (p.max_kv_len > two_from && wgs <= 2 * compute_units());
}

// The workgroups of a prefill call (of one part of the keys).
struct KeyTiles {
    int64_t grid;  // the longest query's tiles for every sequence
    int64_t busy;  // at most this many of them find work
};
KeyTiles row_tiles(const KParams &p, int rows, int heads)
{
    const int tok = rows / heads;
    const int64_t groups = p.num_q_heads / heads, grid = (int64_t)p.num_seqs * ((p.max_q_len + tok - 1) / tok) * groups;
    return KeyTiles{grid, std::min(grid, ((int64_t)p.total_q / tok + p.num_seqs) * groups)};
}
KeyTiles key_tiles(const Instance &inst, const KParams &p)
{
    return row_tiles(p, inst.block_m, inst.heads_per_wg > 0 ? inst.heads_per_wg : split_heads(p.group));
}
// The tiles of the ring kernel's 128-row workgroups: what the choice of a prefill instance takes from the number of tokens (with
// those of 256 rows in small_tiles_fit).
int64_t small_tiles(const KParams &p) { return row_tiles(p, 128, ring_heads(p)).busy; }
// Whether tiles that all cost about the same (no causal mask) are better off in the ring kernel's 128-row workgroups, two per compute
// unit, than in 256-row ones, one per compute unit.  A full round takes the same time for the same rows, within some 5 % in favour of the
// large one, so the small one gains where its last round is no more than half full (each with a compute unit to itself) while the large
// one's is a whole one, and where it has a tenth fewer rows of padding.
bool small_tiles_fit(const KParams &p)
{
    const int64_t cus = compute_units(), small = small_tiles(p), large = row_tiles(p, 256, ring_heads(p)).busy;
    return (small + cus - 1) / cus < 2 * ((large + cus - 1) / cus) || 5 * small < 9 * large;
}
// Whether the ring kernel's 128-row tiles are so few that a workgroup of two wavefront groups, each with half of the keys, is ahead of
// one group per tile (`id`: that instance).  GPU time on 4000 random causal shapes (batch 1-16, 8-8192 new tokens, 0-16384 cached ones,
// 32/8, 64/8, 16/16, 16/4 and 8/2 heads, bf16, built-in choice before against halves):
//  * at most one tile per compute unit: from 700 keys on 1.18x on average at D = 128 and 1.21x at D = 64 (1.24x and 1.25x from 1200
//    keys on), 0.5 and 1.4 % of the shapes lose more than 2 %; at 300-700 keys level on average, with shapes down to 0.77x, and
//    from 8192 keys on 1.07x against the ring kernel in parts (below), which is left to take over where a call brings scratch memory;
//  * up to two per compute unit one whole prompt gains from 1400 keys on (a triangle: the mean tile has half of the longest one's
//    keys): 1.11-1.46x at D = 128, 1.08-1.28x at D = 64, none of 130 loses; with less than 1400 keys 0.93-1.17x, with more tiles
//    0.80-1.18x, behind a cached prefix 0.89-1.0x, several sequences 0.79-1.3x.
// On 1212 other random shapes that take halves, 407 of them without a causal mask and a third fp16: 1.20x, without a mask 1.21x; 8 of 805 and 6
// of 407 lose more than 2 % (0.90x at worst), nearly all of them several sequences with 0.95 to 1 tile per compute unit in a larger
// grid, of which some XCDs are dealt more than their share.  Lines that keep those out (no grid beyond the compute units, or 7/8 of a tile each)
// take 33 to 102 shapes back that gain 1.09-1.18x from it.
bool halves_pay(const KParams &p, int id)
{
    if (id < 0) return false;
    const int64_t busy = small_tiles(p), cus = compute_units();
    const bool whole_prompt = p.num_seqs == 1 && p.causal && p.max_kv_len == p.max_q_len;
    return (busy <= cus && p.max_kv_len >= 700 && p.max_kv_len < 8192) || (whole_prompt && busy <= 2 * cus && p.max_kv_len >= 1400);
}

// ---- prefill whose keys are cut into parts over workgroups (a call that brings scratch memory) -----------------
size_t key_parts_bytes(const Instance &inst, const KParams &p, int parts)
{
    return parts <= 1 ? 0 : (size_t)key_tiles(inst, p).grid * inst.block_m * parts * partial_stride(p.head_dim) * sizeof(float);
}

// Time that a call is expected to take (us), by kernel; fitted to some 5900 random shapes (batch 1-32, 8-1024 new tokens,
// 500-20000 keys, up to 600 tiles of 128 rows) with 1 to 16 parts each.  Workgroups run in rounds of as many as are resident.
//  * Key-split kernel (32 rows): one workgroup per compute unit, 4 us for its start and its merge through LDS, 1.5 us (D = 64:
//    1 us) for each 256 keys.  A few workgroups beyond a round share compute units at little cost while the keys are whole (264 to
//    280 tiles take 1.0 to 1.2 rounds with uneven lengths or at D = 64, and two with even ones).  In parts the empty workgroups of the grid count too: they end at once, but XCDs are dealt
//    workgroups blindly, and some get full ones in excess (counting only the full ones, 2 x 52-133 tokens of 16/16 heads behind 5400 keys, 320
//    workgroups and 224 of them full, were expected to take 26 us, and took 52).
//  * Ring kernel, small workgroup (128 rows): two per compute unit, 8 us (4 us), 6 us (4.5 us) for each 256 keys, 4.5 us (3 us)
//    while each has a compute unit to itself.  Large workgroup (256 rows): one per compute unit, 8 us, 5.5 us for each 256 keys.
// The second kernel costs 5 to 8 us.
int64_t key_steps(const KParams &p, int parts) { return (((int64_t)p.max_kv_len + parts - 1) / parts + 255) / 256; }
double split_model_us(const KParams &p, const KeyTiles &tiles, int parts)
{
    const int64_t cus = compute_units(), n = parts == 1 ? tiles.busy : tiles.grid * parts;
    double rounds = (double)((n + cus - 1) / cus);
    if (parts == 1) {
        const double full = (double)n / (double)cus;
        rounds = std::min(rounds, full <= 1.1 ? std::max(1.0, 1.2 * full) : 1.4 * full);
    }
    return rounds * (4.0 + (p.head_dim == 64 ? 1.0 : 1.5) * (double)key_steps(p, parts)) + (parts > 1 ? 5.0 : 0.0);
}
double ring_model_us(const KParams &p, const KeyTiles &tiles, int parts)
{
    const bool small = p.head_dim == 64;
    const int64_t slots = 2 * compute_units(), n = tiles.busy * parts, rest = n % slots;
    const double steps = (double)key_steps(p, parts), start = small ? 4.0 : 8.0;
    double us = (double)(n / slots) * (start + (small ? 4.5 : 6.0) * steps);
    if (rest > 0) us += start + (2 * rest <= slots ? (small ? 3.0 : 4.5) : (small ? 4.5 : 6.0)) * steps;
    return us + (parts > 1 ? 8.0 : 0.0);
}
// The instance that a plan would replace, with whole keys.
double whole_model_us(const Instance &inst, const KParams &p)
{
    const KeyTiles tiles = key_tiles(inst, p);
    if (inst.heads_per_wg == 0) return split_model_us(p, tiles, 1);
    if (inst.block_m == 128 && inst.waves == 8) {  // halves; the tiles of a whole prompt are a triangle
        const double rounds = (double)tiles.busy / (double)compute_units() * (p.num_seqs == 1 && p.max_kv_len == p.max_q_len ? 0.7 : 1.0);
        return std::max(1.0, rounds) * (7.0 + (p.head_dim == 64 ? 2.5 : 3.6) * (double)p.max_kv_len / 256.0);
    }
    if (inst.block_m == 128) return ring_model_us(p, tiles, 1);
    return std::max(1.0, (double)tiles.busy / (double)compute_units()) * (8.0 + 5.5 * (double)key_steps(p, 1));
}

struct KeyPlan {
    int id = -1;    // instance
    int parts = 1;  // 1: the call does not use scratch memory
};
constexpr int kMaxSplitParts = 32, kMaxRingParts = 16;
// The fastest number of parts of instance `id` by its model, if less than `us`.
void try_parts(const KParams &p, int id, double *us, KeyPlan *plan)
{
    int n;
    const Instance &inst = instances(0, &n)[id];
    const KeyTiles tiles = key_tiles(inst, p);
    const bool ring = inst.heads_per_wg > 0;
    // Four records of 32 rows per compute unit (17 MB); of 128 rows two, not counting every tile's first part, so four at two parts
    // (68 MB) and fewer at more.
    const int64_t most = ring ? 2 * (int64_t)compute_units() + tiles.grid : 4 * (int64_t)compute_units();
    for (int parts = 2; parts <= (ring ? kMaxRingParts : kMaxSplitParts) && tiles.grid * parts <= most; ++parts) {
        const double t = ring ? ring_model_us(p, tiles, parts) : split_model_us(p, tiles, parts);
        if (t < *us) {
            *us = t;
            *plan = KeyPlan{id, parts};
        }
    }
}

// What a prefill call that would otherwise run instance `id` does with scratch memory.  The margins are set so that next to
// nothing loses: of 57100 random calls that take parts (half of the ranges above, down to one new token and with uneven lengths; half
// drawn like the calls of perf/cases.py) 0.2 % are more than 2 % behind no parts and 0.04 % more than 10 %, nearly all of them batches of
// very uneven lengths, whose maxima are all that the host knows; the average gain is 1.7x.  Examples (no parts ->
// parts, GPU time): 2 x 4 tokens behind 5900 keys 44 -> 18 us, 2 x 9-12 behind 14000-18700 103 -> 32, 3 x 17-70 behind 5000-9000 54 -> 42,
// 4 x 200 behind 6000 137 -> 112, 3 x 390-450 of 16/16 heads behind 3900 99 -> 79.
KeyPlan key_plan(const KParams &p, int id, bool forced)
{
    int n;
    const Instance *t = instances(0, &n);
    const bool split = t[id].key_parts && t[id].heads_per_wg == 0, small_ring = t[id].key_parts && !split;
    KeyPlan plan{id, 1};
    if (p.max_kv_len <= 1024) return plan;
    const int64_t cus = compute_units();
    const double whole = whole_model_us(t[id], p);
    if (split) {
        // 15 % ahead or not at all, 25 % from half a workgroup per compute unit on, where uneven lengths decide
        const int64_t busy = key_tiles(t[id], p).busy;
        double us = whole / (2 * busy > cus ? 1.25 : 1.15);
        try_parts(p, id, &us, &plan);
        // tiles of 128 rows, where the new tokens fill at least half of them and that is well ahead
        if (!forced && p.max_kv_len >= (p.head_dim == 64 ? 3000 : 2000)) {
            const int ring = small_ring_instance(p);
            if (ring >= 0 && 2 * key_tiles(t[ring], p).busy <= busy) {
                us = std::min(us, whole / (p.head_dim == 64 ? 1.3 : 1.2));
                try_parts(p, ring, &us, &plan);
            }
        }
        return plan;
    }
    // ring kernels: the small workgroup in parts; level or behind below 2048 keys.  10 % ahead of the instance that it replaces or
    // not at all, 50 % where nearly every compute unit has a tile already and parts only pair them up.
    const int ring = forced ? (small_ring ? id : -1) : small_ring_instance(p);
    if (ring >= 0 && p.max_kv_len >= 2048) {
        double us = whole / (8 * key_tiles(t[ring], p).busy > 7 * cus ? 1.5 : 1.1);
        try_parts(p, ring, &us, &plan);
    }
    return plan;
}

// Part length of the fixed splits (0: whole contexts): enough workgroups to fill the chip several times over, parts no
// shorter than 256 keys.
struct FixedParts {
    int length = 256;
    bool wide = false;        // a long context in few units: longer parts and eight waves per workgroup rather than more than 32 parts
    bool lengthened = false;  // by the bounds of the whole batch
};
FixedParts fixed_part_length(const KParams &p, size_t record_bytes)
{
    const int64_t kv = p.max_kv_len, want = (int64_t)p.num_seqs * p.num_kv_heads * kv / 2048;
    FixedParts f;
    int &sl = f.length;
    auto parts = [&]() { return (kv + sl - 1) / sl; };
    while (sl * 2 <= want && sl < 4096) sl *= 2;
    if (sl >= kv) sl = 0;
    while (sl > 0 && sl < 4096 && parts() > 32) {
        sl *= 2;
        f.wide = true;
    }
    // at most two parts per compute unit in all (the bound `usable` enforces), and records of at most record_bytes
    auto too_many = [&]() {
        return p.num_seqs * parts() > 2 * compute_units() ||
               (uint64_t)(p.num_seqs * parts()) * p.num_q_heads * partial_stride(p.head_dim) * sizeof(float) > record_bytes;
    };
    while (sl > 0 && sl < 4096 && too_many()) {
        sl *= 2;
        f.lengthened = true;
    }
    if (sl >= kv || (sl > 0 && too_many())) sl = 0;
    return f;
}

// Token-balanced decode pays from this many keys of the batch on, whatever the number of heads.
bool very_long_runs(const KParams &p) { return (int64_t)p.num_seqs * p.max_kv_len >= 100000; }

// Whether a decode call without (enough) workspace is served by the unsplit kernel: where the fixed parts alone, without the
// token-balanced kernels' and the short contexts' rules, come to whole contexts, or to a length that the type and head
// size had no split kernel for when callers could first leave the workspace out.  Other calls are refused.
bool served_without_workspace(const KParams &p)
{
    if (p.num_kv_heads >= 4 && very_long_runs(p)) return false;
    const int sl = fixed_part_length(p, SIZE_MAX).length;
    if (p.dtype == kDtypeF16) return p.head_dim == 128 && (sl == 0 || sl == 4096);
    return sl == 0 || (p.head_dim == 64 && sl != 512 && sl != 2048);
}

int heuristic(const KParams &p, int is_decode)
{
    int n;
    const Instance *t = instances(is_decode, &n);
    int id = -1;
    if (!is_decode) {
        if (few_rows_many_keys(p)) id = find_instance(0, p, 8, 0, 32, 32, 0);  // wavefronts split the keys
        if (id >= 0) return id;
        const int hpw = ring_heads(p);
        id = find_instance(0, p, 8, hpw, 32, 128, 0, 1);  // two wavefront groups per 128-row tile
        if (halves_pay(p, id)) return id;
        id = -1;
        // Small (128 rows, two per compute unit, three at D = 64) or large workgroup, and the grid's order: every ring instance timed
        // in graphs on 14000 random causal calls of 400 to 20000 tiles of 128 rows (2 to 800 GFLOP, 1-64 sequences of up to 9000
        // keys, 32/8, 64/8, 16/16, 16/4 and 8/2 heads), and choice before against choice now on 370 of them over 100 ms without a pause
        // (in brackets; a full grid is bound by power, and after a pause the clock starts some 20 % lower).  The large one (one
        // workgroup, 256 rows) moves half of the bytes per flop and wins once its start and end are a small part of its walk and
        // there are many rounds of it.
        //  * D = 128: small up to 4096 keys (against the large one above 2048 keys 1.08x on average, 1.07x behind a prefix [1.02-1.17x,
        //    1.01-1.11x]; but for three to four tiles per compute unit without a prefix, two full rounds of the large one: small there too
        //    is level on average and doubles the shapes that lose more than 2 %, from 3.6 to 6.7 % of 386), and below 8192 where its
        //    tiles make no more than two rounds (four tiles per compute unit behind a prefix: 1.09x [1.02-1.05x]; three else: 1.06x
        //    [1.03-1.1x]).  Beyond, level or behind: one sequence of 8191 tokens 474-485 us large, 496 small; 16 x 512 behind 0-8192
        //    654 and 680.
        //    Behind a prefix 414 shapes above 2048 keys gain 1.060x, 16 % of them lose more than 2 % (0.90x at worst); small_tiles_fit
        //    there would be 1.052x and 7 %, and 167 shapes 0.98x against these lines, down to 0.73x.
        //    Without a causal mask, 2048-8192 keys: what fits (small_tiles_fit).  On 256 shapes 1.09x against the choice before these
        //    lines, 5 % of them more than 2 % behind it (with the lines of the causal calls 19 %, down to 0.86x).
        //  * D = 64: small up to 2048 keys, and up to eight tiles per compute unit (sixteen behind a prefix): 1.05-1.14x [1.03-1.22x].
        //    Beyond, 1.07x but [0.97-1.03x]: 6 x 300-3000 tokens [178 us large, 184 small].  Without a causal mask too (1225 shapes 1.046x
        //    against the choice before, 1.045x with the lines before).
        //  * Order, sequences outermost (their tiles share the keys in one L2) behind a prefix that dominates: 1.02-1.1x; else tiles outermost
        //    (equal costs in flight, small tiles left for the end): D = 128 1.03-1.1x below 32 sequences, and between 2048 and 4096
        //    keys to twelve tiles per compute unit; D = 64, small, also for many sequences up to eight tiles per compute unit (32-64
        //    sequences 1.03-1.17x [1.07-1.24x], beyond 0.96-1.03x) and for five or more sequences above 4096 keys (1.2x; fewer
        //    1.04x, down to 0.74x).
        //  * Without a causal mask all tiles of a sequence cost the same and none is left for the end.  Above 2048 keys sequences outermost:
        //    1.14x at D = 128, 1.10x at D = 64 on 219 shapes of 2-31 sequences, 0.95-1.76x (6 of up to 8823 tokens, 8/2 heads, D = 64, take
        //    444 us tiles outermost, as the lines above would have it, and 320); below, as long as there are fewer than 32, tiles.
        const bool prefix = p.block_table && p.max_kv_len >= 2 * p.max_q_len;
        const int64_t cus = compute_units(), kv = p.max_kv_len, tiles = small_tiles(p);
        bool small_wg, by_seq;
        if (p.head_dim == 64) {
            small_wg = kv <= 2048 || tiles < (prefix ? 16 : 8) * cus;
            by_seq = !small_wg ? kv >= 4096 || p.num_seqs >= 32 : kv <= 2048 ? p.num_seqs >= 32 && tiles >= 8 * cus : kv <= 4096 ? p.num_seqs >= 32 : p.num_seqs < 5;
        } else {
            const bool even = !prefix && tiles > 3 * cus && tiles <= 4 * cus;
            small_wg = kv <= 2048 || (kv <= 4096 && !even) || (kv < 8192 && tiles <= (prefix ? 4 : 3) * cus);
            if (!p.causal && kv > 2048) small_wg = kv < 8192 && small_tiles_fit(p);
            by_seq = kv <= 2048 ? p.num_seqs >= 32 : kv >= 4096 || tiles >= 12 * cus;
        }
        if (!p.causal) by_seq = kv > 2048 || p.num_seqs >= 32;
        const int order = prefix || by_seq ? 1 : 0;
        // a paged context adds the table entry to every transfer's address chain: the deepest prefetch
        // (8 units) measured up to 10 % ahead of 5 on the slower machines there, level elsewhere
        if (!small_wg && p.block_table) id = find_instance(0, p, 8, hpw, 32, 256, 0, order, 8);
        if (id < 0) id = find_instance(0, p, small_wg ? 4 : 8, hpw, 32, small_wg ? 128 : 256, 0, order);  // LDS-ring kernel
        if (id < 0) id = find_instance(0, p, 8, hpw, 32, 256, 0, order);
        if (id < 0) id = find_instance(0, p, 4, hpw, 32, 256, 0, order);
        if (id < 0) id = find_instance(0, p, 4, hpw, 64, 64 * 4, 0);  // register-staged kernel
    } else {
        // Lines from two sweeps of about 1600 random shapes each (batch 1-256, longest context 16-32768 keys, 2-16 KV
        // heads of 1-8 query heads, bf16 and fp16, D = 64 and 128), every instance timed in a graph; against the
        // fastest instance of its shape the choice takes 1.03x on average and 1.14x at the 95th percentile (the
        // rule before, batch x keys alone, 1.08x and 1.36x).  units = workgroups of the kernels that take one KV head
        // each; kv = longest context.
        const int64_t units = (int64_t)p.num_seqs * p.num_kv_heads, kv = p.max_kv_len;
        // Enough keys to give every compute unit a long run: a workgroup owns whole cache blocks (one
        // wavefront per head), the token-balanced kernel (with four KV heads or more; fewer leave its wavefronts
        // idle).  In between, from 500 000 keys over all heads on (64 units: 8000 keys, 512 units: 1000 keys)
        // it is level with the split kernels or up to 1.2x ahead; a few sequences of more than 8192 keys do
        // better with long parts (3 contexts of 24000 keys 1.2x).
        // Here and below a choice that the fixed splits made before does not go to an instance whose records
        // exceed the array of attn_decode_paged_static, which would then refuse the call; attn_decode_paged makes the
        // same choice, because the two entry points give the same bits.  That is only reached with very many query
        // heads; under 128 (8 KV heads, D = 128), token-balanced against split: 50 contexts of 325-1300 keys 44 against
        // 47 us, one such among 50s 18 against 19; 20 of 1000-4000 49 against 57, one such among 50s 20 against 17.
        auto fits_static = [&](int i) { return i >= 0 && instance_workspace_bytes(t[i], p) <= kScratchBytes ? i : -1; };
        if (p.num_kv_heads >= 4 && (very_long_runs(p) || (kv > 512 && kv <= 8192 && units * kv >= 500000))) {
            // two workgroups of four heads per compute unit measured 0.5-2 % ahead of one of eight from
            // eight KV heads on, 1-2 % behind at four
            if (p.num_kv_heads >= 8) id = find_instance(1, p, 4, 16, 32, 0, -1);
            if (id < 0) id = find_instance(1, p, 8, 16, 32, 0, -1);
            if (!very_long_runs(p)) id = fits_static(id);
        }
        // Many short contexts: whole contexts, one wavefront per head, so that a workgroup reads whole cache
        // blocks and has no cross-wave reduction (1.1-1.5x at 1024 units or below 64 keys).
        if (id < 0 && p.num_kv_heads >= 4 && ((units >= 1024 && kv <= 512) || (units >= 512 && kv <= 64)))
            id = find_instance(1, p, 4, 16, 32, 0, 512, 0, 0, true);
        // Short contexts are not split: the merge and its launch cost more than the walk (one context of 200 keys
        // 6.7 -> 5.7 us, 40 of 100-400 17.2 -> 14.3 us).  Where there are units enough to hide one another's
        // latency that holds up to 1024 keys.  Four wavefronts per workgroup up to 128 keys, and up to 512 where
        // there is a unit for every compute unit; eight otherwise (513-1024 keys, 64 to 500 units: four take 1.02-1.3x as
        // long; from 500 units on the two are within 5 %).
        if (id < 0 && kv <= (units >= 128 ? 1024 : p.head_dim == 64 ? 896 : 640))
            id = find_instance(1, p, kv > 128 && (units < compute_units() || kv > 512) ? 8 : 4, 16, 32, 0, 0);
        if (id < 0) {
            // one KV head per workgroup and fixed parts; where fp16 and D = 64 were not split before they also stay
            // within the static record array
            const bool bounded = p.dtype == kDtypeF16 || p.head_dim == 64;
            const FixedParts fixed = fixed_part_length(p, bounded ? kScratchBytes : SIZE_MAX);
            const int sl = fixed.length;
            // many long contexts of few KV heads, too many to split: still better than a serial walk of
            // each (142 contexts of 2000-15000 keys, 8/2 heads, D = 64: 1.8x)
            if (sl == 0 && kv > 2048) {
                id = fits_static(find_instance(1, p, 4, 16, 32, 0, -2));
                if (id < 0) id = fits_static(find_instance(1, p, 8, 16, 32, 0, -1));
            }
            // For fp16 at D = 64 also where the bound leaves parts of 1024 keys or more: one long context among many
            // short ones would be walked in two or three serial parts.  8/2 heads, token-balanced against parts: 175
            // contexts, one of 3338 keys among 50s 11.5 against 25 us, 800-3338 evenly 47 against 43; 120 contexts, one
            // of 9000 14.6 against 46 us, evenly 77 against 79.  (The other types keep the parts, whose error against 64
            // bits is 2-7 % smaller, and so does one KV head, which leaves seven of eight wavefronts idle: 75 against 58.)
            if (fixed.lengthened && sl >= 1024 && p.num_kv_heads > 1 && p.dtype == kDtypeF16 && p.head_dim == 64)
                id = fits_static(find_instance(1, p, 8, 16, 32, 0, -1));
            // eight waves, one chunk each, also where every part has a compute unit to itself: one context of 1900
            // keys 10.9 -> 10.0 us, 3 of 1900 10.6 -> 9.9; two workgroups per unit lose (8 of 1900: 15.8 -> 18.0), and
            // from 4096 keys on the two are within 3 %
            const bool wide = fixed.wide || (sl == 256 && kv < 4096 && units * ((kv + sl - 1) / sl) <= compute_units());
            if (id < 0 && wide) id = find_instance(1, p, 8, 16, 32, 0, sl);
            if (id < 0) id = find_instance(1, p, 4, 16, 32, 0, sl);
            if (id < 0) id = find_instance(1, p, 4, 16, 32, 0, 0);
        }
    }
    if (id >= 0) return id;
    for (int i = 0; i < n; ++i)
        if (usable(t[i], p, is_decode)) return i;
    return -1;
}

// ---- environment key and cache file ------------------------------------------------------------
std::string env_key_impl()
{
    hipDeviceProp_t prop;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) {
        (void)hipGetLastError();
        return std::string("nodevice|cu0|") + build_id();
    }
    int rt = 0, drv = 0;
    (void)hipRuntimeGetVersion(&rt);
    (void)hipDriverGetVersion(&drv);
    std::ostringstream os;
    os << prop.gcnArchName << "|cu" << prop.multiProcessorCount << "|hip" << rt << "|drv" << drv << "|" << build_id();
    return os.str();
}

std::string build_id()
{
    // FNV-1a over the names of all instances, in table order
    uint64_t h = 1469598103934665603ull;
    for (int is_decode = 0; is_decode < 2; ++is_decode) {
        int n;
        const Instance *t = instances(is_decode, &n);
        for (int i = 0; i < n; ++i)
            for (const char *c = t[i].name; *c; ++c) h = (h ^ (unsigned char)*c) * 1099511628211ull;
    }
    char buf[24];
    snprintf(buf, sizeof buf, "k%016llx", (unsigned long long)h);
    return buf;
}

int instance_by_name(int is_decode, const std::string &name)
{
    int n;
    const Instance *t = instances(is_decode, &n);
    for (int i = 0; i < n; ++i)
        if (name == t[i].name) return i;
    return -1;
}

struct CacheLine {
    std::string env, key, inst;
    double us;
};

bool parse_line(const std::string &line, CacheLine *out)
{
    // fields separated by tabs: env, bucket key, instance name, microseconds
    std::vector<std::string> f;
    size_t pos = 0;
    while (true) {
        size_t t = line.find('\t', pos);
        f.push_back(line.substr(pos, t == std::string::npos ? std::string::npos : t - pos));
        if (t == std::string::npos) break;
        pos = t + 1;
    }
    if (f.size() != 4) return false;
    char *end = nullptr;
    double us = strtod(f[3].c_str(), &end);
    if (end == f[3].c_str() || !(us >= 0)) return false;
    *out = CacheLine{f[0], f[1], f[2], us};
    return true;
}

// Reads the lines of a cache file.  A line that does not parse is skipped and counted, never a reason
// to drop the lines after it (they may be other environments' winners).  ATTN_ERR_CACHE_IO for a file
// that is missing or does not start with the magic line.
int read_cache_file(const char *path, std::vector<CacheLine> *lines, int *damaged)
{
    *damaged = 0;
    std::ifstream in(path);
    if (!in) return ATTN_ERR_CACHE_IO;
    std::string line;
    if (!std::getline(in, line) || line != kCacheMagic) return ATTN_ERR_CACHE_IO;
    while (std::getline(in, line)) {
        if (line.empty() || line[0] == '#') continue;
        CacheLine cl;
        if (!parse_line(line, &cl)) {
            ++*damaged;
            continue;
        }
        lines->push_back(cl);
    }
    return ATTN_OK;
}

int load_cache_locked(const char *path)
{
    std::vector<CacheLine> lines;
    int damaged = 0;
    int rc = read_cache_file(path, &lines, &damaged);
    if (rc != ATTN_OK) return rc;
    if (lines.empty() && damaged > 0) return ATTN_ERR_CACHE_IO;  // nothing but damage
    const std::string env = env_key_impl();
    for (const CacheLine &cl : lines) {
        if (cl.env != env) continue;  // measured on another device or library build
        const int is_decode = cl.key.compare(0, 6, "decode") == 0;
        if (!is_decode && cl.key.compare(0, 7, "prefill") != 0) {
            g_named[cl.key] = cl.inst;
            continue;
        }
        const int id = instance_by_name(is_decode, cl.inst);
        if (id < 0) continue;
        g_winner[is_decode][cl.key] = id;
    }
    g_generation.fetch_add(1, std::memory_order_release);
    return ATTN_OK;
}

void maybe_load_env_cache()
{
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_env_cache_tried) return;
    g_env_cache_tried = true;
    const char *path = getenv("ATTN_TUNE_CACHE");
    if (path && *path) (void)load_cache_locked(path);
}

// Everything the choice depends on.  A serving loop calls with the same shape over and over: the
// last answer per thread and call kind is kept, so a hot call pays one comparison of this key
// instead of building the bucket string, taking the lock and walking the instance table.
struct SelectKey {
    int32_t dtype, head_dim, num_q_heads, num_kv_heads, paged, block_size, causal, num_seqs, max_q_len, max_kv_len;
    int64_t kv_stride_block, kv_stride_tok;  // (kernels with 32-bit offsets inside a block refuse large ones)
    bool operator==(const SelectKey &o) const
    {
        return dtype == o.dtype && head_dim == o.head_dim && num_q_heads == o.num_q_heads && num_kv_heads == o.num_kv_heads &&
               paged == o.paged && block_size == o.block_size && causal == o.causal && num_seqs == o.num_seqs &&
               max_q_len == o.max_q_len && max_kv_len == o.max_kv_len && kv_stride_block == o.kv_stride_block &&
               kv_stride_tok == o.kv_stride_tok;
    }
};
// Between which whole numbers of tiles per compute unit a prefill call lies (or on which one): the rules compare with such
// numbers only, 16 the largest, but for small_tiles_fit (a mark of its own).  Calls with the same maxima and other numbers of tokens mostly
// share an answer.
int32_t tile_class(const KParams &p)
{
    const int64_t tiles = small_tiles(p), cus = compute_units(), whole = tiles / cus;
    return (int32_t)std::min<int64_t>(2 * whole + (tiles > whole * cus), 32) + (!p.causal && small_tiles_fit(p) ? 64 : 0);
}
SelectKey select_key(const KParams &p, int dtype)
{
    return SelectKey{dtype, p.head_dim, p.num_q_heads, p.num_kv_heads, p.block_table ? 1 : 0, p.block_size, p.causal,
                     p.num_seqs, p.max_q_len, p.max_kv_len, p.kv_stride_block, p.kv_stride_tok};
}
enum class Origin { built_in, tuned, forced };
struct Selection {
    int id = -1;  // or a negative attn_status
    Origin origin = Origin::built_in;
};
struct SelectMemo {
    uint64_t generation = 0;
    SelectKey key{};
    int32_t total_q = -1, tiles = 0;  // prefill: a call with the number of tokens, and its tile_class
    Selection sel;
};

// ATTN_FORCE_INSTANCE=<exact instance name>: calls of the kind that has an instance of that name use
// it whenever it is valid for the shape (and fall back to the usual choice when it is not), as if
// it were every bucket's winner.  ATTN_LOG=1: one line on stderr whenever a shape is resolved.
// ATTN_DEBUG_VALIDATE=1: hot calls check the device-side integers first.  All are read once.
struct EnvKnobs {
    int forced[2] = {-1, -1};
    bool log = false;
    bool debug_validate = false;
};

const EnvKnobs &env_knobs()
{
    static const EnvKnobs k = [] {
        EnvKnobs e;
        const char *lg = getenv("ATTN_LOG");
        e.log = lg && lg[0] == '1';
        const char *dbg = getenv("ATTN_DEBUG_VALIDATE");
        e.debug_validate = dbg && dbg[0] == '1';
        if (const char *name = getenv("ATTN_FORCE_INSTANCE"))
            for (int d = 0; d < 2; ++d) e.forced[d] = instance_by_name(d, name);
        return e;
    }();
    return k;
}

Selection selection_slow(const KParams &p, int dtype, int is_decode)
{
    int n;
    const Instance *t = instances(is_decode, &n);
    maybe_load_env_cache();
    const EnvKnobs &env = env_knobs();
    const std::string key = bucket_key(p, dtype, is_decode);
    int id = -1;
    Origin origin = Origin::built_in;
    if (env.forced[is_decode] >= 0 && usable(t[env.forced[is_decode]], p, is_decode)) {
        id = env.forced[is_decode];
        origin = Origin::forced;
    }
    if (id < 0) {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_winner[is_decode].find(key);
        if (it != g_winner[is_decode].end() && it->second < n && usable(t[it->second], p, is_decode)) {
            id = it->second;
            origin = Origin::tuned;
        }
    }
    if (id < 0) id = heuristic(p, is_decode);
    if (env.log) {
        const char *why = origin == Origin::forced ? "ATTN_FORCE_INSTANCE" : origin == Origin::tuned ? "tuned" : "heuristic";
        if (id >= 0)
            fprintf(stderr, "[attn] %s %s -> %s (%s)\n", is_decode ? "decode" : "prefill", key.c_str(), t[id].name, why);
        else
            fprintf(stderr, "[attn] %s %s -> no valid instance\n", is_decode ? "decode" : "prefill", key.c_str());
    }
    return Selection{id >= 0 ? id : ATTN_ERR_UNSUPPORTED, origin};
}

Selection selection(const KParams &p, int dtype, int is_decode)
{
    const int forced = g_forced[is_decode].load();
    if (forced >= 0) {
        int n;
        const Instance *t = instances(is_decode, &n);
        return Selection{forced < n && usable(t[forced], p, is_decode) ? forced : ATTN_ERR_UNSUPPORTED, Origin::forced};
    }
    static thread_local SelectMemo memo[2];
    SelectMemo &m = memo[is_decode];
    const SelectKey key = select_key(p, dtype);
    const uint64_t gen = g_generation.load(std::memory_order_acquire);
    const bool known = m.generation == gen && m.key == key;
    if (known && (is_decode || m.total_q == p.total_q)) return m.sel;
    const int32_t tiles = is_decode ? 0 : tile_class(p);  // (its divisions are spared where the number of tokens is the same too)
    if (known && m.tiles == tiles) {
        m.total_q = p.total_q;
        return m.sel;
    }
    const Selection sel = selection_slow(p, dtype, is_decode);
    // the generation is read again: a table change that raced with the slow path must not be memoised
    if (g_generation.load(std::memory_order_acquire) == gen) {
        m.generation = gen;
        m.key = key;
        m.total_q = p.total_q;
        m.tiles = tiles;
        m.sel = sel;
    }
    return sel;
}
int select_instance(const KParams &p, int dtype, int is_decode) { return selection(p, dtype, is_decode).id; }

// What a prefill call with scratch memory runs in place of the selected instance; the last answer per thread is kept like the
// selection's.  Only the built-in choice gives way to another kernel: a tuned winner was measured on this GPU, which the models were
// not, and stands as it is; a forced instance takes parts of its own at most.
KeyPlan planned_parts(const KParams &p, int dtype, Selection sel)
{
    if (sel.origin == Origin::tuned) return KeyPlan{sel.id, 1};
    struct Memo {
        SelectKey key{};
        int total_q = -1;  // (the models' times follow it)
        Selection sel;
        KeyPlan plan;
    };
    static thread_local Memo m;
    const SelectKey key = select_key(p, dtype);
    if (m.sel.id != sel.id || m.sel.origin != sel.origin || m.total_q != p.total_q || !(m.key == key)) {
        m = Memo{key, p.total_q, sel, key_plan(p, sel.id, sel.origin == Origin::forced)};
        if (env_knobs().log && m.plan.parts > 1) {
            int n;
            fprintf(stderr, "[attn] prefill %s with scratch memory -> %s in %d parts\n", bucket_key(p, dtype, 0).c_str(),
                    instances(0, &n)[m.plan.id].name, m.plan.parts);
        }
    }
    return m.plan;
}

// The plan of the prefill call `a` with scratch memory (pointer fields but block_table are ignored).
int prefill_plan(const attn_args *a, KeyPlan *plan)
{
    if (!a) return ATTN_ERR_NULL;
    if (a->struct_bytes != sizeof(attn_args) || a->num_seqs <= 0 || a->total_q <= 0 || a->num_q_heads <= 0 || a->num_kv_heads <= 0 ||
        a->num_q_heads % a->num_kv_heads || a->max_q_len < 0 || a->max_kv_len < 0)
        return ATTN_ERR_SHAPE;
    if (a->head_dim != 64 && a->head_dim != 128) return ATTN_ERR_UNSUPPORTED;
    if (!is16(a->dtype)) return ATTN_ERR_DTYPE;
    const KParams p = to_kparams(a, 0);
    const Selection sel = selection(p, a->dtype, 0);
    if (sel.id < 0) return sel.id;
    *plan = planned_parts(p, a->dtype, sel);
    return ATTN_OK;
}

size_t balanced_workspace_bytes(int num_seqs, int num_q_heads, int head_dim, int wgs)
{
    return (size_t)(wgs + num_seqs) * num_q_heads * partial_stride(head_dim) * sizeof(float) + (size_t)(num_seqs + 1) * sizeof(int32_t);
}

// Workspace bytes instance `inst` needs for the call `p` (0: it writes the output directly).
size_t instance_workspace_bytes(const Instance &inst, const KParams &p_in)
{
    KParams p = p_in;
    apply_split(p, inst);
    if (inst.split_len < 0) return balanced_workspace_bytes(p.num_seqs, p.num_q_heads, p.head_dim, p.num_splits);
    if (p.num_splits <= 1) return 0;
    return (size_t)p.num_seqs * p.num_q_heads * p.num_splits * partial_stride(p.head_dim) * sizeof(float);
}

// The largest need of any instance that may be chosen for this call (cache winner, forced or built-in),
// so the answer does not depend on the state of the winner cache.
size_t decode_workspace_bytes(const KParams &p)
{
    int n;
    const Instance *t = instances(1, &n);
    size_t need = 0;
    for (int i = 0; i < n; ++i)
        if (usable(t[i], p, 1)) need = std::max(need, instance_workspace_bytes(t[i], p));
    return need;
}

// Debug aid, switched on by ATTN_DEBUG_VALIDATE=1 in the environment: the device-side integers that
// the hot call otherwise trusts are copied to the host (the stream is drained first, so the call
// is neither asynchronous nor capturable in this mode) and checked against the host-side bounds.
int debug_validate_device_side(const attn_args *a, int is_decode, hipStream_t stream)
{
    const int B = a->num_seqs;
    if (hipStreamSynchronize(stream) != hipSuccess) return ATTN_ERR_HIP;
    std::vector<int32_t> lens(B), qsl(B + 1, 0), kvsl;
    if (hipMemcpy(lens.data(), a->seq_lens, B * sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess) return ATTN_ERR_HIP;
    if (!is_decode && hipMemcpy(qsl.data(), a->query_start_loc, (B + 1) * sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess)
        return ATTN_ERR_HIP;
    if (is_decode)
        for (int s = 0; s <= B; ++s) qsl[s] = s;
    if (qsl[0] != 0 || qsl[B] != a->total_q) return ATTN_ERR_SHAPE;
    for (int s = 0; s < B; ++s) {
        const int nq = qsl[s + 1] - qsl[s];
        if (nq < 0 || nq > a->max_q_len || lens[s] < 0 || lens[s] > a->max_kv_len) return ATTN_ERR_SHAPE;
        if (a->causal && nq > lens[s]) return ATTN_ERR_SHAPE;  // a query positioned before key 0
    }
    if (a->block_table) {
        std::vector<int32_t> row(a->block_table_stride);
        for (int s = 0; s < B; ++s) {
            const int need = (lens[s] + a->block_size - 1) / a->block_size;
            if (need > a->block_table_stride) return ATTN_ERR_SHAPE;
            if (hipMemcpy(row.data(), a->block_table + (size_t)s * a->block_table_stride, (size_t)need * sizeof(int32_t),
                          hipMemcpyDeviceToHost) != hipSuccess)
                return ATTN_ERR_HIP;
            for (int b = 0; b < need; ++b)
                if (row[b] < 0 || row[b] >= a->num_blocks) return ATTN_ERR_SHAPE;
        }
    } else {
        const int32_t *src = a->kv_start_loc ? a->kv_start_loc : a->query_start_loc;
        kvsl.resize(B + 1);
        if (hipMemcpy(kvsl.data(), src, (B + 1) * sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess) return ATTN_ERR_HIP;
        for (int s = 0; s < B; ++s)
            if (kvsl[s] < 0 || kvsl[s + 1] < kvsl[s] || kvsl[s] + lens[s] > kvsl[s + 1]) return ATTN_ERR_SHAPE;
    }
    return ATTN_OK;
}

// scratch: prefill in parts only
int run(const attn_args *a, int is_decode, hipStream_t stream, int instance_override, void *scratch = nullptr, size_t scratch_bytes = 0)
{
    int rc = validate(a, is_decode);
    if (rc != ATTN_OK) return rc;
    if (a->num_seqs == 0 || a->total_q == 0) return ATTN_OK;
    if (env_knobs().debug_validate) {
        rc = debug_validate_device_side(a, is_decode, stream);
        if (rc != ATTN_OK) {
            (void)hipGetLastError();
            return rc;
        }
    }
    KParams p = to_kparams(a, is_decode);
    if (a->dtype == ATTN_F32) {
        return launch_prefill_f32(p, stream) == hipSuccess ? ATTN_OK : ATTN_ERR_HIP;
    }
    int n;
    const Instance *t = instances(is_decode, &n);
    const Selection sel = instance_override >= 0 ? Selection{instance_override, Origin::forced} : selection(p, a->dtype, is_decode);
    int id = sel.id;
    if (id < 0) return id;
    if (id >= n || !usable(t[id], p, is_decode)) return ATTN_ERR_UNSUPPORTED;
    if (is_decode) {
        size_t need = instance_workspace_bytes(t[id], p);
        if (need > 0 && (!a->workspace || a->workspace_bytes < need)) {
            // (only the built-in choice gives way: neither a tuned nor a forced instance is replaced)
            const int plain = served_without_workspace(p) ? find_instance(1, p, 4, 16, 32, 0, 0) : -1;
            if (plain < 0 || instance_override >= 0 || g_forced[1].load() >= 0 || id != heuristic(p, 1)) return ATTN_ERR_WORKSPACE;
            id = plain;
            need = 0;
        }
        apply_split(p, t[id]);
        if (need > 0 && ((uintptr_t)a->workspace & 7)) return ATTN_ERR_WORKSPACE;  // records are accessed as 8-byte pairs
    } else if (scratch && ((uintptr_t)scratch & 15) == 0) {
        const KeyPlan plan = planned_parts(p, a->dtype, sel);
        if (plan.parts > 1 && scratch_bytes >= key_parts_bytes(t[plan.id], p, plan.parts)) {  // (else: whole key ranges)
            id = plan.id;
            p.num_splits = plan.parts;
            p.workspace = (float *)scratch;
        }
    }
    if (t[id].launch(p, stream) != hipSuccess) return ATTN_ERR_HIP;
    // fixed-split decode merges its parts with a second kernel (the token-balanced launcher brings its own)
    if (is_decode && t[id].split_len >= 0 && p.num_splits > 1 &&
        (p.dtype == kDtypeF16 ? launch_decode_combine_f16(p, stream) : launch_decode_combine(p, stream)) != hipSuccess)
        return ATTN_ERR_HIP;
    return ATTN_OK;
}

// ---- tuner ----------------------------------------------------------------------------------------

// same values as fill_bf16_kernel, stored as fp16
__global__ void fill_f16_kernel(_Float16 *dst, size_t n, uint32_t seed)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        uint32_t h = (uint32_t)i * 2654435761u ^ seed;
        h ^= h >> 15;
        h *= 2246822519u;
        h ^= h >> 13;
        dst[i] = (_Float16)(((int)(h & 0xffff) - 32768) * (1.f / 16384.f));
    }
}

__global__ void fill_bf16_kernel(uint16_t *dst, size_t n, uint32_t seed)
{
    // cheap counter hash -> bf16 in roughly [-2, 2); values only need to be finite and varied
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        uint32_t h = (uint32_t)i * 2654435761u ^ seed;
        h ^= h >> 15;
        h *= 2246822519u;
        h ^= h >> 13;
        const float f = ((int)(h & 0xffff) - 32768) * (1.f / 16384.f);
        dst[i] = (uint16_t)(__float_as_uint(f) >> 16);
    }
}

struct DeviceBuf {
    void *p = nullptr;
    hipError_t alloc(size_t bytes) { return hipMalloc(&p, bytes ? bytes : 16); }
    ~DeviceBuf()
    {
        if (p) (void)hipFree(p);
    }
};

int tune(const attn_args *shape, int is_decode, const char *cache_path, int iters, int flags)
{
    if (!shape) return ATTN_ERR_NULL;
    if (shape->struct_bytes != sizeof(attn_args)) return ATTN_ERR_SHAPE;
    if (!is16(shape->dtype)) return ATTN_ERR_DTYPE;  // the fp32 path has a single kernel
    if (shape->num_seqs <= 0 || shape->num_q_heads <= 0 || shape->num_kv_heads <= 0 ||
        shape->num_q_heads % shape->num_kv_heads || shape->max_kv_len <= 0)
        return ATTN_ERR_SHAPE;
    if (shape->head_dim != 64 && shape->head_dim != 128) return ATTN_ERR_UNSUPPORTED;
    if (iters <= 0) iters = 20;
    const int B = shape->num_seqs, Hq = shape->num_q_heads, Hkv = shape->num_kv_heads, D = shape->head_dim;
    const bool paged = is_decode || shape->block_size > 0;
    const int bs = paged ? (shape->block_size > 0 ? shape->block_size : 16) : 0;
    if (paged && (bs < 16 || (bs & (bs - 1)))) return ATTN_ERR_UNSUPPORTED;
    const int max_q = is_decode ? 1 : std::max(1, shape->max_q_len);
    const int max_kv = std::max(shape->max_kv_len, max_q);

    // lengths: the caller's own batch if it passes seq_lens (and query_start_loc for prefill), else
    // spread evenly between half of the maximum and the maximum
    std::vector<int32_t> qsl(B + 1, 0), kvsl(B + 1, 0), lens(B);
    bool have_lens = false;
    if (shape->seq_lens && (is_decode || shape->query_start_loc)) {
        std::vector<int32_t> hl(B), hq(B + 1, 0);
        have_lens = hipMemcpy(hl.data(), shape->seq_lens, B * sizeof(int32_t), hipMemcpyDeviceToHost) == hipSuccess;
        if (have_lens && !is_decode)
            have_lens = hipMemcpy(hq.data(), shape->query_start_loc, (B + 1) * sizeof(int32_t), hipMemcpyDeviceToHost) == hipSuccess;
        if (!have_lens) (void)hipGetLastError();
        for (int s = 0; s < B && have_lens; ++s) {
            const int nq = is_decode ? 1 : hq[s + 1] - hq[s];
            if (nq < 0 || nq > max_q || hl[s] < nq || hl[s] > max_kv) have_lens = false;  // disagrees with the bounds: ignore
            qsl[s + 1] = qsl[s] + nq;
            kvsl[s + 1] = kvsl[s] + hl[s];
            lens[s] = hl[s];
        }
    }
    for (int s = 0; s < B && !have_lens; ++s) {
        const double f = B > 1 ? 0.5 + 0.5 * (double)((s * 7) % B) / (B - 1) : 1.0;
        int nq = is_decode ? 1 : std::max(1, (int)(max_q * f));
        int nkv = std::max(nq, (int)(max_kv * f));
        if (s == 0) {
            nq = max_q;
            nkv = max_kv;
        }
        qsl[s + 1] = qsl[s] + nq;
        kvsl[s + 1] = kvsl[s] + nkv;
        lens[s] = nkv;
    }
    const int total_q = qsl[B];
    const int64_t total_kv = kvsl[B];
    int width = 0;
    int64_t nblocks = 0;
    std::vector<int32_t> table;
    if (paged) {
        width = (max_kv + bs - 1) / bs;
        for (int s = 0; s < B; ++s) nblocks += (lens[s] + bs - 1) / bs;
        table.assign((size_t)B * width, -1);
        // a random permutation of the pool (Fisher-Yates over a fixed-seed xorshift generator): the
        // block order of a cache that has served for a while.  A regular scatter (a fixed stride) gives
        // the memory channels a regular pattern, and a kernel family can look better on it than it is.
        std::vector<int32_t> perm((size_t)nblocks);
        for (int64_t i = 0; i < nblocks; ++i) perm[(size_t)i] = (int32_t)i;
        uint64_t rng = 0x9e3779b97f4a7c15ull;
        for (int64_t i = nblocks - 1; i > 0; --i) {
            rng ^= rng << 13;
            rng ^= rng >> 7;
            rng ^= rng << 17;
            std::swap(perm[(size_t)i], perm[(size_t)(rng % (uint64_t)(i + 1))]);
        }
        int64_t next = 0;
        for (int s = 0; s < B; ++s)
            for (int b = 0; b < (lens[s] + bs - 1) / bs; ++b) table[(size_t)s * width + b] = perm[(size_t)next++];
    }

    const size_t q_elems = (size_t)total_q * Hq * D;
    const size_t kv_elems = paged ? (size_t)nblocks * bs * Hkv * D : (size_t)total_kv * Hkv * D;
    DeviceBuf dq, dout, dk, dv, dtab, dqsl, dkvsl, dlens, dws;
    if (dq.alloc(q_elems * 2) != hipSuccess || dout.alloc(q_elems * 2) != hipSuccess || dk.alloc(kv_elems * 2) != hipSuccess ||
        dv.alloc(kv_elems * 2) != hipSuccess || dtab.alloc(table.size() * 4) != hipSuccess ||
        dqsl.alloc((B + 1) * 4) != hipSuccess || dkvsl.alloc((B + 1) * 4) != hipSuccess || dlens.alloc(B * 4) != hipSuccess ||
        false) {
        (void)hipGetLastError();
        return ATTN_ERR_HIP;
    }
    if (shape->dtype == ATTN_F16) {
        hipLaunchKernelGGL(fill_f16_kernel, dim3(1024), dim3(256), 0, 0, (_Float16 *)dq.p, q_elems, 1u);
        hipLaunchKernelGGL(fill_f16_kernel, dim3(4096), dim3(256), 0, 0, (_Float16 *)dk.p, kv_elems, 2u);
        hipLaunchKernelGGL(fill_f16_kernel, dim3(4096), dim3(256), 0, 0, (_Float16 *)dv.p, kv_elems, 3u);
    } else {
        hipLaunchKernelGGL(fill_bf16_kernel, dim3(1024), dim3(256), 0, 0, (uint16_t *)dq.p, q_elems, 1u);
        hipLaunchKernelGGL(fill_bf16_kernel, dim3(4096), dim3(256), 0, 0, (uint16_t *)dk.p, kv_elems, 2u);
        hipLaunchKernelGGL(fill_bf16_kernel, dim3(4096), dim3(256), 0, 0, (uint16_t *)dv.p, kv_elems, 3u);
    }
    bool ok = hipMemcpy(dqsl.p, qsl.data(), (B + 1) * 4, hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(dkvsl.p, kvsl.data(), (B + 1) * 4, hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(dlens.p, lens.data(), B * 4, hipMemcpyHostToDevice) == hipSuccess;
    if (paged && ok) ok = hipMemcpy(dtab.p, table.data(), table.size() * 4, hipMemcpyHostToDevice) == hipSuccess;
    if (!ok || hipDeviceSynchronize() != hipSuccess) return ATTN_ERR_HIP;

    attn_args a = *shape;
    a.total_q = total_q;
    a.max_q_len = max_q;
    a.max_kv_len = max_kv;
    a.q = dq.p;
    a.out = dout.p;
    a.k = dk.p;
    a.v = dv.p;
    a.q_stride_tok = a.o_stride_tok = (int64_t)Hq * D;
    a.q_stride_head = a.o_stride_head = D;
    a.kv_stride_head = D;
    a.kv_stride_tok = (int64_t)Hkv * D;
    a.kv_stride_block = paged ? (int64_t)bs * Hkv * D : 0;
    a.block_table = paged ? (const int32_t *)dtab.p : nullptr;
    a.block_table_stride = width;
    a.block_size = bs;
    a.num_blocks = (int32_t)nblocks;
    a.query_start_loc = (const int32_t *)dqsl.p;
    a.kv_start_loc = paged ? nullptr : (const int32_t *)dkvsl.p;
    a.seq_lens = (const int32_t *)dlens.p;
    if (a.scale == 0.f) a.scale = 1.f / std::sqrt((float)D);

    int rc = validate(&a, is_decode);
    if (rc != ATTN_OK) return rc;
    const size_t ws_bytes = is_decode ? decode_workspace_bytes(to_kparams(&a, is_decode)) : 0;
    if (dws.alloc(ws_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return ATTN_ERR_HIP;
    }
    a.workspace = dws.p;
    a.workspace_bytes = ws_bytes;
    const KParams p = to_kparams(&a, is_decode);
    const std::string key = bucket_key(p, a.dtype, is_decode);

    int n;
    const Instance *t = instances(is_decode, &n);
    struct Events {  // destroyed on every way out of this function
        hipEvent_t e0 = nullptr, e1 = nullptr;
        ~Events()
        {
            if (e0) (void)hipEventDestroy(e0);
            if (e1) (void)hipEventDestroy(e1);
        }
    } ev;
    if (hipEventCreate(&ev.e0) != hipSuccess || hipEventCreate(&ev.e1) != hipSuccess) {
        (void)hipGetLastError();
        return ATTN_ERR_HIP;
    }
    const hipEvent_t e0 = ev.e0, e1 = ev.e1;
    // median of `count` timed launches after `warm` untimed ones; < 0 if the instance fails.  A launch
    // slower than `give_up_us` ends the measurement early (the instance cannot win any more).
    auto time_instance = [&](int id, int warm, int count, double give_up_us) -> double {
        for (int w = 0; w < warm; ++w)
            if (run(&a, is_decode, 0, id) != ATTN_OK) return -1.0;
        if (hipDeviceSynchronize() != hipSuccess) {
            (void)hipGetLastError();
            return -1.0;
        }
        std::vector<float> ms;
        for (int i = 0; i < count; ++i) {
            (void)hipEventRecord(e0, 0);
            if (run(&a, is_decode, 0, id) != ATTN_OK) return -1.0;
            (void)hipEventRecord(e1, 0);
            float t = 0.f;
            if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&t, e0, e1) != hipSuccess) {
                (void)hipGetLastError();
                return -1.0;
            }
            ms.push_back(t);
            if (1000.0 * t > give_up_us) break;
        }
        std::sort(ms.begin(), ms.end());
        return 1000.0 * ms[ms.size() / 2];
    };
    struct Cand {
        int id;
        double us;
        bool seed;
    };
    std::vector<Cand> cand;
    for (int id = 0; id < n; ++id)
        if (usable(t[id], p, is_decode)) cand.push_back(Cand{id, 0.0, false});
    if (cand.empty()) return ATTN_ERR_UNSUPPORTED;
    // seeds always survive the first cut: the built-in choice and the winners of the neighbouring buckets
    {
        std::vector<int> seeds;
        const int h = heuristic(p, is_decode);
        if (h >= 0) seeds.push_back(h);
        std::lock_guard<std::mutex> lk(g_mu);
        for (const std::string &nk : neighbour_keys(p, a.dtype, is_decode)) {
            auto it = g_winner[is_decode].find(nk);
            if (it != g_winner[is_decode].end()) seeds.push_back(it->second);
        }
        for (Cand &c : cand)
            for (int sd : seeds) c.seed |= c.id == sd;
    }
    const bool exhaustive = (flags & 2) != 0;
    // Successive halving: a cheap look at every valid instance, a closer one at the best third, the
    // full count only for the last three.  (Exhaustive sweeps are what the paper names as the cost
    // that keeps autotuning out of practice: its requirement list asks for an efficient search.)
    const int plan[2][2] = {{3, 0}, {std::max(5, iters / 2), 0}};
    const int rounds = exhaustive ? 1 : 2;
    int launches = 0;
    for (int r = 0; r < rounds; ++r) {
        const int count = exhaustive ? iters : plan[r][0];
        double best_so_far = 1e30;
        for (Cand &c : cand) {
            c.us = time_instance(c.id, r == 0 ? 2 : 1, count, exhaustive ? 1e30 : 3.0 * best_so_far);
            launches += count + (r == 0 ? 2 : 1);
            if (c.us >= 0 && c.us < best_so_far) best_so_far = c.us;
            if ((flags & 1) && c.us >= 0)
                fprintf(stderr, "[attn_tune] %s :: round %d %-48s %10.2f us\n", key.c_str(), r, t[c.id].name, c.us);
        }
        cand.erase(std::remove_if(cand.begin(), cand.end(), [](const Cand &c) { return c.us < 0; }), cand.end());
        if (cand.empty()) break;
        std::stable_sort(cand.begin(), cand.end(), [](const Cand &x, const Cand &y) { return x.us < y.us; });
        if (r + 1 < rounds) {
            const size_t keep = std::max<size_t>(4, (cand.size() + 2) / 3);
            std::vector<Cand> next;
            for (size_t i = 0; i < cand.size(); ++i)
                if (i < keep || (r == 0 && cand[i].seed)) next.push_back(cand[i]);
            cand.swap(next);
        }
    }
    // The finalists (and the built-in choice, whatever its rank) are measured once more, taking turns
    // launch by launch, so that a drift of the clocks during the measurement hits all of them alike;
    // the median of each decides.  Launch-to-launch noise is a few percent: the built-in choice keeps
    // its place unless a finalist beats it by more than 3 %.
    const int h = heuristic(p, is_decode);
    if (!exhaustive && !cand.empty()) {
        if (cand.size() > 3) cand.resize(3);
        bool has_h = false;
        for (const Cand &c : cand) has_h |= c.id == h;
        if (!has_h && h >= 0 && usable(t[h], p, is_decode)) cand.push_back(Cand{h, 0.0, true});
        std::vector<std::vector<double>> samples(cand.size());
        for (int i = 0; i < iters; ++i)
            for (size_t k = 0; k < cand.size(); ++k) {
                const double us = time_instance(cand[k].id, 0, 1, 1e30);
                ++launches;
                if (us >= 0) samples[k].push_back(us);
            }
        for (size_t k = 0; k < cand.size(); ++k) {
            std::sort(samples[k].begin(), samples[k].end());
            cand[k].us = samples[k].empty() ? -1.0 : samples[k][samples[k].size() / 2];
            if ((flags & 1) && cand[k].us >= 0)
                fprintf(stderr, "[attn_tune] %s :: final   %-48s %10.2f us\n", key.c_str(), t[cand[k].id].name, cand[k].us);
        }
        cand.erase(std::remove_if(cand.begin(), cand.end(), [](const Cand &c) { return c.us < 0; }), cand.end());
        std::stable_sort(cand.begin(), cand.end(), [](const Cand &x, const Cand &y) { return x.us < y.us; });
    }
    int best = cand.empty() ? -1 : cand[0].id;
    double best_us = cand.empty() ? 0.0 : cand[0].us;
    for (const Cand &c : cand)
        if (c.id == h && c.id != best && best_us > 0.97 * c.us) {
            best = c.id;
            best_us = c.us;
        }
    if (flags & 1) fprintf(stderr, "[attn_tune] %s :: %d launches in all\n", key.c_str(), launches);
    if (best < 0) return ATTN_ERR_UNSUPPORTED;
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_winner[is_decode][key] = best;
        g_generation.fetch_add(1, std::memory_order_release);
    }
    if (flags & 1) fprintf(stderr, "[attn_tune] winner %s -> %s (%.2f us)\n", key.c_str(), t[best].name, best_us);
    if (!cache_path) return ATTN_OK;

    return merge_cache_line(cache_path, key, t[best].name, best_us);
}

}  // namespace

std::string environment_key() { return env_key_impl(); }

int merge_cache_line(const char *path, const std::string &key, const std::string &instance_name, double us)
{
    // Read, change and replace under an exclusive lock on a side file, so that two processes tuning into
    // one cache file do not lose each other's lines (the data file itself is replaced by rename and
    // cannot carry the lock).
    struct Lock {
        int fd = -1;
        explicit Lock(const std::string &p)
        {
            fd = open(p.c_str(), O_CREAT | O_RDWR | O_CLOEXEC, 0644);
            if (fd >= 0 && flock(fd, LOCK_EX) != 0) {
                close(fd);
                fd = -1;
            }
        }
        ~Lock()
        {
            if (fd >= 0) {
                (void)flock(fd, LOCK_UN);
                close(fd);
            }
        }
    } lock(std::string(path) + ".lock");
    if (lock.fd < 0) return ATTN_ERR_CACHE_IO;

    // keep every other line, replace this (environment, bucket) pair; damaged lines are dropped, a
    // missing file or one without the magic line starts afresh
    std::vector<CacheLine> lines;
    int damaged = 0;
    (void)read_cache_file(path, &lines, &damaged);
    const std::string env = env_key_impl();
    std::ostringstream text;
    text << kCacheMagic << "\n";
    for (const CacheLine &cl : lines)
        if (!(cl.env == env && cl.key == key)) text << cl.env << "\t" << cl.key << "\t" << cl.inst << "\t" << cl.us << "\n";
    text << env << "\t" << key << "\t" << instance_name << "\t" << us << "\n";
    const std::string body = text.str();

    const std::string tmp = std::string(path) + ".tmp." + std::to_string((long)getpid());
    const int fd = open(tmp.c_str(), O_CREAT | O_TRUNC | O_WRONLY | O_CLOEXEC, 0644);
    if (fd < 0) return ATTN_ERR_CACHE_IO;
    bool ok = true;
    for (size_t done = 0; ok && done < body.size();) {
        const ssize_t w = write(fd, body.data() + done, body.size() - done);
        if (w <= 0)
            ok = false;
        else
            done += (size_t)w;
    }
    ok = ok && fsync(fd) == 0;  // the new contents are on disk before the name points at them
    ok = (close(fd) == 0) && ok;
    if (!ok || rename(tmp.c_str(), path) != 0) {
        (void)remove(tmp.c_str());
        return ATTN_ERR_CACHE_IO;
    }
    return ATTN_OK;
}

void store_named_winner(const std::string &key, const std::string &instance_name)
{
    std::lock_guard<std::mutex> lk(g_mu);
    g_named[key] = instance_name;
}

bool lookup_named_winner(const std::string &key, std::string *instance_name)
{
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_named.find(key);
    if (it == g_named.end()) return false;
    *instance_name = it->second;
    return true;
}

void load_env_cache_once() { maybe_load_env_cache(); }

namespace {
const Instance *all_decode_instances(int *count)
{
    static const std::vector<Instance> all = [] {
        std::vector<Instance> v;
        int n;
        const Instance *t = decode_instances(&n);
        v.insert(v.end(), t, t + n);
        t = decode_f16_instances(&n);
        v.insert(v.end(), t, t + n);
        return v;
    }();
    *count = (int)all.size();
    return all.data();
}
}  // namespace

const Instance *prefill_instances(int *count)
{
    static const std::vector<Instance> all = [] {
        std::vector<Instance> v;
        int n;
        const Instance *t = prefill_ring_instances(&n);
        v.insert(v.end(), t, t + n);
        t = prefill_staged_instances(&n);
        v.insert(v.end(), t, t + n);
        t = prefill_ring_f16_instances(&n);
        v.insert(v.end(), t, t + n);
        t = prefill_staged_f16_instances(&n);
        v.insert(v.end(), t, t + n);
        t = prefill_split_instances(&n);
        v.insert(v.end(), t, t + n);
        return v;
    }();
    *count = (int)all.size();
    return all.data();
}

}  // namespace attn

using namespace attn;

// ---- the entry point that allocates nothing ------------------------------------------------------
// Split-K records of attn_decode_paged_static live in this array instead of a caller workspace.  Every
// GPU the library runs on holds its own copy, at its own address, until the process ends.  In host
// code the name `scratch` is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, resolved once per device (with that device
// current); nullptr if the runtime refuses.
void *scratch_on_current_device()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

extern "C" {

int attn_decode_paged_static(const attn_args *args, void *hip_stream)
{
    int rc = validate(args, 1);
    if (rc != ATTN_OK) return rc;
    if (args->num_seqs == 0 || args->total_q == 0) return ATTN_OK;
    // the need of the instance this call will take, against the fixed size of the array
    const KParams p = to_kparams(args, 1);
    int n;
    const Instance *t = instances(1, &n);
    const int id = select_instance(p, args->dtype, 1);
    if (id < 0) return id;
    if (id >= n || !usable(t[id], p, 1)) return ATTN_ERR_UNSUPPORTED;
    if (instance_workspace_bytes(t[id], p) > kScratchBytes) return ATTN_ERR_WORKSPACE;
    void *ptr = scratch_on_current_device();
    if (!ptr) return ATTN_ERR_HIP;
    attn_args a = *args;
    a.workspace = ptr;
    a.workspace_bytes = kScratchBytes;
    return run(&a, 1, (hipStream_t)hip_stream, id);
}

size_t attn_static_scratch_bytes(void) { return kScratchBytes; }

int attn_prefill_varlen(const attn_args *args, void *hip_stream) { return run(args, 0, (hipStream_t)hip_stream, -1); }

int attn_prefill_varlen_parts(const attn_args *args, void *scratch, size_t scratch_bytes, void *hip_stream)
{
    return run(args, 0, (hipStream_t)hip_stream, -1, scratch, scratch_bytes);
}

int attn_decode_paged(const attn_args *args, void *hip_stream) { return run(args, 1, (hipStream_t)hip_stream, -1); }

size_t attn_workspace_bytes(const attn_args *a, int is_decode)
{
    if (!a || a->struct_bytes != sizeof(attn_args) || !is_decode) return 0;
    if (a->num_seqs <= 0 || a->num_q_heads <= 0 || a->num_kv_heads <= 0 || a->num_q_heads % a->num_kv_heads || a->max_kv_len < 0 ||
        (a->head_dim != 64 && a->head_dim != 128) || !is16(a->dtype))
        return 0;
    KParams p = to_kparams(a, 1);
    // pointer fields are ignored: decode is always paged, whatever block_table holds at this point
    static const int32_t dummy_table = 0;
    p.block_table = &dummy_table;
    if (p.block_size <= 0) {
        p.block_size = a->block_size > 0 ? a->block_size : 16;
        p.block_shift = ilog2_ceil(p.block_size);
    }
    return decode_workspace_bytes(p);
}

size_t attn_prefill_scratch_bytes(const attn_args *a)
{
    KeyPlan plan;
    if (prefill_plan(a, &plan) != ATTN_OK) return 0;
    int n;
    return key_parts_bytes(instances(0, &n)[plan.id], to_kparams(a, 0), plan.parts);
}

int attn_prefill_parts_instance(const attn_args *a, int32_t *parts)
{
    KeyPlan plan;
    const int rc = prefill_plan(a, &plan);
    if (rc != ATTN_OK) return rc;
    if (parts) *parts = plan.parts;
    return plan.id;
}

int attn_tune(const attn_args *shape_like, int is_decode, const char *cache_path, int iters, int flags)
{
    return tune(shape_like, is_decode ? 1 : 0, cache_path, iters, flags);
}

int attn_environment_key(char *buf, size_t buf_bytes)
{
    const std::string k = env_key_impl();
    if (buf && buf_bytes) snprintf(buf, buf_bytes, "%s", k.c_str());
    return (int)k.size();
}

int attn_load_cache(const char *cache_path)
{
    if (!cache_path) return ATTN_ERR_NULL;
    std::lock_guard<std::mutex> lk(g_mu);
    return load_cache_locked(cache_path);
}

void attn_clear_cache(void)
{
    std::lock_guard<std::mutex> lk(g_mu);
    g_winner[0].clear();
    g_winner[1].clear();
    g_named.clear();
    g_generation.fetch_add(1, std::memory_order_release);
}

int attn_num_instances(int is_decode)
{
    int n;
    (void)instances(is_decode ? 1 : 0, &n);
    return n;
}

int attn_instance_name(int is_decode, int id, char *buf, size_t buf_bytes)
{
    int n;
    const Instance *t = instances(is_decode ? 1 : 0, &n);
    if (id < 0 || id >= n) return ATTN_ERR_SHAPE;
    if (!buf || buf_bytes == 0) return ATTN_ERR_NULL;
    snprintf(buf, buf_bytes, "%s", t[id].name);
    return (int)strlen(buf);
}

int attn_selected_instance(const attn_args *a, int is_decode)
{
    is_decode = is_decode ? 1 : 0;
    if (!a || a->struct_bytes != sizeof(attn_args)) return ATTN_ERR_NULL;
    if (!is16(a->dtype)) return ATTN_ERR_DTYPE;
    if (a->num_q_heads <= 0 || a->num_kv_heads <= 0 || a->num_q_heads % a->num_kv_heads) return ATTN_ERR_SHAPE;
    const KParams p = to_kparams(a, is_decode);
    return select_instance(p, a->dtype, is_decode);
}

void attn_force_instance(int is_decode, int id) { g_forced[is_decode ? 1 : 0].store(id); }

const char *attn_status_string(int status)
{
    switch (status) {
        case ATTN_OK: return "ok";
        case ATTN_ERR_NULL: return "a required pointer is NULL";
        case ATTN_ERR_SHAPE: return "inconsistent sizes, strides or head counts";
        case ATTN_ERR_DTYPE: return "dtype not supported by this entry point";
        case ATTN_ERR_UNSUPPORTED: return "no kernel instance for this head_dim / block_size / group size";
        case ATTN_ERR_WORKSPACE: return "workspace missing or too small";
        case ATTN_ERR_HIP: return "HIP runtime error";
        case ATTN_ERR_CACHE_IO: return "tuning cache file could not be read or written";
        default: return "unknown status";
    }
}

}  // extern "C"
