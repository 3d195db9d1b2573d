// Causal variable-length prefill on bf16 (or fp16) MFMA (gfx950): LDS-ring, software-pipelined variant.
//
// Same operation and same operand layout as prefill_bf16.hip (tiled online-softmax
// attention, the FlashAttention-2 formulation of the paper's kernel, section
// "Method and Investigated Kernels"; causal, variable-length, grouped-query heads),
// restructured so that the matrix cores and the vector ALU work at the same time:
//
//  * K and V travel HBM -> LDS with global_load_lds (no registers, no ds_write) into a
//    ring of NSLOT slots of 32 keys; PF units are in flight, counted with s_waitcnt
//    vmcnt, one workgroup barrier per 32-key unit.  The 16-byte chunks of a row are
//    XOR-swizzled (by choosing which global chunk each lane fetches) so that both the
//    128-bit K reads and the transposing 64-bit V reads are free of bank conflicts
//    without padding.
//  * The unit loop is software pipelined: while the MFMAs of S(u+1) = K(u+1) Q^T run,
//    the ALU exponentiates S(u); while the MFMAs of O += V(u) P(u) run, it takes the
//    row maxima of S(u+1) and applies the masks.
//  * At D = 128 the running maximum is only moved when it would grow by more than 2^kSlack
//    (then O and l are rescaled); otherwise exponentials are taken against the stale
//    reference.  Numerator and denominator carry the same reference, so only the rounding
//    of the weights differs, and the rescale of the accumulators becomes rare.
//  * The output tile is transposed through LDS and written as whole rows, and the queries arrive the same way.
//  * Start of a workgroup: everything that can be asked for is asked for before anything is waited for (table entries, whole
//    query rows, the first units), the first scores wait for the queries and unit 0 alone, and no unit past the last one is
//    requested to fill the ring (only the loop unrolled once round it still asks in every iteration, and may repeat the last unit up
//    to PF - 1 times at its end).  With the queries loaded in operand order, the sign of the scale applied to them as they came, all
//    units of the ring awaited and the last unit repeated to fill it (GPU time, before -> now, the four together): 8 x 30 tokens, paged,
//    32/8 heads 6.6 -> 6.0 us, 4 x 40-100 behind 10-100 keys 9.2 -> 8.5, 16 x 100-500 40.3 -> 36.7, 24 x 100-1200 of 16/4
//    heads 95.8 -> 89.8, 8 x 256-2048 128.8 -> 124.0, D = 64 4 x 40-100 5.8 -> 5.6.
//  * Where a call has fewer tiles than the chip has room for, and brings scratch memory, the keys are cut into parts (PARTS;
//    grid dimension y): a part's workgroup runs the same loop over its own keys and leaves its accumulators as a record
//    for prefill_ring_merge_kernel.  3 x 17-70 tokens behind 5000-9000 keys (56 tiles, 512 places): 141 us in one part, 42 in
//    eight, against 51-57 for the key-split kernel; 3 x 390-450 of 16/16 heads behind 3900 99 -> 79 us.  Built for the small
//    workgroups only; key_plan in attn_api.hip has the rule.
//  * Where a call has about as many 128-row tiles as there are compute units, two groups of four wavefronts ("halves", KG = 2) share
//    a tile: each walks half of its keys through a ring of its own, which is the work of two small workgroups on a compute
//    unit, and their states meet in LDS at the end (each group finishes half of the channels).  The longest tile's serial walk bounds such
//    calls, and one small workgroup alone takes 0.57 us for 32 keys where two take 1.0 us together.  One prompt of 1500 tokens of
//    32/8 heads 37.9 -> 33.2 us, 2000 of 16/16 44.5 -> 36.9, 4000 of 16/4 99.8 -> 81.8, 2 x 300-450 behind 500-1500
//    30.8 -> 26.0, 1 x 900 behind 4000 113 -> 82; the meeting costs about 1 us.  halves_pay in attn_api.hip has the rule.
//
// Head sizes 128 and 64.  At D = 64 a unit has half the MFMAs for the same softmax, so the vector ALU is the bound
// (16 MFMAs of two row blocks: 512 cycles of matrix pipe, about 780 of the vector issue port, and 128 more for each
// block whose reference moves, which on a flat softmax is nearly every unit of the first thousand keys); a wave takes two
// 32-row blocks (QB = 2) where there is work enough, which halves its LDS reads and transfers per flop with the same
// registers as one block at D = 128, and four waves (a 1 KB transfer moves eight 128-byte rows, so that is
// how many share a unit).  Against the register-staged kernel that served D = 64 before (32/8 heads, calls in turn):
// 6 fp16 sequences of 300-3000 tokens 473 -> 190 us (289 -> 718 TFLOP/s; 171 us with a reference that may lag by 2^8, see
// kSlack), one bf16 sequence of 8191 tokens 318 us (864 TFLOP/s).  An eight-slot ring with five units in flight is 2-6 % ahead of four slots there; one row block with
// four slots and three workgroups per compute unit leads up to 2048 keys and up to about eight of its tiles per compute unit.
#include "kernel_params.hpp"
#include "prefill_parts.hpp"

namespace attn {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The two 16-bit element types the kernel is instantiated for: how a 32x32x16 product and the packing
// of two weights are spelled.  Everything else (transfers, swizzles,
// transposing reads, masks, the fp32 softmax) is the same code.
struct ElemBf16 {
    typedef __bf16 elem;
    typedef bf16x8 x8;
    typedef bf16x2 x2;
    static constexpr int kDtype = kDtypeBf16;
    static __device__ __forceinline__ f32x16 mfma(x8 a, x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
};
struct ElemF16 {
    typedef _Float16 elem;
    typedef f16x8 x8;
    typedef f16x2 x2;
    static constexpr int kDtype = kDtypeF16;
    static __device__ __forceinline__ f32x16 mfma(x8 a, x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
};
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void gbl_void;

constexpr int kUnit = 32;          // keys per pipeline unit
// log2 of the largest weight tolerated before the reference moves.  At D = 64 the reference follows the running maximum,
// so that the heaviest weight of a row is exactly 1 and those next to it lie at the top of their binade: with a
// slack of 8 the rounding of the weights cost 3-6 % of error against 64 bits on a flat softmax of 256 to 3000 keys and
// 15-23 % on a peaked one (scale 4 / sqrt(D)).
template <int HD>
constexpr float kSlack = HD == 64 ? 0.f : 8.f;
// Reference of a row that has seen nothing but -inf scores: finite, so that -inf minus it stays -inf, and below
// every later score, so that the first finite one becomes the reference.
constexpr float kLowest = -3.0e38f;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// value of the same register in lane ^ 32
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

// LDS traffic of the unit loop is issued behind the compiler's back, as inline assembly, and waited
// for by count.  Two reasons.  The compiler cannot tell that a transposing read never touches a ring
// slot with a transfer in flight and would drain the whole prefetch queue (s_waitcnt vmcnt(0)) in
// front of the builtin.  And once any of the loop's LDS operations is hidden from it, it waits for
// the ones it still sees with lgkmcnt(0), i.e. for the read it issued a moment ago, several times per
// unit.  LDS operations of a wave complete in order, so "at most N operations outstanding" means
// that everything but the N youngest has returned: every consumer below waits with the number of LDS
// operations issued after the one it needs (lds_wait_upto), counted at compile time along the unrolled code.
__device__ __forceinline__ s16x4 lds_read_tr16_b64_untracked(const unsigned char *p)
{
    s16x4 r;
    const unsigned addr = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(r) : "v"(addr) : "memory");
    return r;
}
__device__ __forceinline__ unsigned lds_addr(const unsigned char *p)
{
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
}
template <int OFFSET>
__device__ __forceinline__ u32x4 lds_read_b128_untracked(unsigned addr)
{
    u32x4 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFFSET) : "memory");
    return r;
}
// V^T image fragment f: the index becomes the instruction's immediate offset
__device__ __forceinline__ u32x4 lds_read_fragment(unsigned img, int f)
{
    switch (f) {
        case 0: return lds_read_b128_untracked<0 * 1024>(img);
        case 1: return lds_read_b128_untracked<1 * 1024>(img);
        case 2: return lds_read_b128_untracked<2 * 1024>(img);
        case 3: return lds_read_b128_untracked<3 * 1024>(img);
        case 4: return lds_read_b128_untracked<4 * 1024>(img);
        case 5: return lds_read_b128_untracked<5 * 1024>(img);
        case 6: return lds_read_b128_untracked<6 * 1024>(img);
        default: return lds_read_b128_untracked<7 * 1024>(img);
    }
}
__device__ __forceinline__ void lds_write_b128_untracked(unsigned addr, s16x8 v)
{
    asm volatile("ds_write_b128 %0, %1" : : "v"(addr), "v"(v) : "memory");
}
// at most n LDS operations of this wave are still outstanding (n is a constant once the loops around
// the call are unrolled, so the switch folds to one instruction); `r` is tied so that its use stays below
template <typename T>
__device__ __forceinline__ void lds_wait_upto(int n, T &r)
{
#define LDS_WAIT_CASE(N) case N: asm volatile("s_waitcnt lgkmcnt(" #N ")" : "+v"(r)::"memory"); break;
    switch (n < 0 ? 0 : n) {
        LDS_WAIT_CASE(0) LDS_WAIT_CASE(1) LDS_WAIT_CASE(2) LDS_WAIT_CASE(3) LDS_WAIT_CASE(4) LDS_WAIT_CASE(5) LDS_WAIT_CASE(6)
        LDS_WAIT_CASE(7) LDS_WAIT_CASE(8) LDS_WAIT_CASE(9) LDS_WAIT_CASE(10) LDS_WAIT_CASE(11) LDS_WAIT_CASE(12) LDS_WAIT_CASE(13)
        LDS_WAIT_CASE(14)
        default: asm volatile("s_waitcnt lgkmcnt(15)" : "+v"(r)::"memory"); break;  // the counter's largest value
    }
#undef LDS_WAIT_CASE
}

// s_waitcnt with only vmcnt constrained (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// 16-byte chunk swizzle of a row inside a unit (XOR).  D = 128, rows of 256 bytes: rows r..r+15 get 16 distinct
// values (128-bit K reads), rows r..r+3 differ in the upper two bits (64-bit transposing V reads).  D = 64, two
// rows in 256 bytes: the eight row pairs of rows r..r+15 get eight distinct values, and the pairs of rows
// r..r+3 differ in the upper bit.
template <int HD>
__device__ __forceinline__ int swz(int row)
{
    if (HD == 64) return (((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1) | ((row >> 3) & 1);
    return ((row & 3) << 2) | ((row >> 2) & 3);
}

template <int HD, int QB, int HPW, int NSLOT, int PF, int WAVES, int KG>
struct RingCfg {
    static constexpr int kWaves = WAVES;
    static constexpr int kRowBytes = HD * 2;
    static constexpr int kVOff = kUnit * kRowBytes;      // V rows behind the K rows of a slot
    static constexpr int kSlotBytes = 2 * kVOff;         // 32 K rows + 32 V rows
    static constexpr int kRowsPerDma = 1024 / kRowBytes;
    static constexpr int kRowsPerWave = kUnit / WAVES;   // rows of a unit that one wave transfers
    static constexpr int kDmaPerWave = kRowsPerWave / kRowsPerDma;  // 1 KB transfers per wave, for K and again for V
    static constexpr int kTSub = kWaves / HPW;
    static constexpr int kWaveTok = 32 * QB;
    static constexpr int kTok = kTSub * kWaveTok;
    static constexpr int kThreads = KG * WAVES * 64;
    static constexpr int kFrags = HD / 16;               // V^T fragments of one unit (1 KB each)
    static constexpr int kImgBytes = kFrags * 1024;      // all of them, in MFMA operand order
    static constexpr int kFragsPerWave = kFrags / WAVES; // fragments each wave transposes per unit
    // two waves per SIMD for the small workgroups (four of one row block at D = 64: 40 KB of LDS, 168 registers)
    static constexpr int kMinWaves = KG > 1 ? 2 : WAVES == 4 && QB == 1 && HD == 64 ? 3 : WAVES == 4 && QB * HD <= 128 ? 2 : 1;
    static constexpr int kGroupBytes = NSLOT * kSlotBytes + 2 * kImgBytes;  // ring and images of the wavefronts that walk the same keys
    static constexpr size_t kLdsBytes = (size_t)KG * kGroupBytes;
    // epilogue of two key groups: accumulators that change wavefronts, (reference, sum) of every row, output staging
    static constexpr int kSwapBytes = 32 * HD * 4 / 2, kPairsAt = KG * WAVES * kSwapBytes, kStageAt = KG > 1 ? kPairsAt + KG * WAVES * 32 * 8 : 0;
    static constexpr int kOutRowBytes = kRowBytes / KG;  // what a wavefront stores of a row
    // Queries reach the registers through LDS too: a wavefront's own share of the V^T images and of the K and V rows of the last
    // kLate slots (kShare bytes each) holds its rows until it has read them.
    static constexpr int kShare = kRowsPerWave * kRowBytes;
    static constexpr int kQRegions = kWaveTok / kRowsPerWave;
    static constexpr int kLate = (kQRegions - 2) / 2;
    static constexpr int kEarly = PF < NSLOT - kLate ? PF : NSLOT - kLate;  // units whose slots are free from the start
    static_assert(kShare == kFragsPerWave * 1024 && kQRegions * kShare == kWaveTok * kRowBytes && kEarly >= 3, "room for the queries");
    static_assert(WAVES == 4 || WAVES == 8, "4 or 8 wavefronts");
    static_assert(kDmaPerWave >= 1 && kFragsPerWave >= 1, "every wave transfers and transposes its share");
    // during iteration u the slots of units u+1 (V, transposed for the next iteration) and u+2 (K) are
    // read and units u+3..u+PF are in flight; unit u+PF reuses the slot of unit u+PF-NSLOT <= u
    static_assert(NSLOT >= PF, "ring too small for the prefetch distance");
    static_assert(PF >= 3, "K of unit u+2 is read one iteration ahead, so three units must be resident");
    static_assert(kWaves % HPW == 0, "waves must split evenly over heads");
    static_assert(KG == 1 || (KG == 2 && QB == 1), "one key group or two");
    static_assert(kLdsBytes >= (size_t)kStageAt + KG * kWaves * kWaveTok * kOutRowBytes, "epilogue staging must fit in the ring");
};

// What a workgroup of the grid stands for: HPW query heads of one KV head x kTok tokens of one sequence (t0 outside
// [0, n_q): nothing).
struct RingTile {
    int kvh, hsub, s, q0, n_q, n_kv, off, t0;
    int kv0;  // packed keys: row of the sequence's first one
};
template <typename C, int HPW>
__device__ __forceinline__ RingTile ring_tile(const KParams &p, int bid)
{
    // All lines of the argument struct at once (touch_args in kernel_params.hpp), with the fields that the block index is taken
    // apart with, or their loads end up inside the divisions' branches.
    asm volatile("" : : "s"(p.seq_lens), "s"(p.kv_stride_tok), "s"(p.group), "s"(p.num_splits), "s"(p.num_kv_heads), "s"(p.num_seqs),
                 "s"(p.max_q_len), "s"(p.tile_order), "s"(p.causal), "s"(p.scale_log2e), "s"(p.workspace), "s"(p.query_start_loc),
                 "s"(p.kv_start_loc), "s"(p.block_table), "s"(p.q), "s"(p.q_stride_tok), "s"(p.q_stride_head), "s"(p.k), "s"(p.v));
    RingTile t;
    // Workgroups go to the eight XCDs round-robin, so with the KV head innermost every XCD (and its
    // own L2) serves one KV head when Hkv is a multiple or a divisor of eight.
    const QuotRem by_kvh = divmod_uniform(bid, p.num_kv_heads);
    const QuotRem by_hsub = divmod_uniform(by_kvh.quot, p.group / HPW);
    t.kvh = by_kvh.rem;
    t.hsub = by_hsub.rem;
    bid = by_hsub.quot;
    const int q_tiles = (p.max_q_len + C::kTok - 1) / C::kTok;  // the grid's tile dimension
    // Workgroups start in block-index order as slots come free, so the order is the schedule: work that
    // costs most (most keys to visit) goes first, and small tiles are left to fill the end.
    int s, r;
    if (p.tile_order == 0) {
        // tile index outermost, counted down from the longest sequence's last tile: the tiles in flight
        // cost about the same in every sequence, and every sequence keeps its cheap first tiles for the end.
        // The sequence index rotates with the tile index: inside an XCD the dispatcher deals workgroups
        // to its four shader engines round-robin by index and waits for the engine whose turn it is,
        // so with a fixed sequence-to-index map (say 8 sequences) a long sequence would load one
        // engine with all of its tiles and the other three would wait for it (measured: 20 % imbalance
        // on 8 sequences of 400-1800 tokens).
        const QuotRem by_seq = divmod_uniform(bid, p.num_seqs);
        r = by_seq.quot;
        s = divmod_uniform(by_seq.rem + r, p.num_seqs).rem;
    } else {
        // sequences outermost (all tiles of a sequence run side by side on the XCD of their KV head and
        // stream its K/V together), heaviest tile first.  For the same reason as above the tiles swap
        // places inside each group of four, differently from one sequence to the next (with a tile
        // count that is a multiple of four every engine would otherwise get the same tile of each
        // group from all sequences, the first engine always the heaviest); the order stays heaviest
        // first to within three places, which matters for the last sequence.
        const QuotRem by_tile = divmod_uniform(bid, q_tiles);
        s = by_tile.quot;
        r = by_tile.rem;
        if (r < (q_tiles & ~3)) r ^= s & 3;
    }

    t.s = s;
    int q0 = load_uniform(p.query_start_loc, s), q1 = load_uniform(p.query_start_loc, s + 1), n_kv = load_uniform(p.seq_lens, s), kv0 = 0;
    if (!p.block_table) kv0 = load_uniform(p.kv_start_loc, s);
    asm volatile("" : "+s"(q0), "+s"(q1), "+s"(n_kv), "+s"(kv0));  // one round trip, ahead of every branch
    t.q0 = q0;
    t.n_q = q1 - q0;
    t.n_kv = n_kv;
    t.kv0 = kv0;
    t.off = t.n_kv - t.n_q;
    const int n_tiles_q = (t.n_q + C::kTok - 1) / C::kTok;
    t.t0 = ((p.tile_order == 0 ? q_tiles : n_tiles_q) - 1 - r) * C::kTok;
    return t;
}

// The parts that the keys of a sequence are cut into (few query rows over many keys): equal ones of the sequence, not of the
// tile, so that the tiles of a sequence read the same keys at about the same time; whole trips round the ring.
struct RingParts {
    int length, count;  // count: parts with keys that the tile sees (at least 1)
};
__device__ __forceinline__ RingParts ring_parts(const KParams &p, const RingTile &t, int tok)
{
    int end = t.n_kv;
    if (p.causal) {
        const int last_tok = t.t0 + tok < t.n_q ? t.t0 + tok : t.n_q;
        end = t.off + last_tok < t.n_kv ? t.off + last_tok : t.n_kv;
    }
    const int length = ((t.n_kv + p.num_splits - 1) / p.num_splits + 255) & ~255;
    return RingParts{length, end > length ? (end + length - 1) / length : 1};
}

template <typename E, int HD, int QB, int HPW, int NSLOT, int PF, int WAVES, int KG, bool PAGED, bool PARTS>
__global__ __launch_bounds__(KG * WAVES * 64, (RingCfg<HD, QB, HPW, NSLOT, PF, WAVES, KG>::kMinWaves)) void prefill_ring_kernel(const KParams p)
{
    using C = RingCfg<HD, QB, HPW, NSLOT, PF, WAVES, KG>;
    using elem = typename E::elem;
    using x8 = typename E::x8;
    using x2 = typename E::x2;
    constexpr int KSTEPS = HD / 16;
    constexpr int DB = HD / 32;
    constexpr int CPR = HD / 8;  // 16-byte chunks of a row
    constexpr int kRowBytes = C::kRowBytes, kSlotBytes = C::kSlotBytes, kVOff = C::kVOff;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_all[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const RingTile T = ring_tile<C, HPW>(p, blockIdx.x);
    if (T.t0 < 0 || T.t0 >= T.n_q) return;
    const int kvh = T.kvh, s = T.s, q0 = T.q0, n_q = T.n_q, off = T.off, t0 = T.t0;
    // the keys of this workgroup's part: all of them, or part blockIdx.y.  From here on keys count from kv_begin.
    int kv_begin = 0, n_kv = T.n_kv;
    if (PARTS) {
        const RingParts parts = ring_parts(p, T, C::kTok);
        if ((int)blockIdx.y >= parts.count) return;
        kv_begin = (int)blockIdx.y * parts.length;
        n_kv = n_kv - kv_begin < parts.length ? n_kv - kv_begin : parts.length;
    }

    // (KG = 2: eight wavefronts, four for each half of the keys)
    const int kgroup = KG > 1 ? __builtin_amdgcn_readfirstlane(tid / (WAVES * 64)) : 0;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) - kgroup * WAVES;
    unsigned char *const lds = lds_all + kgroup * C::kGroupBytes;
    const int lhalf = lane >> 5;
    const int l32 = lane & 31;
    const int l16 = lane & 15;
    const int head = kvh * p.group + T.hsub * HPW + (wave % HPW);
    const int t0w = t0 + (wave / HPW) * C::kWaveTok;

    // scores are exponentiated as 2^(c*s - ref); a negative scale is moved into Q (sign flips are exact)
    const float c = fabsf(p.scale_log2e);
    const bool negate_q = p.scale_log2e < 0.f;

    // ---- key range -------------------------------------------------------------------------------
    int pos0 = off - kv_begin;  // key that query 0 sits at
    int kv_end = n_kv;
    if (p.causal) {
        const int last_tok = t0 + C::kTok < n_q ? t0 + C::kTok : n_q;
        kv_end = pos0 + last_tok < n_kv ? pos0 + last_tok : n_kv;
    }
    int n_units = (kv_end + kUnit - 1) / kUnit;

    elem *obase = (elem *)p.out;
    if (n_units <= 0) {  // no visible key at all (an empty context; also lengths that break seq_lens >= n_q): zeros
        if (kgroup > 0) return;
        for (int i = lane; i < C::kWaveTok * CPR; i += 64) {
            const int t = t0w + i / CPR;
            if (t < n_q)
                *(u32x4 *)(obase + (int64_t)(q0 + t) * p.o_stride_tok + (int64_t)head * p.o_stride_head + 8 * (i % CPR)) =
                    u32x4{0u, 0u, 0u, 0u};
        }
        return;
    }

    // Two key groups: the first takes the first half of the units (the larger one), the second the rest, and both count keys from
    // their first one.  The groups meet at the same barriers; one that runs out of units early goes on with those alone (a unit of
    // hidden keys instead would multiply their values by zero, and infinities among them would become NaN).
    int n_share = n_units;  // units of the group that has most
    if (KG > 1) {
        n_share = (n_units + KG - 1) / KG;
        const int first = kgroup * n_share;
        n_units = n_units - first < n_share ? n_units - first : n_share;
        kv_begin += first * kUnit;
        pos0 -= first * kUnit;
        n_kv -= first * kUnit;
        if (kgroup == 0 && n_kv > n_share * kUnit) n_kv = n_share * kUnit;
    }

    // ---- table entries of the first units, queries: requested before anything else is worked out -----------
    constexpr int RPW = C::kRowsPerWave, NDMA = C::kDmaPerWave;
    const int last_unit0 = (n_kv - 1) & ~(kUnit - 1);  // first key of the last unit that holds a real key
    // The block table is read through the scalar cache (constant address space): a vector load would
    // share the counter of the LDS transfers, and waiting for it would drain the whole transfer queue
    // once per unit.
    typedef const __attribute__((address_space(4))) int32_t *table_ptr;
    const table_ptr bt_row = PAGED ? (table_ptr)(p.block_table + (int64_t)s * p.block_table_stride) : (table_ptr) nullptr;
    // Wave-uniform table entry of the block that holds this wave's rows of `unit` (clamped to the sequence), requested with an
    // untracked scalar load (inline assembly): the value may only be used after an s_waitcnt lgkmcnt(0) that follows
    // the request (scalar loads return out of order).
    auto table_entry_request = [&](int unit) -> int {
        if (!PAGED) return 0;
        int u0 = unit * kUnit < last_unit0 ? unit * kUnit : last_unit0;
        int row = u0 + RPW * wave;
        row = row < n_kv ? row : n_kv - 1;
        const unsigned byte_off = (unsigned)((__builtin_amdgcn_readfirstlane(row) + kv_begin) >> p.block_shift) * 4u;
        int r;
        asm volatile("s_load_dword %0, %1, %2" : "=s"(r) : "s"(bt_row), "s"(byte_off) : "memory");
        return r;
    };
    int entries[PF + 1];
#pragma unroll
    for (int u = 0; u <= PF; ++u) entries[u] = table_entry_request(u);
    // ---- queries: whole rows to LDS, 1 KB a transfer --------------------------------------------------
    // (Loaded in MFMA operand order straight from memory, an instruction touches 32 rows: the address unit takes twice as long, and a
    // row's lines are asked for four times over.)
    constexpr int RPD = C::kRowsPerDma;
    const elem *qbase = (const elem *)p.q + (int64_t)head * p.q_stride_head;
    // where the wave's rows 0..RPW-1 of region r go
    auto q_region = [&](int r) -> unsigned {
        const bool image = r >= C::kQRegions - 2;
        return (unsigned)((image ? NSLOT * kSlotBytes + (r - (C::kQRegions - 2)) * C::kImgBytes : (NSLOT - C::kLate + r / 2) * kSlotBytes + (r & 1) * kVOff) +
                          wave * C::kShare);
    };
#pragma unroll
    for (int i = 0; i < C::kWaveTok / RPD; ++i) {
        const int row = RPD * i + lane / CPR;
        const int t = t0w + row < n_q ? t0w + row : n_q - 1;
        const elem *src = qbase + (int64_t)(q0 + t) * p.q_stride_tok + 8 * ((lane % CPR) ^ swz<HD>(row & 31));
        __builtin_amdgcn_global_load_lds((gbl_void *)src, (lds_void *)(lds + q_region(RPD * i / RPW) + RPD * i % RPW * kRowBytes), 16, 0, 0);
    }

    // first key position of this wave's rows, and the first unit that needs masking for this wave
    const int qpos_lo = p.causal ? pos0 + t0w : 0x7fffff00;
    int first_masked = (qpos_lo + 1) / kUnit;             // units below lie entirely at or before qpos_lo
    first_masked = first_masked < n_kv / kUnit ? first_masked : n_kv / kUnit;  // and entirely inside the sequence
    first_masked = first_masked < n_units ? first_masked : n_units;
    int qrel[QB];  // key index (relative to the lane's first key of a unit) up to which a row sees keys
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int qp = p.causal ? pos0 + t0w + qb * 32 + l32 : 0x7fffff00;
        const int lim = qp < n_kv - 1 ? qp : n_kv - 1;  // last visible key
        qrel[qb] = lim - 4 * lhalf;
    }

    // ---- DMA of one unit: wave w moves its share of the rows of K and of V, 1 KB a transfer -------------
    // The address of a transfer is a wave-uniform 64-bit base (SGPRs: pool block or packed row of the
    // unit, KV head) plus a 32-bit per-lane offset (row inside the block, swizzled 16-byte chunk).
    // The rows of a wave never straddle a 16-key block, so the table entry is wave-uniform.
    const unsigned char *kbase = (const unsigned char *)p.k + (int64_t)kvh * p.kv_stride_head * 2;
    const unsigned char *vbase = (const unsigned char *)p.v + (int64_t)kvh * p.kv_stride_head * 2;
    const int kv0 = T.kv0 + kv_begin;
    const int dma_row = RPW * wave + lane / CPR;  // + RPD*i, row inside the unit
    const uint32_t tok_bytes = (uint32_t)p.kv_stride_tok * 2;
    // Per-lane byte offset of a transfer from the first row of this wave's share of a unit: the lane's
    // row and its swizzled 16-byte chunk.  It is the same in every unit whose rows all exist; in a
    // ragged last unit (and in the repeats of it past the end) the rows past the end re-read the last
    // key (finite, masked), which gives a second set of offsets.  Everything else about a transfer's
    // address is wave-uniform: scalar arithmetic.
    uint32_t dma_off[NDMA], dma_off_last[NDMA];
    const uint32_t block_bytes = (uint32_t)(p.kv_stride_block * 2);  // (ring_valid checks that it fits)
    {
        const int wrow_last = last_unit0 + RPW * wave < n_kv ? last_unit0 + RPW * wave : n_kv - 1;
#pragma unroll
        for (int i = 0; i < NDMA; ++i) {
            const uint32_t chunk = 16 * ((lane % CPR) ^ swz<HD>(dma_row + RPD * i));
            dma_off[i] = (uint32_t)(lane / CPR + RPD * i) * tok_bytes + chunk;
            int row = last_unit0 + dma_row + RPD * i;
            row = row < n_kv ? row : n_kv - 1;
            dma_off_last[i] = (uint32_t)(row - wrow_last) * tok_bytes + chunk;
        }
    }
    auto issue_unit = [&](int unit, int entry) {
        unsigned char *slot = lds + (unit % NSLOT) * kSlotBytes + RPW * wave * kRowBytes;
        const int u0 = unit * kUnit < last_unit0 ? unit * kUnit : last_unit0;  // units past the end repeat the last one
        const bool ragged = u0 + kUnit > n_kv;
        int wrow = u0 + RPW * wave;  // first row of this wave's share
        wrow = wrow < n_kv ? wrow : n_kv - 1;
        // the rows of a wave never straddle a 16-key block: one table entry (PAGED) or one packed run of rows
        const uint64_t base = PAGED ? (uint64_t)(uint32_t)entry * block_bytes + (uint32_t)((wrow + kv_begin) & (p.block_size - 1)) * tok_bytes
                                    : (uint64_t)(kv0 + wrow) * tok_bytes;
        const unsigned char *kb = kbase + base, *vb = vbase + base;
#pragma unroll
        for (int i = 0; i < NDMA; ++i) {
            uint32_t o = ragged ? dma_off_last[i] : dma_off[i];
            // (kept opaque: a loop-invariant offset would be widened and added to the array bases once, and
            // the transfers would then carry 64-bit per-lane addresses instead of scalar base + 32-bit offset)
            asm volatile("" : "+v"(o));
            __builtin_amdgcn_global_load_lds((gbl_void *)(kb + o), (lds_void *)(slot + 1024 * i), 16, 0, 0);
            __builtin_amdgcn_global_load_lds((gbl_void *)(vb + o), (lds_void *)(slot + kVOff + 1024 * i), 16, 0, 0);
        }
    };

    // Publish the ring: this wait, then a bare s_barrier (the fence of __syncthreads would drain vmcnt to zero and with it the
    // whole prefetch queue).  Each wave issues 2*NDMA transfers per unit and memory operations complete in order, so once at
    // most 2*NDMA*n are outstanding, this wave's transfers of every unit but the newest n have landed.  All LDS reads of
    // the slot about to be refilled have returned, because their values fed MFMAs issued earlier.
    // `units`: how many of the units requested so far may still be on their way; towards the end of the keys, where nothing
    // more is requested, fewer than PF-3 (the wait may then be stricter than asked).
    auto wait_units = [&](int units) {
        if (units >= PF - 3)
            wait_vmcnt<2 * NDMA * (PF - 3)>();
        else if (PF > 4 && units >= 1)
            wait_vmcnt<2 * NDMA>();
        else
            wait_vmcnt<0>();
    };
    // V^T fragment images: a wave transposes its share of the V fragments of a unit once
    // (ds_read_b64_tr_b16, the slow path) and stores them in MFMA A-operand order; every wave then
    // fetches all kFrags fragments with plain 128-bit reads.  Two images alternate.
    unsigned char *img_base = lds + NSLOT * kSlotBytes;
    // where inside a slot each of this lane's transposing reads goes (the same in every unit)
    int tr_off[C::kFragsPerWave][2];
#pragma unroll
    for (int i = 0; i < C::kFragsPerWave; ++i) {
        const int f = wave * C::kFragsPerWave + i;  // f = ks2 * DB + db
        const int db = f % DB, ks2 = f / DB;
        const int a = l16 >> 2, h1 = (lane >> 4) & 1, h0 = (lane & 3) >> 1;
#pragma unroll
        for (int rd = 0; rd < 2; ++rd) {
            const int row = 16 * ks2 + 8 * rd + 4 * lhalf + a;
            tr_off[i][rd] = kVOff + row * kRowBytes + 16 * ((4 * db + 2 * h1 + h0) ^ swz<HD>(row)) + 8 * (lane & 1);
        }
    }
    auto transpose_load = [&](int unit, s16x4 (&raw)[C::kFragsPerWave][2]) {
        const unsigned char *vt = lds + (unit % NSLOT) * kSlotBytes;
#pragma unroll
        for (int i = 0; i < C::kFragsPerWave; ++i) {
#pragma unroll
            for (int rd = 0; rd < 2; ++rd) raw[i][rd] = lds_read_tr16_b64_untracked(vt + tr_off[i][rd]);
        }
    };
    // ---- per-lane LDS read offsets ----------------------------------------------------------------
    int koff[KSTEPS];
    {
        const int kx = swz<HD>(l32);
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) koff[ks] = l32 * kRowBytes + 16 * ((2 * ks + lhalf) ^ kx);
    }
    // ---- state ---------------------------------------------------------------------------------------
    f32x16 oacc[QB][DB];
    f32x16 s_cur[QB], s_nxt[QB];
    float m_ref[QB], l_run[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_ref[qb] = -INFINITY;
        l_run[qb] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[qb][db][v] = 0.f;
    }

    // Move the reference of the rows whose new maximum outgrew it by more than the slack; wave-uniform per
    // row block, so that a block's accumulators are only touched when one of its rows needs it.
    auto reference_outgrown = [&](int qb, float bm) -> bool { return __builtin_amdgcn_ballot_w64(bm > m_ref[qb] + kSlack<HD>) != 0; };
    auto rescale_to = [&](int qb, float bm) {
        float m_new = fmaxf(m_ref[qb], bm);
        m_new = fmaxf(m_new, kLowest);
        const float alpha = fast_exp2(m_ref[qb] - m_new);
        m_ref[qb] = m_new;
        l_run[qb] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[qb][db][v] *= alpha;
    };
    // Row maxima of the first score tile (masked if MASK), which set the reference (kLowest for a row of nothing
    // but -inf).  With MASK the tile is left scaled (x = c*s, masked entries -inf); without, it stays raw.
    auto settle = [&](int unit, f32x16 (&sacc)[QB], auto mask_tag) {
        constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            if (MASK) {
                const int rel = qrel[qb] - unit * kUnit;  // entries with 8*(v/4) + (v%4) > rel are hidden
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float x = sacc[qb][v] * c;
                    sacc[qb][v] = (8 * (v >> 2) + (v & 3)) > rel ? -INFINITY : x;
                }
            }
            float mx = fmaxf(fmaxf(sacc[qb][0], sacc[qb][1]), sacc[qb][2]);
#pragma unroll
            for (int v = 3; v < 15; v += 2) mx = fmaxf(fmaxf(mx, sacc[qb][v]), sacc[qb][v + 1]);
            mx = fmaxf(mx, sacc[qb][15]);
            mx = swap32_max(mx);
            rescale_to(qb, MASK ? mx : mx * c);
        }
    };
    // ---- prologue: PF units in flight, S(0) ready ------------------------------------------------
    // Everything that can be asked for is asked for before anything is waited for: the queries and all table entries, then
    // the transfers of the first units, then (when those are there) the fragments of K(0) and K(1) and V(0) to transpose.
    if (PAGED) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int u = 0; u <= PF; ++u) asm volatile("" : "+s"(entries[u]));
    }
    if (KG == 1 || n_units > 0) {  // (uniform over a group)
    // (units past the last are not requested here, nor by iterations whose slots are not compile-time constants; their slots then hold
    // anything, which nothing uses)
#pragma unroll
    for (int u = 0; u < C::kEarly; ++u)
        if (u < n_units) issue_unit(u, entries[u]);
    int entry_cur = entries[PF];
    // the queries and unit 0
    if (n_units >= C::kEarly)
        wait_vmcnt<2 * NDMA * (C::kEarly - 1)>();
    else
        wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    x8 qf[QB][KSTEPS];
    u32x4 kf[KSTEPS];  // K fragments of the next unit, fetched one iteration ahead
    bool cur_masked = first_masked <= 0;
    using Masked = std::integral_constant<bool, true>;
    using Plain = std::integral_constant<bool, false>;
    {
        u32x4 k0[KSTEPS], qraw[QB][KSTEPS];
        s16x4 raw[C::kFragsPerWave][2];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int row = 32 * qb + l32;
            const unsigned at = lds_addr(lds) + q_region(row / RPW) + row % RPW * kRowBytes;
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) qraw[qb][ks] = lds_read_b128_untracked<0>(at + 16 * ((2 * ks + lhalf) ^ swz<HD>(l32)));
        }
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) k0[ks] = lds_read_b128_untracked<0>(lds_addr(lds + koff[ks]));
        transpose_load(0, raw);
        constexpr int kBehindQ = KSTEPS + 2 * C::kFragsPerWave;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) {
                lds_wait_upto(kBehindQ, qraw[qb][ks]);
                if (negate_q) qraw[qb][ks] ^= 0x80008000u;
                qf[qb][ks] = __builtin_bit_cast(x8, qraw[qb][ks]);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = C::kEarly; u < PF; ++u)  // the slots that held queries
            if (u < n_units) issue_unit(u, entries[u]);
        __builtin_amdgcn_sched_barrier(0);
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        const unsigned img = lds_addr(img_base + lane * 16);
        int stored = 0;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            lds_wait_upto(KSTEPS - 1 - ks + 2 * C::kFragsPerWave + stored, k0[ks]);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) s_cur[qb] = E::mfma(__builtin_bit_cast(x8, k0[ks]), qf[qb][ks], ks == 0 ? zero : s_cur[qb]);
            if (ks == KSTEPS - 2) {
#pragma unroll
                for (int i = 0; i < C::kFragsPerWave; ++i) {
                    lds_wait_upto(2 * (C::kFragsPerWave - 1 - i) + stored, raw[i][0]);
                    lds_wait_upto(15, raw[i][1]);  // already there: only ties the register below the wait
                    lds_write_b128_untracked(img + (wave * C::kFragsPerWave + i) * 1024, __builtin_shufflevector(raw[i][0], raw[i][1], 0, 1, 2, 3, 4, 5, 6, 7));
                    ++stored;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (cur_masked)
            settle(0, s_cur, Masked{});
        else
            settle(0, s_cur, Plain{});
        wait_units(n_units < PF ? 0 : PF - 3);  // units 1 and 2
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the image is written
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) kf[ks] = lds_read_b128_untracked<(1 % NSLOT) * kSlotBytes>(lds_addr(lds + koff[ks]));
    }

    // ---- main loop ------------------------------------------------------------------------------------
    // Invariant at the top of iteration u: S(u) settled in `cur`; units u and u+1 resident; units up to
    // u+PF-1 issued.
    // One iteration is written as groups of "one MFMA plus the vector and LDS work that hides under
    // it", fenced by scheduling barriers, because a wavefront issues in order: the matrix pipe only
    // stays busy if independent ALU work sits between consecutive MFMAs in program order.
    //   phase X: S(u+1) += K(u+1) Q^T, one MFMA per group, with the exponentials of one pair of
    //            scores of S(u) and one or two transposing V(u) reads per group;
    //   phase Y: O += V(u) P(u), one MFMA per group, with the row maxima (and masks) of S(u+1), the
    //            K(u+2) fragment reads for the next iteration and the transfers of unit u+PF.
    // Invariant at the top of iteration u: S(u) settled in `cur`; kf = K(u+1); units <= u+2 resident;
    // units <= u+PF-1 issued.  The last unit of a tile has an iteration of its own (LAST).
    // LDS operations of one iteration, in issue order (the same in every iteration, so the position of
    // an operation of the previous iteration is known too):
    //   phase X: V^T image fragments f = 0..KSTEPS-1 (one per step of the phase), after fragment kTrAfter the wave's
    //            transposing reads of V(u+1) (2 per fragment it owns), after fragment kWriteAfter the
    //            wave's image stores of V(u+1);
    //   phase Y: K(u+2) fragments ks = 0..KSTEPS-1, kKPerGroup per group from the first group on.
    // A consumer waits until at most as many operations are outstanding as were issued after the one it
    // needs.  Nothing in the loop waits for "all": the image stores are older than the last image
    // fragments the same wave waits for in phase Y, so they have been performed when the wave reaches
    // the barrier; the K reads stay in flight across the barrier.
    // (at D = 64 a unit has four image fragments and four K fragments: the transposing reads go behind
    // fragment 0, the stores behind fragment 2)
    constexpr int kTrAfter = HD == 64 ? 0 : 1, kWriteAfter = HD == 64 ? 2 : 5;
    constexpr int kKPerGroup = 2;
    // Block-table entry of the unit that the next iteration transfers (entry_cur, set up in the prologue):
    // requested (scalar cache) at the top of an iteration, awaited at its barrier -- the one place where
    // this wave waits for everything it has in flight, because scalar loads share the LDS counter and
    // return out of order.
    // LDS addresses of this lane's K fragment reads inside slot 0, and the same 64 KiB further on: with
    // the slot known at compile time (the plain units' loop below is unrolled over the ring) the slot
    // becomes the read's 16-bit immediate offset instead of an addition per read.
    unsigned kaddr[KSTEPS], kaddr_far[KSTEPS];
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        kaddr[ks] = lds_addr(lds + koff[ks]);
        kaddr_far[ks] = kaddr[ks] + 65536u;
        if (NSLOT * kSlotBytes > 65536) asm volatile("" : "+v"(kaddr_far[ks]));  // a register of its own, not an addition at every use
    }
    // SLOT2 >= 0: the ring slot of unit u+2, known at compile time
    // LAST: nothing follows, so no scores are computed, nothing is fetched for later and nobody is waited for.  Against an ordinary
    // iteration over hidden scores (GPU time): 8 x 30 tokens 6.0 -> 5.6 us, 40 x 2-17 of 16/16 heads 9.4 -> 8.6, 16 x 100-500 36.7 -> 34.0, 8 x
    // 256-2048 124 -> 122.
    // The last unit's scores are left raw where it hides nothing from this wave (like a plain unit's) and scaled where it does; either
    // way the exponent comes from one fused multiply-add, exact in the first case and the plain difference in the second.
    // (64 bytes of instructions more than subtractions, which the shortest calls notice: 9 tokens at D = 64 4.01 -> 4.11 us, 7 behind 120 keys
    // 4.93 -> 4.98, D = 128 level.  The products in a block of their own in front of subtractions: another 0.05 us.)
    const float c_last = first_masked == n_units ? c : 1.f;
    auto iteration = [&](int u, f32x16 (&cur)[QB], f32x16 (&nxt)[QB], auto cur_tag, auto nxt_tag, auto slot_tag, auto last_tag) {
        constexpr bool LAST = decltype(last_tag)::value;
        constexpr bool CUR_MASK = decltype(cur_tag)::value;
        constexpr bool NXT_MASK = decltype(nxt_tag)::value;
        constexpr int SLOT2 = decltype(slot_tag)::value;
        constexpr int G = KSTEPS * QB;  // MFMAs per product
        static_assert(KSTEPS == 2 * DB, "as many MFMAs per row block in O += V P as in S = K Q^T");
        const unsigned img_rd = lds_addr(img_base + (u & 1) * C::kImgBytes + lane * 16);
        const unsigned img_wr = lds_addr(img_base + ((u + 1) & 1) * C::kImgBytes + lane * 16);
        const unsigned char *kt2 = lds + ((u + 2) % NSLOT) * kSlotBytes;

        x8 pf[QB][2];
        u32x4 vfrag[2 * DB];
        s16x4 raw[C::kFragsPerWave][2];
        float sum[QB][2];
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        int seq = 0;        // LDS operations issued so far in this iteration
        int vpos[2 * DB];   // position of image fragment f in this iteration's sequence
        int tr_last = 0;    // position of the last transposing read
        int entry_nxt = 0;
        if (!LAST) entry_nxt = table_entry_request(u + 1 + PF);
        // weights 2p, 2p+1 of row block qb: exponentials, rounding, row sum.  The exponentials are spread over
        // both phases (half under the score MFMAs, half under the first PV MFMAs, which only need the
        // first half), so that neither phase has more vector work than matrix work to hide it under.
        // Two steps, a group apart: the exponentials are issued under one MFMA and their results are
        // rounded and summed under the next, so that nothing waits for the transcendental unit's
        // latency (a wavefront issues in order: a use right behind the exponential stalls it).
        float e_pending[QB][2][2];  // two pairs may be pending (D = 64)
        auto exp_issue = [&](int qb, int pair) {
            const int v = 2 * pair;
            float(&e)[2] = e_pending[qb][pair & 1];
            const bool fma = LAST || !CUR_MASK;
            const float f = LAST ? c_last : c;
            e[0] = fast_exp2(fma ? __builtin_fmaf(cur[qb][v], f, -m_ref[qb]) : cur[qb][v] - m_ref[qb]);
            e[1] = fast_exp2(fma ? __builtin_fmaf(cur[qb][v + 1], f, -m_ref[qb]) : cur[qb][v + 1] - m_ref[qb]);
            asm volatile("" : "+v"(e[0]), "+v"(e[1]));  // issued here, not where they are used
        };
        auto exp_finish = [&](int qb, int pair) {
            const int v = 2 * pair;
            const float e0 = e_pending[qb][pair & 1][0], e1 = e_pending[qb][pair & 1][1];
            x2 pr;
            pr[0] = (elem)e0;
            pr[1] = (elem)e1;
            // Row sums with plain adds, two chains per row block (even and odd pairs).  The dot-product
            // instruction that would sum the rounded pair in one go occupies the matrix pipe for about
            // half an MFMA (measured), so it is not free under the MFMAs; the sum of the unrounded
            // weights differs from the sum of the rounded ones by rounding errors that average out.
            sum[qb][pair & 1] = pair < 2 ? e0 + e1 : sum[qb][pair & 1] + (e0 + e1);  // pairs come in order: 0 and 1 start the chains
            pf[qb][v >> 3][v & 7] = pr[0];
            pf[qb][v >> 3][(v & 7) + 1] = pr[1];
        };
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int ks = g / QB, qb = g % QB;
            // K(u+1) fragment ks was read in phase Y of the previous iteration, whose last KSTEPS LDS operations the
            // K reads are; behind it the KSTEPS - 1 - ks later ones and `seq` operations of this iteration were issued
            if (!LAST) {
                if (qb == 0) lds_wait_upto((KSTEPS - 1 - ks) + seq, kf[ks]);
                nxt[qb] = E::mfma(__builtin_bit_cast(x8, kf[ks]), qf[qb][ks], ks == 0 ? zero : nxt[qb]);
            }
            // weights of keys 0..15 (the B operand of the first four PV MFMAs): issued under the even steps,
            // finished under the odd ones (D = 64, half as many MFMAs for the same weights: one pair per step)
            if (HD == 64) {
                if (ks > 0) exp_finish(qb, ks - 1);
                exp_issue(qb, ks);
            } else if (ks % 2 == 0)
                exp_issue(qb, ks / 2);
            else
                exp_finish(qb, ks / 2);
            if (qb == QB - 1) {
                const int f = ks;
                vfrag[f] = lds_read_fragment(img_rd, f);
                vpos[f] = seq++;
                if (!LAST && f == kTrAfter) {  // this wave's share of V(u+1): transposed here, stored a few groups later
                    transpose_load(u + 1, raw);
                    seq += 2 * C::kFragsPerWave;
                    tr_last = seq - 1;
                }
                if (!LAST && f == kWriteAfter) {  // image (u+1)&1 was last read in iteration u-1, before the barrier
#pragma unroll
                    for (int i = 0; i < C::kFragsPerWave; ++i) {
                        lds_wait_upto(seq - 1 - tr_last, raw[i][0]);
                        lds_wait_upto(15, raw[i][1]);  // already there: only ties the register below the wait
                        const s16x8 both = __builtin_shufflevector(raw[i][0], raw[i][1], 0, 1, 2, 3, 4, 5, 6, 7);
                        lds_write_b128_untracked(img_wr + (wave * C::kFragsPerWave + i) * 1024, both);
                        ++seq;
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }

        float mx[QB], bm[QB];
        bool outgrown[QB];
        int rel[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) rel[qb] = qrel[qb] - (u + 1) * kUnit;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int f = g / QB, qb = g % QB;  // f = ks2 * DB + db
            // weights of keys 16..31, needed from the fifth PV MFMA on: each pair is finished a group after
            // it was issued (the last one just ahead of the MFMA that needs it)
            if (HD == 64) {
                if (f == 0) exp_finish(qb, 3);
                if (f == 1 || f == 2) {
                    exp_finish(qb, 2 + 2 * f);
                    exp_finish(qb, 3 + 2 * f);
                }
            } else if (f >= 1 && f <= DB)
                exp_finish(qb, 3 + f);
            if (qb == 0) lds_wait_upto(seq - 1 - vpos[f], vfrag[f]);
            oacc[qb][f % DB] = E::mfma(__builtin_bit_cast(x8, vfrag[f]), pf[qb][f / DB], oacc[qb][f % DB]);
            if (HD == 64 && f < DB) {
                exp_issue(qb, 4 + 2 * f);
                exp_issue(qb, 5 + 2 * f);
            } else if (f < DB)
                exp_issue(qb, 4 + f);
            // The second half of the phase (the last S MFMAs have drained) has vector slots to spare: the row
            // maxima of S(u+1), eight scores per group, and right behind them the test whether a reference
            // has to move, so that the answer is there when the last MFMA of the iteration has been issued.
            const int sl = HD == 64 ? g - (G - 2 * QB - 1) : g - 4 * QB;
            if (!LAST && sl >= 0 && sl < 2 * QB) {
                const int q2 = sl / 2, v0 = 8 * (sl % 2);
                if (NXT_MASK) {
#pragma unroll
                    for (int v = v0; v < v0 + 8; ++v) {
                        const float x = nxt[q2][v] * c;
                        nxt[q2][v] = (8 * (v >> 2) + (v & 3)) > rel[q2] ? -INFINITY : x;
                    }
                }
                float m3 = fmaxf(fmaxf(nxt[q2][v0], nxt[q2][v0 + 1]), nxt[q2][v0 + 2]);
                m3 = fmaxf(fmaxf(m3, nxt[q2][v0 + 3]), nxt[q2][v0 + 4]);
                m3 = fmaxf(fmaxf(m3, nxt[q2][v0 + 5]), nxt[q2][v0 + 6]);
                mx[q2] = v0 == 0 ? fmaxf(m3, nxt[q2][v0 + 7]) : fmaxf(fmaxf(mx[q2], m3), nxt[q2][v0 + 7]);
            }
            if (!LAST && sl == 2 * QB) {
#pragma unroll
                for (int q2 = 0; q2 < QB; ++q2) {
                    const float m = swap32_max(mx[q2]);
                    bm[q2] = NXT_MASK ? m : m * c;
                    outgrown[q2] = reference_outgrown(q2, bm[q2]);
                }
            }
            // K fragments of unit u+2 (the fragments of u+1 were consumed in phase X), in order, early in
            // the phase: they are a few groups old when the next iteration asks for them
#pragma unroll
            for (int j = 0; j < kKPerGroup; ++j) {
                const int ks = g * kKPerGroup + j;
                if (!LAST && ks < KSTEPS) {
                    if (SLOT2 < 0)
                        kf[ks] = lds_read_b128_untracked<0>(lds_addr(kt2 + koff[ks]));
                    else
                        kf[ks] = lds_read_b128_untracked<(SLOT2 < 0 ? 0 : SLOT2 * kSlotBytes % 65536)>(SLOT2 * kSlotBytes >= 65536 ? kaddr_far[ks]
                                                                                                                                  : kaddr[ks]);
                    ++seq;
                }
            }
            // Refill: unit u+PF replaces unit u+PF-NSLOT <= u.  With compile-time slots always, which keeps the count of transfers the
            // same in every iteration: past the last unit that is the last one again, into a slot that nothing reads any more.
            if (!LAST && g == G - 3 && (SLOT2 >= 0 || u + PF < n_units)) issue_unit(u + PF, entry_cur);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            l_run[qb] += sum[qb][0] + sum[qb][1];
            if (!LAST && outgrown[qb]) rescale_to(qb, bm[qb]);
        }
        if (LAST) return;
        // Publish.  This wave's transfers of every unit up to u+3 have landed (wait_units; the unrolled loop requests one in every iteration);
        // its image stores have been performed (phase Y waited for younger reads); its K reads may still
        // be in flight, they target a slot that no transfer touches before the barrier after next.
        if (PAGED) asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(entry_nxt)::"memory");
        if (SLOT2 >= 0)
            wait_vmcnt<2 * NDMA * (PF - 3)>();
        else
            wait_units(n_units - 4 - u);
        entry_cur = entry_nxt;
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto copy_back = [&]() {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) s_cur[qb] = s_nxt[qb];
    };
    int u = 0;
    using AnySlot = std::integral_constant<int, -1>;
    using More = std::integral_constant<bool, false>;
    using Last = std::integral_constant<bool, true>;
    // plain units whose successors are plain too, one trip round the ring per pass (u is a multiple of
    // NSLOT here, so unit u+2+i sits in slot (2+i) % NSLOT)
    for (; u + NSLOT < first_masked; u += NSLOT) {
        iteration(u, s_cur, s_nxt, Plain{}, Plain{}, std::integral_constant<int, 2 % NSLOT>{}, More{});
        iteration(u + 1, s_nxt, s_cur, Plain{}, Plain{}, std::integral_constant<int, 3 % NSLOT>{}, More{});
        iteration(u + 2, s_cur, s_nxt, Plain{}, Plain{}, std::integral_constant<int, 4 % NSLOT>{}, More{});
        iteration(u + 3, s_nxt, s_cur, Plain{}, Plain{}, std::integral_constant<int, 5 % NSLOT>{}, More{});
        if (NSLOT == 8) {
            iteration(u + 4, s_cur, s_nxt, Plain{}, Plain{}, std::integral_constant<int, 6 % NSLOT>{}, More{});
            iteration(u + 5, s_nxt, s_cur, Plain{}, Plain{}, std::integral_constant<int, 7 % NSLOT>{}, More{});
            iteration(u + 6, s_cur, s_nxt, Plain{}, Plain{}, std::integral_constant<int, 8 % NSLOT>{}, More{});
            iteration(u + 7, s_nxt, s_cur, Plain{}, Plain{}, std::integral_constant<int, 9 % NSLOT>{}, More{});
        }
    }
    static_assert(NSLOT == 4 || NSLOT == 8, "the loop above is written out for rings of four and eight slots");
    // the rest of them, two per trip so that the two score tiles swap roles
    for (; u + 2 < first_masked; u += 2) {
        iteration(u, s_cur, s_nxt, Plain{}, Plain{}, AnySlot{}, More{});
        iteration(u + 1, s_nxt, s_cur, Plain{}, Plain{}, AnySlot{}, More{});
    }
    if (u + 1 < first_masked) {
        iteration(u, s_cur, s_nxt, Plain{}, Plain{}, AnySlot{}, More{});
        copy_back();
        ++u;
    }
    // (All waves meet at the same n_units - 1 barriers whichever way their units go; the last unit's iteration has none.)
    if (first_masked < n_units) {
        if (!cur_masked) {  // the last plain unit: its successor is masked
            iteration(u, s_cur, s_nxt, Plain{}, Masked{}, AnySlot{}, More{});
            copy_back();
            ++u;
        }
        for (; u + 2 < n_units; u += 2) {
            iteration(u, s_cur, s_nxt, Masked{}, Masked{}, AnySlot{}, More{});
            iteration(u + 1, s_nxt, s_cur, Masked{}, Masked{}, AnySlot{}, More{});
        }
        if (u + 1 < n_units) {
            iteration(u, s_cur, s_nxt, Masked{}, Masked{}, AnySlot{}, More{});
            copy_back();
            ++u;
        }
    }
    iteration(u, s_cur, s_nxt, Masked{}, Masked{}, AnySlot{}, Last{});
    // Nobody uses the K fragments that were read ahead for a unit behind the last one.  They have landed (the last iteration waited for
    // younger reads), but the compiler does not know when: their registers are tied to a wait here, behind those waits, so that it cannot hand
    // them to anything else while a read may still land in them.
    if constexpr (KSTEPS == 8)
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(kf[0]), "+v"(kf[1]), "+v"(kf[2]), "+v"(kf[3]), "+v"(kf[4]), "+v"(kf[5]), "+v"(kf[6]), "+v"(kf[7])::"memory");
    else
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(kf[0]), "+v"(kf[1]), "+v"(kf[2]), "+v"(kf[3])::"memory");

    }
    if (KG > 1)  // the other group's barriers
        for (int i = n_units > 0 ? n_units : -1; i < n_share; ++i) __builtin_amdgcn_s_barrier();

    // ---- epilogue: O / l, transposed through LDS, whole rows to HBM ------------------------------
    wait_vmcnt<0>();
    __syncthreads();  // the ring is free: every wave is past its last V read and no DMA is in flight
    // What this wave finishes: all channels, or (two key groups) its group's half of them, with the other group's share added
    constexpr int ODB = DB / KG;
    f32x16 out[QB][ODB];
    float l_row[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) l_row[qb] = swap32_sum(l_run[qb]);
    if constexpr (KG > 1) {
        unsigned char *mine = lds_all + (kgroup * WAVES + wave) * C::kSwapBytes, *theirs = lds_all + ((1 - kgroup) * WAVES + wave) * C::kSwapBytes;
        float2 *pairs = (float2 *)(lds_all + C::kPairsAt);
        auto leave = [&](const f32x16 &a, int i) {
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) *(f32x4 *)(mine + ((4 * i + vq) * 64 + lane) * 16) = f32x4{a[4 * vq], a[4 * vq + 1], a[4 * vq + 2], a[4 * vq + 3]};
        };
        if (kgroup == 0) {
#pragma unroll
            for (int i = 0; i < ODB; ++i) leave(oacc[0][ODB + i], i), out[0][i] = oacc[0][i];
        } else {
#pragma unroll
            for (int i = 0; i < ODB; ++i) leave(oacc[0][i], i), out[0][i] = oacc[0][ODB + i];
        }
        if (lhalf == 0) pairs[(kgroup * WAVES + wave) * 32 + l32] = float2{m_ref[0], l_row[0]};
        __syncthreads();
        const float2 other = pairs[((1 - kgroup) * WAVES + wave) * 32 + l32];
        const float m = fmaxf(m_ref[0], other.x), f = fast_exp2(m_ref[0] - m), g = fast_exp2(other.x - m);
        m_ref[0] = m;
        l_row[0] = l_row[0] * f + other.y * g;
#pragma unroll
        for (int i = 0; i < ODB; ++i)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                const f32x4 o = *(const f32x4 *)(theirs + ((4 * i + vq) * 64 + lane) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) out[0][i][4 * vq + e] = out[0][i][4 * vq + e] * f + o[e] * g;
            }
    } else {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int db = 0; db < DB; ++db) out[qb][db] = oacc[qb][db];
    }
    static_assert(!PARTS || KG == 1, "records are those of one group");
    if (PARTS) {
        const RingParts parts = ring_parts(p, T, C::kTok);
        if (parts.count > 1) {  // one of several: a record of each row block in register order, left for the merge
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                float *rec = p.workspace + (((int64_t)blockIdx.x * WAVES + wave) * QB + qb) * p.num_splits * kRecordFloats<HD> +
                             (int64_t)blockIdx.y * kRecordFloats<HD>;
                if (t0w + qb * 32 + l32 >= n_q) continue;  // (the merge reads no rows past the last token either)
#pragma unroll
                for (int db = 0; db < ODB; ++db)
#pragma unroll
                    for (int vq = 0; vq < 4; ++vq)
                        *(f32x4 *)(rec + (4 * db + vq) * 256 + 4 * lane) =
                            f32x4{out[qb][db][4 * vq], out[qb][db][4 * vq + 1], out[qb][db][4 * vq + 2], out[qb][db][4 * vq + 3]};
                if (lhalf == 0) *(float2 *)(rec + 32 * HD + 2 * l32) = float2{m_ref[qb], l_row[qb]};
            }
            return;
        }
    }
    constexpr int OCPR = CPR / KG;  // 16-byte chunks of a row that a wave stores
    // [token][HD / KG] elements, chunk-swizzled by token
    unsigned char *stage = lds_all + C::kStageAt + (kgroup * WAVES + wave) * (C::kWaveTok * C::kOutRowBytes);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float inv = l_row[qb] > 0.f ? 1.f / l_row[qb] : 0.f;
        const int tl = qb * 32 + l32;
#pragma unroll
        for (int db = 0; db < ODB; ++db) {
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                x2 a, b;
                a[0] = (elem)(out[qb][db][4 * vq + 0] * inv);
                a[1] = (elem)(out[qb][db][4 * vq + 1] * inv);
                b[0] = (elem)(out[qb][db][4 * vq + 2] * inv);
                b[1] = (elem)(out[qb][db][4 * vq + 3] * inv);
                const int chunk = 4 * db + vq;  // 16-byte chunk of the row; lhalf selects its 8-byte half
                u32x2 w;
                w[0] = __builtin_bit_cast(uint32_t, a);
                w[1] = __builtin_bit_cast(uint32_t, b);
                *(u32x2 *)(stage + tl * C::kOutRowBytes + 16 * (chunk ^ (tl % OCPR)) + 8 * lhalf) = w;
            }
        }
    }
    // wave-private staging: the wave's own LDS writes are ordered before its reads
#pragma unroll
    for (int i = 0; i < C::kWaveTok * OCPR / 64; ++i) {
        const int tl = (64 / OCPR) * i + lane / OCPR;
        const int chunk = lane % OCPR;
        const u32x4 row = *(const u32x4 *)(stage + tl * C::kOutRowBytes + 16 * (chunk ^ (tl % OCPR)));
        const int t = t0w + tl;
        if (t < n_q)
            *(u32x4 *)(obase + (int64_t)(q0 + t) * p.o_stride_tok + (int64_t)head * p.o_stride_head + 8 * (kgroup * OCPR + chunk)) = row;
    }
}

// Merges the parts of a tile: a thread owns four channels of a row (the records are in the accumulators' register order, so
// that both sides move whole kilobytes; the 8-byte stores of the outputs are 2 / parts of what is read).
template <typename E, int HD, int QB, int HPW, int NSLOT, int PF, int WAVES, int KG>
__global__ __launch_bounds__(kMergeThreads) void prefill_ring_merge_kernel(const KParams p)
{
    using C = RingCfg<HD, QB, HPW, NSLOT, PF, WAVES, KG>;
    using elem = typename E::elem;
    typedef elem x4 __attribute__((ext_vector_type(4)));
    const int i = (int)blockIdx.x % kMergeBlocks<HD> * kMergeThreads + (int)threadIdx.x;
    const int block = (int)blockIdx.x / kMergeBlocks<HD>;  // 32-row block
    const int qb = block % QB, wave = block / QB % WAVES, tile = block / QB / WAVES;
    const RingTile T = ring_tile<C, HPW>(p, tile);
    const int row = i & 31, ch = 8 * (i >> 6) + 4 * (i >> 5 & 1);
    const int t = T.t0 + (wave / HPW) * C::kWaveTok + 32 * qb + row;
    if (T.t0 < 0 || t >= T.n_q) return;
    const RingParts parts = ring_parts(p, T, C::kTok);
    if (parts.count <= 1) return;
    const float4 o = merge_records<HD>(p.workspace + (int64_t)block * p.num_splits * kRecordFloats<HD>, parts.count, i, row);
    *(x4 *)((elem *)p.out + (int64_t)(T.q0 + t) * p.o_stride_tok + (int64_t)(T.kvh * p.group + T.hsub * HPW + wave % HPW) * p.o_stride_head + ch) =
        x4{(elem)o.x, (elem)o.y, (elem)o.z, (elem)o.w};
}

template <typename E, int HD, int QB, int HPW, int NSLOT, int PF, int WAVES>
bool ring_valid(const KParams &p)
{
    // (a cache block of 4 GiB or more would need 64-bit block arithmetic in the transfers, and so would rows 128 MiB apart)
    return p.dtype == E::kDtype && p.head_dim == HD && p.group % HPW == 0 && (!p.block_table || (uint64_t)p.kv_stride_block * 2 < (1ull << 32)) &&
           (uint64_t)p.kv_stride_tok * 2 * kUnit < (1ull << 32);
}

template <typename E, int HD, int QB, int HPW, int NSLOT, int PF, int WAVES, int KG, bool PAGED, bool PARTS>
hipError_t ring_launch_impl(const KParams &p, hipStream_t stream, int64_t blocks)
{
    using C = RingCfg<HD, QB, HPW, NSLOT, PF, WAVES, KG>;
    auto kern = prefill_ring_kernel<E, HD, QB, HPW, NSLOT, PF, WAVES, KG, PAGED, PARTS>;
    static std::atomic<uint64_t> granted{0};
    const hipError_t allowed = allow_dynamic_lds((const void *)kern, C::kLdsBytes, granted);
    if (allowed != hipSuccess) return allowed;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks, PARTS ? (unsigned)p.num_splits : 1u), dim3(C::kThreads), C::kLdsBytes, stream, p);
    return hipGetLastError();
}

// Instances whose keys can be cut into parts: the small workgroups.
template <int QB, int WAVES, int KG>
constexpr bool kHasParts = QB == 1 && WAVES == 4 && KG == 1;

template <typename E, int HD, int QB, int HPW, int NSLOT, int PF, int WAVES, int KG, int ORDER>
hipError_t ring_launch(const KParams &p_in, hipStream_t stream)
{
    KParams p = p_in;
    p.tile_order = ORDER;
    using C = RingCfg<HD, QB, HPW, NSLOT, PF, WAVES, KG>;
    const int64_t q_tiles = (p.max_q_len + C::kTok - 1) / C::kTok;
    const int64_t nhg = (int64_t)p.num_kv_heads * (p.group / HPW);
    const int64_t blocks = q_tiles * p.num_seqs * nhg;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    if constexpr (kHasParts<QB, WAVES, KG>) {
        if (p.num_splits > 1) {
            if (blocks * WAVES * kMergeBlocks<HD> > 0x7fffffff) return hipErrorInvalidConfiguration;
            const hipError_t e = p.block_table ? ring_launch_impl<E, HD, QB, HPW, NSLOT, PF, WAVES, KG, true, true>(p, stream, blocks)
                                               : ring_launch_impl<E, HD, QB, HPW, NSLOT, PF, WAVES, KG, false, true>(p, stream, blocks);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL((prefill_ring_merge_kernel<E, HD, QB, HPW, NSLOT, PF, WAVES, KG>), dim3((unsigned)(blocks * WAVES * kMergeBlocks<HD>)),
                               dim3(kMergeThreads), 0, stream, p);
            return hipGetLastError();
        }
    }
    return p.block_table ? ring_launch_impl<E, HD, QB, HPW, NSLOT, PF, WAVES, KG, true, false>(p, stream, blocks)
                         : ring_launch_impl<E, HD, QB, HPW, NSLOT, PF, WAVES, KG, false, false>(p, stream, blocks);
}

// This file is compiled twice: as it stands for bf16, and included by prefill_f16_ring.hip with
// ATTN_RING_ELEM_F16 defined for fp16 inputs (a smaller set of instances).
#ifdef ATTN_RING_ELEM_F16
#define RING_ELEM ElemF16
#define RING_NAME "prefill_f16_ring"
#else
#define RING_ELEM ElemBf16
#define RING_NAME "prefill_bf16_ring"
#endif

#define RING_ONE(HD, QB, HPW, NSLOT, PF, WAVES, KG, ALL_WAVES, ORDER, TAG)                                         \
    {                                                                                                              \
        RING_NAME " d" #HD " qb" #QB " w" #ALL_WAVES " hpw" #HPW " slots" #NSLOT " pf" #PF TAG, WAVES * 32 * QB, kUnit, ALL_WAVES, \
            HPW, PF, 0, ring_valid<RING_ELEM, HD, QB, HPW, NSLOT, PF, WAVES>,                                      \
            ring_launch<RING_ELEM, HD, QB, HPW, NSLOT, PF, WAVES, KG, ORDER>, ORDER, false, kHasParts<QB, WAVES, KG> \
    }
// both grid orders of one compiled kernel
#define RING_INSTANCE(HD, QB, HPW, NSLOT, PF, WAVES) \
    RING_ONE(HD, QB, HPW, NSLOT, PF, WAVES, 1, WAVES, 0, ""), RING_ONE(HD, QB, HPW, NSLOT, PF, WAVES, 1, WAVES, 1, " seqmajor")
// the keys of a tile over two groups of four wavefronts, the tiles of a sequence side by side
#define RING_HALVES(HD, HPW) RING_ONE(HD, 1, HPW, 4, 4, 4, 2, 8, 1, " halves seqmajor")

}  // namespace

#ifdef ATTN_RING_ELEM_F16
const Instance *prefill_ring_f16_instances(int *count)
{
    static const Instance table[] = {
        RING_INSTANCE(128, 1, 4, 8, 5, 8), RING_INSTANCE(128, 1, 2, 8, 5, 8), RING_INSTANCE(128, 1, 1, 8, 5, 8),
        RING_INSTANCE(128, 1, 4, 8, 6, 8), RING_INSTANCE(128, 1, 4, 4, 4, 4), RING_INSTANCE(128, 1, 2, 4, 4, 4),
        RING_INSTANCE(128, 1, 1, 4, 4, 4),
        RING_INSTANCE(64, 2, 4, 8, 5, 4), RING_INSTANCE(64, 2, 2, 8, 5, 4), RING_INSTANCE(64, 2, 1, 8, 5, 4),
        RING_INSTANCE(64, 1, 4, 4, 4, 4), RING_INSTANCE(64, 1, 2, 4, 4, 4), RING_INSTANCE(64, 1, 1, 4, 4, 4),
        RING_HALVES(64, 4), RING_HALVES(64, 2), RING_HALVES(64, 1), RING_HALVES(128, 4), RING_HALVES(128, 2), RING_HALVES(128, 1),
    };
    *count = (int)(sizeof(table) / sizeof(table[0]));
    return table;
}
#else
// (The first and the last hpw1 entries are D = 128: a host test takes the last one as another valid instance of a D = 128
// bucket.)
const Instance *prefill_ring_instances(int *count)
{
    static const Instance table[] = {
        RING_INSTANCE(128, 1, 4, 8, 5, 8), RING_INSTANCE(128, 1, 8, 8, 5, 8),
        RING_INSTANCE(128, 1, 2, 8, 5, 8), RING_INSTANCE(128, 1, 1, 8, 5, 8), RING_INSTANCE(128, 1, 4, 8, 6, 8),
        RING_INSTANCE(64, 2, 4, 8, 5, 4), RING_INSTANCE(64, 2, 2, 8, 5, 4), RING_INSTANCE(64, 2, 1, 8, 5, 4),
        RING_INSTANCE(64, 1, 4, 4, 4, 4), RING_INSTANCE(64, 1, 2, 4, 4, 4), RING_INSTANCE(64, 1, 1, 4, 4, 4),
        RING_HALVES(64, 4), RING_HALVES(64, 2), RING_HALVES(64, 1), RING_HALVES(128, 4), RING_HALVES(128, 2), RING_HALVES(128, 1),
        RING_INSTANCE(128, 1, 4, 8, 8, 8), RING_INSTANCE(128, 1, 1, 8, 8, 8), RING_INSTANCE(128, 1, 4, 4, 4, 4),
        RING_INSTANCE(128, 1, 1, 4, 4, 4), RING_INSTANCE(128, 1, 2, 4, 4, 4),
    };
    *count = (int)(sizeof(table) / sizeof(table[0]));
    return table;
}
#endif

}  // namespace attn
