// Device side of libdc_mi355x: chunk decode kernels for gfx950 (CDNA4, wave64).
//
// Paper: Section 3.3 ("Inference Process", "Throughput Analysis"): compressed chunks resident in GPU
// memory are decompressed by the GPU into a decompression buffer; "Speed Adaptive Partial
// Compression": some chunks are raw and only need a copy.  The stored format is in include/dc.h.
//
// Work decomposition: a lane owns one sub-stream, a wavefront owns one stream set (64 sub-streams
// whose 16-byte blocks are stored interleaved in the order the wavefront asks for them), a workgroup
// owns one chunk (S/64 wavefronts; with S = 32 one wavefront owns two chunks, lanes 0-31 / 32-63).
// Per chunk the LDS holds the decode table (2048 x u16: symbol << 8 | length, indexed by the next
// 11 stream bits).  Per wavefront the LDS holds a ring of 16 stream words per lane.  Before every
// half group of 8 symbols the lanes that are short of look-ahead each take the next block of the
// wavefront's region (consecutive lanes, consecutive blocks: one coalesced load, and the region is
// read front to back exactly once); the block goes into the ring two steps later (the look-ahead of
// DC_LOOKAHEAD_BITS bits in the format allows for it), so the per-symbol loop does not wait on memory.  The four
// words that hold a half group come out of the ring together and are only shifted from there on (decode8; where a launch has
// about one wavefront to a SIMD, step_and_decode8_few, which arranges the same work around the chain of look-ups).  A lane
// packs 16 decoded bytes and writes them with one 128-bit store; the lanes of a chunk write S*16 contiguous bytes per round.
//
// The container's second coder (tANS, 2048 states; Section 4.2 of the paper settles on ANS) runs through the
// same kernel with another table and another symbol step: the table holds one 32-bit entry per state
// (build_tans_table), the lane carries the state, and a symbol costs one table read and the state's field
// of stream bits (two_symbols).  Rings, block placement, the words in registers, stores and the fused epilogues are shared.
#include <hip/hip_runtime.h>

#include <atomic>
#include <type_traits>

#include "dc.h"
#include "dc_device.h"

using namespace dcdev;

namespace {

constexpr int kPeekBits = DC_MAX_CODE_LEN;
constexpr int kTableEntries = 1 << kPeekBits;
constexpr int kRingWords = 16;                 // per lane
constexpr uint32_t kBlockBytes = DC_BLOCK_BYTES; // bitstream fetch granule

// kModeGemv adds the partial sums in a fixed order (per wave in registers, per chunk through LDS, per row in
// dc_gemv_ordered_finish_kernel); kModeGemvAtomic is the same product with one atomic per run of lanes, for
// shapes with more rows to a chunk than a wave has lanes.
// kModeGemvRows and kModeGemvW8A8Rows are the products of calls whose chunks hold whole rows: the chunk's workgroup
// scales its rows' sums and writes them, and the call is one launch.
enum Mode { kModeI8 = 0, kModeBf16 = 1, kModeGemv = 2, kModeGemvW8A8 = 3, kModeGemvAtomic = 4, kModeGemvRows = 5, kModeGemvW8A8Rows = 6 };
constexpr uint32_t kPartialSlots = 64; // fp32 partial sums a chunk leaves in the workspace of the ordered product

template <int S> struct Geometry {
    static constexpr int kLanesPerChunk = S < 64 ? S : 64;       // lanes of one wave that serve a chunk
    static constexpr int kChunksPerWave = 64 / kLanesPerChunk;   // 2 when S = 32
    static constexpr int kWaves = S <= 64 ? 1 : S / 64;          // wavefronts of the workgroup
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kThreadsPerChunk = S < 64 ? S : kThreads;
    static constexpr int kSymbolsPerLane = 256 / kThreadsPerChunk; // header values a thread ranks in the table build
};

// One matrix of a fused call: its chunks are table entries [first_chunk, next matrix's first_chunk).
struct MatrixArgs {
    uint64_t first_chunk;
    uint32_t rows, cols;
    const float *row_scale;
    void *dst;              // kModeBf16: bf16 [rows][cols]
    const uint16_t *x_bf16; // kModeGemv
    float *y_accum;         // kModeGemv; kModeGemvW8A8: int32 sums until the finish kernel has run
    uint16_t *y_bf16;       // both products, may be null
    const int8_t *x_i8;     // kModeGemvW8A8
    float x_scale;          // kModeGemvW8A8
};

// What every decode takes.  Alone the arguments of kModeI8 (104 bytes, not the fused modes' 1.4 KB, which every launch copies).
struct BytesArgs {
    const uint8_t *blob;
    uint64_t blob_bytes;
    const dc_chunk *table;
    uint64_t n_chunks;
    uint32_t chunk_bytes;
    uint32_t trailer[4]; // what the blob's last 16 bytes must be for this launch to decode it
    uint64_t *trace;     // traced launches: four words per workgroup (see dc_decompress_chunks_traced), else null
    // kModeI8: all chunks decode into one buffer of dst_cap bytes
    void *dst;
    uint64_t dst_cap;
};
struct DecodeArgs : BytesArgs {
    // kModeGemv: kPartialSlots sums per chunk (slot r: the chunk's share of the r-th row it touches)
    float *partial;
    // fused modes: the matrices, in table order, and the first chunks of the second to the last (beyond them, no chunk's number).  (Behind
    // the matrices they are a cache line of arguments of their own: a layer of seven 100.1 instead of 99.7 us, one matrix alone 0.5 % less.)
    uint32_t n_mats;
    uint32_t next_first[DC_MAX_MATRICES - 1];
    MatrixArgs mats[DC_MAX_MATRICES];
};
template <int MODE> using ArgsOf = std::conditional_t<MODE == kModeI8, BytesArgs, DecodeArgs>;

// Sums `val` (float or int32) over runs of consecutive lanes with equal `key` (keys do not decrease with
// the lane; key 0xFFFFFFFF = lane takes no part) and adds each run's sum to y[key] with one atomic,
// issued by the last lane of the run.
template <bool HALVES, typename T> __device__ __forceinline__ void lanes_add_by_key(T *__restrict__ y, uint32_t key, T val)
{
    static_assert(sizeof(T) == 4, "one register");
#define DC_SEG_STEP(CTRL, MASK)                                                                              \
    {                                                                                                        \
        const uint32_t k2 = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)key, CTRL, MASK, 0xF, false);     \
        const T v2 = __builtin_bit_cast(T, dpp_or_zero<CTRL, MASK>(__builtin_bit_cast(uint32_t, val)));      \
        val += k2 == key ? v2 : T(0);                                                                        \
    }
    DC_SEG_STEP(0x111, 0xF)
    DC_SEG_STEP(0x112, 0xF)
    DC_SEG_STEP(0x114, 0xF)
    DC_SEG_STEP(0x118, 0xF)
    DC_SEG_STEP(0x142, 0xA)
    if (!HALVES) DC_SEG_STEP(0x143, 0xC)
#undef DC_SEG_STEP
    // 0x130: the value of the lane above (lane 63 reads the fill value)
    uint32_t above = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)key, 0x130, 0xF, 0xF, false);
    if (HALVES && (threadIdx.x & 31u) == 31u) above = 0xFFFFFFFFu;
    if (key != 0xFFFFFFFFu && above != key) atomicAdd(y + key, val);
}

// The same sums, kept in the wave: the sum of every run goes to the lane whose number is the run's `slot`
// (slot < 64, the same for all lanes of a run), where it is added to `mine`.  Runs are taken in lane order and
// each lane adds at most one value per call, so the result does not depend on timing.
template <bool HALVES, typename T> __device__ __forceinline__ void lanes_add_runs_to_slots(T &mine, uint32_t key, uint32_t slot, T val)
{
    static_assert(sizeof(T) == 4, "one register");
    auto of_lane = [](T v, uint32_t from) { return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), from)); };
    if (!HALVES) {
        // the usual case with rows of some kilobytes: all 64 lanes hold the same row (or none): one plain sum
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)key);
        if (__all(key == first)) {
            if (first != 0xFFFFFFFFu) {
                const T v = of_lane(lanes_sum(val), 63);
                const uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot) & 63u;
                mine += (threadIdx.x & 63u) == to ? v : T(0);
            }
            return;
        }
    }
#define DC_SEG_STEP(CTRL, MASK)                                                                              \
    {                                                                                                        \
        const uint32_t k2 = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)key, CTRL, MASK, 0xF, false);     \
        const T v2 = __builtin_bit_cast(T, dpp_or_zero<CTRL, MASK>(__builtin_bit_cast(uint32_t, val)));      \
        val += k2 == key ? v2 : T(0);                                                                        \
    }
    DC_SEG_STEP(0x111, 0xF)
    DC_SEG_STEP(0x112, 0xF)
    DC_SEG_STEP(0x114, 0xF)
    DC_SEG_STEP(0x118, 0xF)
    DC_SEG_STEP(0x142, 0xA)
    if (!HALVES) DC_SEG_STEP(0x143, 0xC)
#undef DC_SEG_STEP
    uint32_t above = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)key, 0x130, 0xF, 0xF, false);
    if (HALVES && (threadIdx.x & 31u) == 31u) above = 0xFFFFFFFFu;
    uint64_t ends = __ballot(key != 0xFFFFFFFFu && above != key); // the last lane of every run
    const uint32_t lane = threadIdx.x & 63u;
    while (ends) {
        const uint32_t from = (uint32_t)__builtin_ctzll(ends);
        const uint32_t to = (uint32_t)__builtin_amdgcn_readlane((int)slot, from) & 63u;
        const T v = of_lane(val, from);
        mine += lane == to ? v : T(0);
        ends &= ends - 1;
    }
}

// One sub-stream as its lane sees it.  Stream words travel memory -> blk -> LDS ring -> r.
// The ring of a wave is 4 KiB, 4 KiB aligned; ring word j of the lane sits at byte
// (j % 16) * 256 + lane * 4 of it, so the lanes of a wave never collide on a bank.  Positions and block counts are
// kept times 8 (a block is 128 bits = 1024 units): bits 8-11 of a position are then the slot of its word as they
// stand, and bits 10-11 of a block count the slot of the block's first word.
// Huffman positions are kept one bit early (kLead): a window that begins there is "the next 11 bits, times 2" under a
// mask, which is the byte offset of the table entry, so a look-up needs no shift of its own.
// FEW: launches of few wavefronts (step_and_decode8_few).  A wave's 4 KiB of ring are followed by 4 KiB that hold the ring's first
// four words again, so that words behind one another in the stream can be read without a wrap, and four words for blocks that are
// nobody's.  Where the LDS is busier the second copy costs more than it saves: with four waves to a chunk (4096 x 4096 at
// 256 sub-streams 14.3 instead of 13.7 us), and where order_of_work says so.
constexpr int kMany = 0, kFew = 1, kFewAgain = 2; // the order of a decoder's work: one of the latter two for FEW, kFewAgain with the second copy
template <int ORDER> struct Ring {
    static constexpr int kStride = ORDER != kMany ? 2048 : kRingWords * 64; // words of LDS a wave
    static constexpr bool kAgain = ORDER == kFewAgain;
    static constexpr uint32_t kAgainAt = 4096, kNowhereAt = 5120; // bytes from the ring's start
};

template <int CODEC> struct Lead { static constexpr uint32_t kBits = CODEC == DC_CODEC_TANS ? 0 : 1; };
struct Stream {
    uint32_t pos;     // 8 * (position in bits - kLead)
    uint32_t asked;   // 1024 * (blocks asked for so far, f of the placement rule)
    uint32_t end;     // 1024 * (blocks of the stream)
    uint32_t r[4];    // the words at the position and behind it: all a half group can need (FEW: three, shifted to begin at it)
    uint32_t next;    // FEW: the table entry of the symbol at the position
    uint32_t nowhere; // FEW: the ring place of a block that is not the stream's
    uint32_t again[2]; // FEW: where blk[p] goes a second time
    uint32_t x4;      // tANS: 4 * state = byte offset of the state's table entry
    u32x4 blk[2];     // a block travels for two steps: asked for at step h, put into the ring at step h + 2
    uint32_t slot[2]; // where in the ring blk[p] goes
    bool pend[2];     // whether blk[p] is a block of this stream (asked for at the last step of parity p)
};

// What the lanes of one stream set share: where the block region of the set's area stands.
struct Region {
    const uint8_t *payload8;
    uint32_t next_block; // in 16-byte units from the payload start
    uint32_t max_off;    // last payload offset 20 bytes may be loaded from without leaving the blob
    uint64_t lanes;      // the lanes of the wave that belong to the set
};

// 16 bytes at an address that is a multiple of 4 only
typedef uint32_t u32x4_align4 __attribute__((ext_vector_type(4), aligned(4)));

// A block goes to the four ring words from `slot` on (block number b of a stream: ring words 4b .. 4b+3).
__device__ __forceinline__ void push_block(uint32_t slot, const u32x4 &blk)
{
    lds_u32 *w = (lds_u32 *)(uintptr_t)slot;
    w[0] = blk[0];
    w[64] = blk[1];
    w[128] = blk[2];
    w[192] = blk[3];
}

// The four words from the position on.  KEEP_FIRST: the word at the position is only read when the position has
// moved to another word, because its slot may have been given to a later block since (see stream_step).
template <bool KEEP_FIRST> __device__ __forceinline__ void read_window(Stream &s, uint32_t before, uint32_t ring_lane)
{
    const uint32_t first = lds_load32((s.pos & 0xF00u) | ring_lane);
    s.r[0] = KEEP_FIRST && ((s.pos ^ before) < 256u) ? s.r[0] : first;
#pragma unroll
    for (uint32_t k = 1; k < 4; k++) s.r[k] = lds_load32(((s.pos + 256u * k) & 0xF00u) | ring_lane);
}

// The lanes with `want` each take the next block of the region, in lane order.
template <bool UNIFORM>
__device__ __forceinline__ void take_blocks(Stream &s, Region &rg, bool want, u32x4 &dst)
{
    const uint64_t m = __ballot(want) & rg.lanes;
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (want) {
        dst = *reinterpret_cast<const u32x4 *>(rg.payload8 + (rg.next_block + rank) * kBlockBytes);
        s.asked += 1024;
    }
    rg.next_block += (uint32_t)__popcll(m);
    if (UNIFORM) rg.next_block = __builtin_amdgcn_readfirstlane(rg.next_block);
}

// One step of the placement rule (before every half group; P = the step's parity): the block asked for two
// steps before goes into the ring, then the lanes short of look-ahead ask for their next block.  The rule's
// 128*f - c < DC_LOOKAHEAD_BITS reads, times 8, asked < pos + 8*DC_LOOKAHEAD_BITS.
// Every lane loads; a lane that asks for nothing loads, and drops, a block that a lane below it asks for, or the
// one after the last asked for (stream_fetch has checked that the region and one block more lie inside the blob).
// A load that is always issued lets the wait for an earlier load be exact (it counts the loads issued
// since), so a block can stay in flight across the next step's load.
//
// The words of half group h are read when half group h - 1 is done, before step h, so that the step's arithmetic runs
// while they come.  Why they are there: a stream has at least DC_LOOKAHEAD_BITS - 88 = 304 bits placed beyond its
// position before its decision at any step, or all of its blocks; the ring lacks what was asked for at steps h - 1
// and h - 2; so beyond the position of h it holds at least 304 - 2*88 = 128 bits, and half a group uses at most 88.
// Why their slots are still theirs: block b goes into the slot of block b - 4 two steps after a position beyond
// 128*b - DC_LOOKAHEAD_BITS = 128*(b - 3) - 8, and is there from the next read on, three half groups after that
// position.  24 Huffman codes take at least 24 bits, so the position has left block b - 4.  tANS fields may be
// empty: its last 7 bits may still be needed then, but they lie in one word, which the lane has held since its
// position entered that word (KEEP_FIRST).
template <bool UNIFORM, int P, int CODEC>
__device__ __forceinline__ void stream_step(Stream &s, Region &rg, uint32_t ring_lane)
{
    if (s.pend[P]) push_block(s.slot[P], s.blk[P]);
    const uint32_t bound = s.pos + 8u * (DC_LOOKAHEAD_BITS + Lead<CODEC>::kBits);
    const bool want = s.asked < (bound < s.end ? bound : s.end);
    const uint64_t m = UNIFORM ? __ballot(want) : __ballot(want) & rg.lanes;
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    s.blk[P] = *reinterpret_cast<const u32x4 *>(rg.payload8 + (rg.next_block + rank) * kBlockBytes);
    s.slot[P] = (s.asked & 0xC00u) | ring_lane;
    s.asked += want ? 1024u : 0u;
    s.pend[P] = want;
    rg.next_block += (uint32_t)__popcll(m);
    if (UNIFORM) rg.next_block = __builtin_amdgcn_readfirstlane(rg.next_block);
}

// The table entry of the symbol that follows the first `by` bits of w (Huffman).
__device__ __forceinline__ uint32_t look_up(uint32_t w, uint32_t by, uint32_t tbl)
{
    return lds_load16(tbl + ((w >> (by & 31u)) & (2 * kTableEntries - 2)));
}

// N words, and word N behind them, shifted down by `by` < 32 bits.
template <int N> __device__ __forceinline__ void shift_down(uint32_t *w, uint32_t by)
{
#pragma unroll
    for (int i = 0; i < N; i++) w[i] = __builtin_amdgcn_alignbit(w[i + 1], w[i], by);
}

// Start of a sub-stream.  Block 0 of a stream is short: its first pad = 16 - hb bytes do not exist and
// its hb bytes lie among the heads, which follow the whole blocks of the set in lane order.  The lane
// loads the 20 bytes from the 4-byte boundary at or before the place where block 0 would start and
// shifts them down, so the ring holds block 0 with foreign bytes in front, and starts reading behind
// them.  Then step 0 of the rule runs for the three further times (a stream takes a block while it
// has blocks left and fewer than DC_LOOKAHEAD_BITS bits beyond its position 8*pad), and the first words
// are read.  (The step at the head of the decode loop is the fifth time; a tANS stream has read its
// first state by then.)
// What stream_fetch has asked memory for and stream_start puts into the ring.
struct StreamFetch {
    u32x4_align4 v; // the 20 bytes around the head of the stream
    uint32_t v4;
    uint32_t shift; // bytes to shift them down by
    uint32_t pad;   // bytes that block 0 lacks
    bool has_head;
    u32x4 b[3];     // up to three further blocks
    bool got[3];
};

// First half of the set-up: loads only, so that it can run before the decode table is built (the rings share
// their LDS with the scratch of the table build).
template <bool UNIFORM>
__device__ __forceinline__ void stream_fetch(Stream &s, Region &rg, uint32_t field, StreamFetch &f)
{
    // header field of the stream: blocks in all, and the bytes of block 0 less one
    uint32_t nb = field & 0xFFFu;
    const uint32_t hb = nb ? ((field >> 12) & 15u) + 1 : 0;
    const uint32_t pad = nb ? kBlockBytes - hb : 0;
    const uint32_t whole_incl = lanes_prefix_sum<!UNIFORM>(nb ? nb - 1 : 0);
    const uint32_t heads_incl = lanes_prefix_sum<!UNIFORM>(hb);
    uint32_t whole_total = (uint32_t)__builtin_amdgcn_readlane((int)whole_incl, 63);
    if (!UNIFORM) {
        const uint32_t lower = (uint32_t)__builtin_amdgcn_readlane((int)whole_incl, 31);
        whole_total = (threadIdx.x & 32u) ? whole_total : lower;
    }
    // The set's lanes take whole_total blocks in all, whatever the payload holds, and look one block further at most.
    // A region that the blob does not hold (a corrupt payload) is not read: its streams have no blocks then.
    if (rg.next_block + whole_total > rg.max_off / kBlockBytes) {
        nb = 0;
        rg.next_block = 0;
    }
    s.end = nb << 10;
    s.asked = 0;
    s.pend[0] = s.pend[1] = false;
    s.slot[0] = s.slot[1] = 0;
    f.pad = pad;
    f.has_head = nb != 0;
    f.shift = 0;
    if (nb) {
        uint32_t at = (rg.next_block + whole_total) * kBlockBytes + (heads_incl - hb) - pad; // the header lies before it
        at = at < rg.max_off ? at : rg.max_off;
        const uint8_t *p = rg.payload8 + (at & ~3u);
        f.v = *reinterpret_cast<const u32x4_align4 *>(p);
        f.v4 = *reinterpret_cast<const uint32_t *>(p + 16);
        f.shift = at & 3u;
        s.asked = 1024;
    }
#pragma unroll
    for (int t = 0; t < 3; t++) {
        f.got[t] = s.asked < s.end && s.asked < ((8u * pad + DC_LOOKAHEAD_BITS) << 3); // 128 f < c + look-ahead, times 8
        take_blocks<UNIFORM>(s, rg, f.got[t], f.b[t]);
    }
}

// Second half: block 0 shifted into place and the further blocks go into the ring, and the first words are read.
// A tANS stream reads its first state, its first 11 bits, and the words after them.
template <int CODEC, int S, int ORDER>
__device__ __forceinline__ void stream_start(Stream &s, const StreamFetch &f, uint32_t ring_lane, uint32_t tbl)
{
    using R = Ring<ORDER>;
    if (f.has_head) {
        const u32x4 b0 = {__builtin_amdgcn_alignbyte(f.v[1], f.v[0], f.shift), __builtin_amdgcn_alignbyte(f.v[2], f.v[1], f.shift),
                          __builtin_amdgcn_alignbyte(f.v[3], f.v[2], f.shift), __builtin_amdgcn_alignbyte(f.v4, f.v[3], f.shift)};
        push_block(ring_lane, b0);
        if (R::kAgain) push_block(ring_lane + R::kAgainAt, b0);
    }
#pragma unroll
    for (int t = 0; t < 3; t++)
        if (f.got[t]) push_block(ring_lane + ((t + 1) << 10), f.b[t]);
    s.pos = 64u * f.pad - 8u * Lead<CODEC>::kBits; // the stream begins `pad` bytes into block 0
    read_window<false>(s, 0, ring_lane);
    if (ORDER != kMany) {
        s.nowhere = ring_lane + R::kNowhereAt;
#pragma unroll
        for (int p = 0; p < 2; p++) {
            s.slot[p] = s.again[p] = s.nowhere;
            s.blk[p] = u32x4{0, 0, 0, 0};
        }
        shift_down<3>(s.r, s.pos >> 3);
        s.next = look_up(s.r[0], 0, tbl);
    }
    s.x4 = 0;
    if (CODEC == DC_CODEC_TANS) {
        const uint32_t before = s.pos;
        s.x4 = (__builtin_amdgcn_alignbit(s.r[1], s.r[0], s.pos >> 3) & (kTableEntries - 1)) << 2;
        s.pos += 8u * kPeekBits;
        read_window<true>(s, before, ring_lane);
    }
}

// The next two symbols out of the 32 bits of w (at most 22, and the lead, are used): their table entries, symbol in
// byte 1.  Returns the bits used in its low byte.
// Huffman: entry = length | symbol << 8; w begins one bit early, so the byte offsets of the entries are w and
// w >> length_0 under the mask.
// tANS: table entry of a state = nb | value << 8 | (4 * base) << 16, where nb is the width of the state's
// field and base the next state before the field is added; bits 4-7 are 0, so that the low five bits of an
// entry can be used as a field width or offset as they are.
template <int CODEC> __device__ __forceinline__ uint32_t two_symbols(uint32_t w, uint32_t &x4, uint32_t tbl, uint32_t e[2])
{
    constexpr uint32_t kOffsetMask = 2 * kTableEntries - 2;
    if (CODEC == DC_CODEC_TANS) {
        e[0] = lds_load32(tbl + x4);
        x4 = (e[0] >> 16) + (__builtin_amdgcn_ubfe(w, 0u, e[0]) << 2);
        e[1] = lds_load32(tbl + x4);
        x4 = (e[1] >> 16) + (__builtin_amdgcn_ubfe(w, e[0], e[1]) << 2);
    } else {
        e[0] = lds_load16(tbl + (w & kOffsetMask));
        e[1] = lds_load16(tbl + ((w >> (e[0] & 31u)) & kOffsetMask));
    }
    return e[0] + e[1];
}

// bytes 1 of four entries -> one little-endian word of four symbols
__device__ __forceinline__ uint32_t pack4(uint32_t e0, uint32_t e1, uint32_t e2, uint32_t e3)
{
    const uint32_t lo = __builtin_amdgcn_perm(e1, e0, 0x0c0c0501u);
    const uint32_t hi = __builtin_amdgcn_perm(e3, e2, 0x0c0c0501u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// Half a group: the table entries of 8 symbols, at most 88 bits, out of the four words in r.  The words are shifted down once by the position
// inside its word (96 bits are left, the lead among them) and then by the bits every pair of symbols has used, so that every pair starts at
// bit 0 of w0: no lane waits for another's refill, and nothing is conditional.  A lane past its stream's last symbol
// decodes on over what the ring holds (it has no blocks left to ask for, so its position no longer matters) and its
// symbols are dropped where they would be stored.
template <int CODEC>
__device__ __forceinline__ void decode8(Stream &s, uint32_t tbl, uint32_t ring_lane, uint32_t e[8])
{
    const uint32_t o = s.pos >> 3; // shifts read the low 5 bits
    uint32_t w0 = __builtin_amdgcn_alignbit(s.r[1], s.r[0], o);
    uint32_t w1 = __builtin_amdgcn_alignbit(s.r[2], s.r[1], o);
    uint32_t w2 = __builtin_amdgcn_alignbit(s.r[3], s.r[2], o);
    const uint32_t u0 = two_symbols<CODEC>(w0, s.x4, tbl, e);
    w0 = __builtin_amdgcn_alignbit(w1, w0, u0);
    w1 = __builtin_amdgcn_alignbit(w2, w1, u0);
    w2 >>= u0 & 31u;
    const uint32_t u1 = two_symbols<CODEC>(w0, s.x4, tbl, e + 2);
    w0 = __builtin_amdgcn_alignbit(w1, w0, u1);
    w1 = __builtin_amdgcn_alignbit(w2, w1, u1);
    const uint32_t u2 = two_symbols<CODEC>(w0, s.x4, tbl, e + 4);
    w0 = __builtin_amdgcn_alignbit(w1, w0, u2);
    const uint32_t u3 = two_symbols<CODEC>(w0, s.x4, tbl, e + 6);
    const uint32_t before = s.pos;
    s.pos += ((u0 + u1 + u2 + u3) & 0xFFu) << 3;
    read_window<CODEC == DC_CODEC_TANS>(s, before, ring_lane);
}

// Work of the caller that half a group's look-ups can hide: early() while the second entry is on its way, late(0) and late(1)
// while the fifth and sixth are.
struct Nothing {
    __device__ __forceinline__ void early() const {}
    __device__ __forceinline__ void late(int) const {}
};
template <typename F> struct Early {
    F early;
    __device__ __forceinline__ void late(int) const {}
};
template <typename F> struct Late {
    F late;
    __device__ __forceinline__ void early() const {}
};
template <typename F> __device__ __forceinline__ Early<F> early(F f) { return {f}; }
template <typename F> __device__ __forceinline__ Late<F> late(F f) { return {f}; }

// FEW: a step of the placement rule and half a group for launches that have one or two wavefronts to a SIMD (Huffman).  Such a wave has
// nothing but its own instructions to fill the time that a look-up takes, 27 ns of the 33 that a link of the chain (read, shift, mask)
// takes by itself; with the step, then the half group, then the next words one after the other a link took 43 ns.  So the order
// is fixed here: the next look-up is asked for as soon as an entry has come, and everything that does not decide it stands behind
// it.  The words of the next half group are read when 6 of the 8 symbols are known, and its first look-up ends this one; a
// block goes into the ring without a branch, to a place of its own if the lane asked for none, so that all of it is one
// block of code.  77 instead of 94 us for 256 chunks of 64 KiB at 32 sub-streams, 39 instead of 47 at 64.
// Reading at the 7th symbol and not at the 9th leaves what stream_step says of the ring as it is: no step lies between, so what has been
// put into the ring is the same, the bits needed end where they did, and the position is still 22 codes beyond the one at which
// the youngest block in the ring was asked for, 22 bits at least, the lead among them, and so past block b - 4.
template <bool UNIFORM, int P, bool AGAIN, typename Meanwhile>
__device__ __forceinline__ void step_and_decode8_few(Stream &s, Region &rg, uint32_t tbl, uint32_t ring_lane, uint32_t e[8], Meanwhile meanwhile)
{
    uint32_t w[4] = {s.r[0], s.r[1], s.r[2], 0};
    e[0] = s.next;
    keep_order();
    e[1] = look_up(w[0], e[0], tbl);
    keep_order();
    shift_down<3>(w, e[0]);
    push_block(s.slot[P], s.blk[P]);
    if (AGAIN) push_block(s.again[P], s.blk[P]);
    keep_order();
    meanwhile.early();
    keep_order();
    e[2] = look_up(w[0], e[1], tbl);
    keep_order();
    shift_down<3>(w, e[1]);
    const uint32_t bound = s.pos + 8u * (DC_LOOKAHEAD_BITS + Lead<DC_CODEC_HUFFMAN>::kBits);
    const bool want = s.asked < (bound < s.end ? bound : s.end);
    const uint64_t m = UNIFORM ? __ballot(want) : __ballot(want) & rg.lanes;
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    keep_order();
    e[3] = look_up(w[0], e[2], tbl);
    keep_order();
    shift_down<2>(w, e[2]); // from here on two words hold what may still be needed, one after the sixth symbol
    s.blk[P] = *reinterpret_cast<const u32x4 *>(rg.payload8 + (rg.next_block + rank) * kBlockBytes);
    s.slot[P] = want ? (s.asked & 0xC00u) | ring_lane : s.nowhere;
    if (AGAIN) s.again[P] = s.slot[P] == ring_lane ? ring_lane + Ring<kFewAgain>::kAgainAt : s.nowhere;
    s.asked += want ? 1024u : 0u;
    rg.next_block += (uint32_t)__popcll(m);
    if (UNIFORM) rg.next_block = __builtin_amdgcn_readfirstlane(rg.next_block);
    keep_order();
    e[4] = look_up(w[0], e[3], tbl);
    keep_order();
    shift_down<2>(w, e[3]);
    meanwhile.late(0);
    keep_order();
    e[5] = look_up(w[0], e[4], tbl);
    keep_order();
    w[2] = 0;
    shift_down<2>(w, e[4]);
    meanwhile.late(1);
    keep_order();
    e[6] = look_up(w[0], e[5], tbl);
    keep_order();
    shift_down<1>(w, e[5]);
    s.pos += ((e[0] + e[1] + e[2] + e[3] + e[4] + e[5]) & 0xFFu) << 3;
    uint32_t v[5]; // from 31 bits before the position to 129 behind it; two symbols and half a group may need 110, and the lead
    const uint32_t at = (s.pos & 0xF00u) | ring_lane;
#pragma unroll
    for (uint32_t k = 0; k < 5; k++) v[k] = lds_load32(AGAIN ? at + 256u * k : ((s.pos + 256u * k) & 0xF00u) | ring_lane);
    keep_order();
    e[7] = look_up(w[0], e[6], tbl);
    keep_order();
    shift_down<4>(v, s.pos >> 3);
    v[4] = 0;
    shift_down<4>(v, e[6]);
    keep_order();
    s.next = look_up(v[0], e[7], tbl);
    keep_order();
    shift_down<3>(v, e[7]);
#pragma unroll
    for (int i = 0; i < 3; i++) s.r[i] = v[i];
    s.pos += ((e[6] + e[7]) & 0xFFu) << 3;
}

// A step of the placement rule and the half group behind it.
template <int S, int P, int CODEC, int ORDER, typename Meanwhile = Nothing>
__device__ __forceinline__ void step_and_decode8(Stream &s, Region &rg, uint32_t tbl, uint32_t ring_lane, uint32_t e[8],
                                                 Meanwhile meanwhile = Meanwhile())
{
    constexpr bool UNIFORM = S >= 64;
    if constexpr (ORDER != kMany) {
        step_and_decode8_few<UNIFORM, P, Ring<ORDER>::kAgain>(s, rg, tbl, ring_lane, e, meanwhile);
    } else {
        stream_step<UNIFORM, P, CODEC>(s, rg, ring_lane);
        decode8<CODEC>(s, tbl, ring_lane, e);
    }
}

// One whole group of 16 symbols with the two steps of the placement rule that precede its halves.
template <int S, int CODEC, int ORDER, typename Meanwhile = Nothing>
__device__ __forceinline__ void decode16(Stream &s, Region &rg, uint32_t tbl, uint32_t ring_lane, uint32_t out[4],
                                         Meanwhile meanwhile = Meanwhile())
{
    uint32_t e[8], f[8];
    step_and_decode8<S, 0, CODEC, ORDER>(s, rg, tbl, ring_lane, e, meanwhile);
    if constexpr (ORDER != kMany) {
        step_and_decode8<S, 1, CODEC, ORDER>(s, rg, tbl, ring_lane, f, late([&](int i) {
            out[i] = pack4(e[4 * i], e[4 * i + 1], e[4 * i + 2], e[4 * i + 3]);
            in_register<false>(out[i]);
        }));
    } else {
        out[0] = pack4(e[0], e[1], e[2], e[3]);
        out[1] = pack4(e[4], e[5], e[6], e[7]);
        step_and_decode8<S, 1, CODEC, ORDER>(s, rg, tbl, ring_lane, f);
    }
    out[2] = pack4(f[0], f[1], f[2], f[3]);
    out[3] = pack4(f[4], f[5], f[6], f[7]);
}

__device__ __forceinline__ uint32_t bf16x2(float a, float b)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    bf16x2_t v;
    v[0] = (__bf16)a;
    v[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
}

// acc + a.lo * b.lo + a.hi * b.hi for two pairs of bf16 values
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc)
{
    // The builtin, not inline assembly: the result of a dot product may be read by another instruction three wait states
    // later at the earliest, and the compiler only keeps that distance for instructions it knows.
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc, false);
}

// int8 value number N of a word as fp32: one v_cvt_f32_i32 whose operand selects the byte and sign-extends it
template <int N> __device__ __forceinline__ float byte_f32(uint32_t w) { return (float)(int)(int8_t)(w >> (8 * N)); }

// Four int8 values in a word -> fp32, times the row scale (one rounding, as the dequantisation is defined).
__device__ __forceinline__ void word_to_scaled_f32(uint32_t w, float s, float f[4])
{
    f[0] = byte_f32<0>(w) * s;
    f[1] = byte_f32<1>(w) * s;
    f[2] = byte_f32<2>(w) * s;
    f[3] = byte_f32<3>(w) * s;
}

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }


// The tANS table of a chunk (S >= 64: the workgroup's threads are the chunk's).  front: 4 KiB of LDS not yet
// in use (the rings); tbl: the LDS address of the 2048 entries; cumq: 256 words; wave_sum: one word per wave.  The threads
// read the 256 frequencies, take their prefix sums (value v owns places cum[v] .. cum[v] + q[v] - 1) and mark
// the first place of every value; then every thread takes 2048/threads consecutive places, finds each
// place's value, and numbers the place among the places of its value by the order of the states (the places
// with their 11 bits reversed): place p of a value with places a .. e-1 has as many states below it as there are
// places p' of the value whose reversal is smaller, that is, for every set bit i of p, the places of the value that agree with p
// below bit i and have bit i clear: those that leave c = p mod 2^i when divided by M = 2^(i+1),
// (e + M - 1 - c) div M - (a + M - 1 - c) div M of them.  The sums over a and over e are kept in the halves of one word, which neither
// additions nor, with a mask, shifts let into each other: four plain operations a bit for both.
// (What bounds it: the vector ALU, and registers, which set how many wavefronts run through the whole decode.  All eleven bits of
// every place were 530 of the 720 vector operations of a wave at 256 sub-streams, whose loop over 64 KiB takes 2400.  Only the bits
// that can count, with a place's value, frequency, distance and number in a word each, took 217 registers at 64 sub-streams and 107 at
// 128, where the LDS lets 168 and 96 be used: 2500 chunks of 64 KiB 84 -> 119 us, 12000 of 16 KiB 117 -> 126.  As it is now, 142 and
// 82 registers: 77.2 and 102.4; 2200 chunks of 64 KiB at 128 sub-streams 66 -> 78 -> 61.7; at 256 16000 of 4 KiB 84.6 -> 69.2 -> 63.3.
// The same halves by packed operations of 16 bits, three a bit, take up to 4 % longer: their encoding is twice as long.)
// Returns false (for every thread alike) when the frequencies do not add up to 2048; nothing is decoded then.
template <int S>
__device__ __forceinline__ bool build_tans_table(const uint8_t *payload8, uint32_t ct, uint32_t lane, uint32_t wave,
                                                 uint32_t *front, uint32_t tbl, uint32_t *cumq, uint32_t *wave_sum)
{
    using G = Geometry<S>;
    constexpr int WAVES = G::kWaves;
    constexpr int TPC = G::kThreadsPerChunk;
    constexpr int SPL = G::kSymbolsPerLane;
    constexpr int EPT = kTableEntries / TPC;
    constexpr uint32_t L = kTableEntries;
    uint16_t *marks = reinterpret_cast<uint16_t *>(front);
    {
        uint4 *z = reinterpret_cast<uint4 *>(marks);
        for (uint32_t i = ct; i < kTableEntries * 2 / 16; i += TPC) z[i] = make_uint4(0, 0, 0, 0);
    }
    uint32_t q[SPL], mine = 0;
#pragma unroll
    for (int s = 0; s < SPL; s++) {
        const uint32_t v = ct * SPL + s;
        const uint8_t *g = payload8 + 3 * (v >> 1); // two 12-bit frequencies in three bytes
        q[s] = (v & 1u) ? ((uint32_t)g[1] >> 4 | (uint32_t)g[2] << 4) : ((uint32_t)g[0] | ((uint32_t)g[1] & 15u) << 8);
        mine += q[s];
    }
    const uint32_t incl = lanes_prefix_sum<false>(mine);
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t cum = incl - mine, total = 0;
#pragma unroll
    for (int w = 0; w < WAVES; w++) {
        const uint32_t c = wave_sum[w];
        if ((uint32_t)w < wave) cum += c;
        total += c;
    }
    if (total != L) return false;
#pragma unroll
    for (int s = 0; s < SPL; s++) {
        const uint32_t v = ct * SPL + s;
        cumq[v] = cum | q[s] << 16;
        if (q[s]) {
            marks[cum] = (uint16_t)(v + 1);
            // also at the first place of every later wave that the value reaches into
            for (uint32_t p = (cum / (L / WAVES) + 1) * (L / WAVES); p < cum + q[s]; p += L / WAVES) marks[p] = (uint16_t)(v + 1);
        }
        cum += q[s];
    }
    __syncthreads();
    uint32_t w16[EPT / 2];
    {
        const uint4 *m4 = reinterpret_cast<const uint4 *>(marks + EPT * ct);
#pragma unroll
        for (int i = 0; i < EPT / 8; i++) {
            const uint4 v = m4[i];
            w16[4 * i] = v.x; w16[4 * i + 1] = v.y; w16[4 * i + 2] = v.z; w16[4 * i + 3] = v.w;
        }
    }
    uint32_t tail = 0; // last mark among this thread's places
#pragma unroll
    for (int i = 0; i < EPT / 2; i++) {
        const uint32_t lo = w16[i] & 0xFFFFu, hi = w16[i] >> 16;
        tail = lo ? lo : tail;
        tail = hi ? hi : tail;
    }
    uint32_t cur = lanes_last_nonzero_below<false>(tail);
    // of a place: its value, the halves a and e, and the sums over them, whose difference will be the number of the place's state
    uint32_t value[EPT], span[EPT], sum[EPT], most = 0;
#pragma unroll
    for (int i = 0; i < EPT; i++) {
        const uint32_t m = (i & 1) ? w16[i / 2] >> 16 : w16[i / 2] & 0xFFFFu;
        cur = m ? m : cur;
        value[i] = (cur - 1) & 255u;
        const uint32_t cq = cumq[value[i]];
        span[i] = sum[i] = cq + (cq << 16);
        most = cq > most ? cq : most;
    }
    // Bit b of the place counts where the value has more than 2^b places: of 2^b places in a row no other agrees with this one below
    // bit b.  So the loop ends with the most frequent value that the wave holds; and the lowest bits are the same in every thread.
    auto both = [](uint32_t v) { return v << 16 | v; };
    constexpr uint32_t LOW = EPT == 32 ? 5 : EPT == 16 ? 4 : 3; // EPT = 2^LOW
#pragma unroll
    for (uint32_t b = 0; b < LOW; b++)
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)EPT; i++)
            if (i >> b & 1u) sum[i] += (span[i] + both((2u << b) - 1 - (i & ((1u << b) - 1)))) >> (b + 1) & both(0xFFFFu >> (b + 1));
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)EPT; i++) span[i] -= both(i); // from here on c is what EPT * ct leaves
#pragma unroll
    for (uint32_t b = LOW; b < (uint32_t)kPeekBits; b++) {
        if (!__any(most >> 16 > 1u << b)) break;
        const uint32_t from = both((2u << b) - 1 - EPT * (ct & ((1u << (b - LOW)) - 1)));
        const uint32_t mask = ct >> (b - LOW) & 1u ? both(0xFFFFu >> (b + 1)) : 0u;
#pragma unroll
        for (int i = 0; i < EPT; i++) sum[i] += (span[i] + from) >> (b + 1) & mask;
    }
#pragma unroll
    for (int i = 0; i < EPT; i++) {
        const uint32_t p = EPT * ct + i, k = (sum[i] >> 16) - (sum[i] & 0xFFFFu);
        const uint32_t nb = (uint32_t)__builtin_clz(k | 1u) - (31 - kPeekBits);
        const uint32_t base = ((k << nb) - L) & (L - 1);
        *(lds_u32 *)(uintptr_t)(tbl + 4 * (__brev(p) >> (32 - kPeekBits))) = nb | value[i] << 8 | base << 18;
    }
    __syncthreads();
    return true;
}

// The decode table of a chunk, by its TPC threads (WAVES waves; HALVES: each half of a wave for a chunk of its own), of which this one is number ct.
// nib: the code lengths of its values ct * SPL + s, four bits each.  Slot p of the table in code order (p = the next 11 stream bits, first bit
// most significant) belongs to the code that covers p; codes in canonical order cover consecutive runs of 2^(11-length) slots.
// (1) A value's rank among those of its length comes from a ballot for each length (four or eight values a lane: from counters of the lengths, three to
// a register, summed over the lanes), the counts of the waves before from LDS.  Lane l has the counts of length l, and the first
// slots of the lengths are a prefix sum over the lanes.  (2) Every value marks the first slot of its run.  A mark
// is the run's first slot above the table entry, so that the mark that covers a slot is the largest up to it: every thread takes
// 2048/threads consecutive slots, extends the marks forward over them, and writes the entries to the table at the
// bit-reversed slot numbers (the stream is read least significant bit first).
// (With the counters at 256 sub-streams too, the first codes added up by one lane, and marks without their slot, which a comparison and a
// selection each carry forward, it took 370 instructions there, 215 now: a chunk alone on its compute unit 0.8 instead of 1.2 us.)
// marks: 2048 words of the rings, SHARED: and of the place of the tables; counts: 16 words a wave at the place of the table (several waves);
// table: the LDS address of 2048 entries of 16 bits.
template <int TPC, int WAVES, bool HALVES, bool SHARED>
__device__ __forceinline__ void build_code_table(uint32_t nib, uint32_t ct, uint32_t wave, uint32_t *marks, uint32_t (*counts)[16], uint32_t table)
{
    constexpr int SPL = 256 / TPC;
    constexpr uint32_t EPT = kTableEntries / TPC; // slots a thread fills
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t l = HALVES ? lane & 31u : lane; // the length that this lane has the counts of
#pragma unroll
    for (uint32_t i = 0; i < EPT / 4; i++) reinterpret_cast<u32x4 *>(marks)[ct + i * TPC] = u32x4{0, 0, 0, 0};
    uint32_t len[SPL], rank[SPL], all = 0, waves_before = 0;
#pragma unroll
    for (int s = 0; s < SPL; s++) {
        len[s] = (nib >> (4 * s)) & 15u;
        if (len[s] > DC_MAX_CODE_LEN) len[s] = 0;
        rank[s] = 0;
    }
    if constexpr (SPL <= 2) {
#pragma unroll
        for (uint32_t n = 1; n <= DC_MAX_CODE_LEN; n++) {
            uint32_t total = 0, before = 0; // of this length: in the wave, with the lanes before
            uint64_t m[SPL];
#pragma unroll
            for (int s = 0; s < SPL; s++) {
                m[s] = __ballot(len[s] == n);
                before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[s] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[s], before));
                total += (uint32_t)__popcll(m[s]);
            }
            rank[0] = len[0] == n ? before : rank[0];
            if (SPL == 2) rank[SPL - 1] = len[SPL - 1] == n ? before + (len[0] == n ? 1u : 0u) : rank[SPL - 1];
            all = with_lane(all, n, total);
        }
        if (lane < 16) counts[wave][lane] = all;
        __syncthreads();
        all = 0;
#pragma unroll
        for (int w = 0; w < WAVES; w++) {
            const uint32_t c = counts[0][16 * w + lane]; // (of no use from lane 16 on)
            waves_before += (uint32_t)w < wave ? c : 0u;
            all += c;
        }
    } else {
        // ten bits a length: length n in register (n-1)/3
        uint32_t before[4] = {0, 0, 0, 0}, total = 0;
#pragma unroll
        for (int s = 0; s < SPL; s++)
#pragma unroll
            for (uint32_t r = 0; r < 4; r++)
                if (len[s] != 0 && (len[s] - 1) / 3 == r) before[r] += 1u << (10 * ((len[s] - 1) % 3));
#pragma unroll
        for (uint32_t r = 0; r < 4; r++) {
            const uint32_t incl = lanes_prefix_sum<HALVES>(before[r]);
            before[r] = incl - before[r];
            const uint32_t t = (uint32_t)__shfl((int)incl, TPC - 1, TPC);
            total = (l - 1) / 3 == r ? t : total;
        }
        all = (total >> (10 * ((l - 1) % 3))) & 1023u;
#pragma unroll
        for (int s = 0; s < SPL; s++) {
            const uint32_t r = (len[s] - 1) / 3, sh = 10 * ((len[s] - 1) % 3);
            const uint32_t packed = r == 0 ? before[0] : r == 1 ? before[1] : r == 2 ? before[2] : before[3];
            rank[s] = (packed >> sh) & 1023u;
#pragma unroll
            for (uint32_t q = 0; q < 4; q++)
                if (r == q && len[s] != 0) before[q] += 1u << sh;
        }
        __syncthreads(); // the marks are clear
    }
    const uint32_t up = l <= DC_MAX_CODE_LEN ? kPeekBits - l : 0u;
    uint32_t first = l != 0 && l <= DC_MAX_CODE_LEN ? all << up : 0u; // slots of this length, then of those up to it
    const uint32_t own = first;
    first += dpp_or_zero<0x111, 0xF>(first);
    first += dpp_or_zero<0x112, 0xF>(first);
    first += dpp_or_zero<0x114, 0xF>(first);
    first += dpp_or_zero<0x118, 0xF>(first);
    first += (waves_before << up) - own; // the first slot of this wave's first value of the length
    // Thread ct's slots lie from word EPT * ct on, by fours in an order in which the lanes of a read spread over the banks.
    constexpr uint32_t FOURS = EPT / 4;
    auto place = [&](uint32_t p) { return p ^ ((p >> 6) & (FOURS - 1)) << 2; };
#pragma unroll
    for (int s = 0; s < SPL; s++) {
        const uint32_t run = (uint32_t)kTableEntries >> len[s];
        const uint32_t start = (uint32_t)__shfl((int)first, (int)len[s], HALVES ? 32 : 64) + (rank[s] << (kPeekBits - len[s]));
        if (len[s] != 0 && start < (uint32_t)kTableEntries) {
            const uint32_t mark = start << 16 | (ct * SPL + s) << 8 | len[s]; // never 0: the length is not
            marks[place(start)] = mark;
            // also at the first slot of every later wave that the run reaches into, so that no wave needs a mark from another wave's slots
            if (WAVES > 1) {
                constexpr uint32_t SHARE = kTableEntries / WAVES;
                const uint32_t end = start + run < (uint32_t)kTableEntries ? start + run : kTableEntries;
#pragma unroll 1
                for (uint32_t p = (start | (SHARE - 1)) + 1; p < end; p += SHARE) marks[place(p)] = mark;
            }
        }
    }
    __syncthreads();
    uint32_t w[EPT], tail = 0; // the last mark among this thread's slots
    const uint32_t turned = place(EPT * ct) - EPT * ct; // 4 times what the number of a four is combined with
#pragma unroll
    for (uint32_t i = 0; i < FOURS; i++) {
        const u32x4 v = *reinterpret_cast<const u32x4 *>(marks + EPT * ct + (turned ^ (4 * i)));
#pragma unroll
        for (int j = 0; j < 4; j++) {
            w[4 * i + j] = v[j];
            tail = v[j] > tail ? v[j] : tail;
        }
    }
    uint32_t cur = lanes_largest_below<HALVES>(tail);
    if (SHARED) __syncthreads(); // the marks have been read
    // slot EPT*ct + j in code order = slot bitrev(j) << (11-e) | bitrev(ct) in stream order, EPT = 2^e
    constexpr int E = EPT == 64 ? 6 : EPT == 32 ? 5 : EPT == 16 ? 4 : 3;
    const uint32_t out = table + 2 * (__brev(ct) >> (32 - (kPeekBits - E)));
#pragma unroll
    for (uint32_t i = 0; i < EPT; i++) {
        cur = w[i] > cur ? w[i] : cur;
        *(lds_u16 *)(uintptr_t)(out + 2 * ((__brev(i) >> (32 - E)) << (kPeekBits - E))) = (uint16_t)cur;
    }
    __syncthreads();
}

// A row's result from its sum.  y_i = scale_i * sum; W8A8: y_i = (float(sum) * scale_i) * x_scale, each step rounded
// once, in this order.
__device__ __forceinline__ float scaled_sum(const MatrixArgs &m, float scale, float sum) { return scale * sum; }
__device__ __forceinline__ float scaled_sum(const MatrixArgs &m, float scale, int32_t sum) { return ((float)sum * scale) * m.x_scale; }
__device__ __forceinline__ void store_row(const MatrixArgs &m, uint32_t row, float y)
{
    m.y_accum[row] = y;
    if (m.y_bf16) m.y_bf16[row] = (uint16_t)(bf16x2(y, 0.0f) & 0xFFFFu);
}

template <int S, int MODE, int CODEC, bool FEW = false, bool TRACE = false, bool AGAIN = FEW && S < 256>
__global__ __launch_bounds__(Geometry<S>::kThreads) void dc_decode_kernel(ArgsOf<MODE> a)
{
    using G = Geometry<S>;
    // traced launches: when the workgroup began and ended (ticks of the constant 100 MHz clock), where it ran (the
    // HW_ID register, the XCC_ID register above it) and what it did with its chunk
    const uint64_t began = TRACE ? wall_clock64() : 0;
    auto leave_record = [&](uint32_t did) {
        if (TRACE && threadIdx.x == 0) {
            uint64_t *r = a.trace + 4 * (size_t)blockIdx.x;
            r[0] = began;
            r[1] = wall_clock64();
            r[2] = (uint64_t)(uint32_t)__builtin_amdgcn_s_getreg((32 - 1) << 11 | 4) |
                   (uint64_t)(uint32_t)__builtin_amdgcn_s_getreg((32 - 1) << 11 | 20) << 32;
            r[3] = did;
        }
    };
    constexpr int LPC = G::kLanesPerChunk;
    constexpr int CPW = G::kChunksPerWave;
    constexpr int WAVES = G::kWaves;
    constexpr int TPC = G::kThreadsPerChunk;
    constexpr int SPL = G::kSymbolsPerLane;
    static_assert(CODEC == DC_CODEC_HUFFMAN || S >= 64, "tANS: the workgroup's threads are the chunk's");
    static_assert(CODEC == DC_CODEC_HUFFMAN || !FEW, "tANS keeps the word its position lies in (see stream_step)");
    constexpr uint32_t kFront = CODEC == DC_CODEC_TANS ? 384 : 128; // code description at the start of a payload
    constexpr uint32_t kHeader = (kFront + 2 * S + 4 * (S / Geometry<S>::kLanesPerChunk) + 15) / 16 * 16;

    // One block of LDS: the rings (4 KiB a wave, 4 KiB aligned) and then the decode tables.  While
    // the tables are built, before any ring is used, the front part holds the slot markers (8 KiB a chunk; where the rings are
    // smaller, they reach into the tables) and the start of the table part holds the waves' counts of the lengths.
    constexpr int ORDER = AGAIN ? kFewAgain : FEW ? kFew : kMany;
    static_assert(FEW || !AGAIN, "a second copy of what only FEW reads");
    constexpr int kRingStride = Ring<ORDER>::kStride;
    constexpr int kFrontWords = FEW ? WAVES * kRingStride : (WAVES > CPW ? WAVES : CPW) * kRingStride;
    // (tANS: 2048 entries of 32 bits, then 256 words of (first place, frequency) and a word per wave)
    constexpr int kTableWords = CODEC == DC_CODEC_TANS ? kTableEntries + 256 + 16 : CPW * kTableEntries / 2;
    __shared__ __attribute__((aligned(4 * kRingStride))) uint32_t lds_all[kFrontWords + kTableWords];
    uint32_t(*lds_counts)[16] = reinterpret_cast<uint32_t(*)[16]>(lds_all + kFrontWords); // [wave][length]

    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = threadIdx.x >> 6;
    const uint32_t sub = lane / LPC;
    const uint32_t cl = lane % LPC;              // lane inside the chunk's share of the wave
    const uint32_t ct = wave * 64 + cl;          // thread inside the chunk = sub-stream number
    const uint64_t k = (uint64_t)blockIdx.x * CPW + sub;

    // ---- the blob's trailer: a blob of another format, or of other parameters, is left undecoded
    const u32x4 closing = *reinterpret_cast<const u32x4 *>(a.blob + a.blob_bytes - DC_TRAILER_BYTES);
    // ---- chunk table entry, checked so that nothing below can leave the blob or the destination
    // (asked for together with the trailer, and every word of that at once: compared word by word, with a branch behind each, they were four
    // trips one after the other and the entry a fifth)
    const dc_chunk ent = a.table[k < a.n_chunks ? k : a.n_chunks - 1];
    if (G::kChunksPerWave == 1) in_registers(closing, ent.off, ent.comp_bytes, ent.raw_bytes_flags);
    auto two = [](uint32_t low, uint32_t high) { return (uint64_t)high << 32 | low; };
    bool active = two(closing[0], closing[1]) == two(a.trailer[0], a.trailer[1]) && two(closing[2], closing[3]) == two(a.trailer[2], a.trailer[3]) &&
                  k < a.n_chunks;
    const uint32_t raw = ent.raw_bytes_flags & ~DC_CHUNK_RAW;
    const bool is_raw = (ent.raw_bytes_flags & DC_CHUNK_RAW) != 0;
    // fused modes: the matrix the chunk belongs to, and the chunk's number inside it
    const MatrixArgs none = {};
    const MatrixArgs &mat = [&]() -> const MatrixArgs & {
        if constexpr (MODE == kModeI8) {
            return none; // nothing below asks for it
        } else {
            uint32_t mi = 0;
            if (a.n_mats > 1) // (one load and no loop: a loop over the descriptors was a trip to memory for each of them)
#pragma unroll
                for (uint32_t i = 0; i < DC_MAX_MATRICES - 1; i++) mi += (uint32_t)k >= a.next_first[i] ? 1u : 0u;
            return a.mats[mi];
        }
    }();
    const uint64_t dst_cap = MODE == kModeI8 ? a.dst_cap : (uint64_t)mat.rows * mat.cols;
    // first decoded byte of the chunk (in the buffer, or in its matrix)
    const uint64_t dst_pos = (MODE == kModeI8 ? k : k - mat.first_chunk) * (uint64_t)a.chunk_bytes;
    active = active && raw >= 1 && raw <= a.chunk_bytes && (ent.off & 15) == 0 && ent.off <= a.blob_bytes &&
             ent.comp_bytes <= a.blob_bytes - ent.off && ent.comp_bytes >= 16 && dst_pos + raw <= dst_cap &&
             (is_raw ? ent.comp_bytes >= ((raw + 15u) & ~15u) : ent.comp_bytes >= kHeader);
    const uint8_t *payload8 = a.blob + (active ? ent.off : 0);
    const uint32_t *payload = reinterpret_cast<const uint32_t *>(payload8);
    const bool huff = active && !is_raw;

    // The chunk's table, as a place in lds_all and not as the address of a pointer: what a pointer to any memory becomes in LDS depends on
    // whether it is null, and where the compiler does not see through that, the address is no constant and each look-up adds it to
    // its index: 190 instead of 172 instructions a round of bytes at 64 sub-streams, 219 instead of 200 of tANS at 256.
    const uint32_t tbl_addr = lds_address(lds_all) + 4 * kFrontWords + 2 * kTableEntries * sub;
    const uint32_t ring_lane = lds_address(lds_all + wave * kRingStride + lane);
    constexpr bool UNI = CPW == 1; // all lanes of the wave belong to one stream set

    // ---- products of whole rows: the rows of the chunk, and what lane r of the chunk's first wave does with the sum of
    // the r-th.  Its scale is asked for now: at the end the trip to memory would be one that nothing hides.  (Not by a wave alone with its
    // chunk, which has nothing that hides it now either: asked for at the end 4096 chunks of a row of 4 KiB at 64 sub-streams take 12.2 instead of 12.7
    // us, longer chunks the same.  At 32 sub-streams, two chunks to a wave, the end is 2 to 3 % slower.)
    constexpr bool kRows = MODE == kModeGemvRows || MODE == kModeGemvW8A8Rows;
    const uint32_t own_row = kRows ? (uint32_t)(dst_pos / mat.cols) + cl : 0u;
    const bool has_row = kRows && k < a.n_chunks && wave == 0 && cl < a.chunk_bytes / mat.cols && own_row < mat.rows;
    float own_scale = 0.0f;
    constexpr bool kScaleNow = S != 64;
    if (kScaleNow && has_row) own_scale = mat.row_scale[own_row];
    auto finish_rows = [&](auto sum) {
        if (has_row) store_row(mat, own_row, scaled_sum(mat, kScaleNow ? own_scale : mat.row_scale[own_row], decltype(sum)(0) + sum));
    };
    // ---- ordered product: the same for the sums that the chunk leaves in the workspace.  One for every row that the chunk's
    // place in the matrix touches, whatever its table entry says, because the finish kernel adds them all up.
    auto leave_partial_sums = [&](float sum) {
        if constexpr (MODE != kModeI8) {
            const uint64_t end = dst_pos + a.chunk_bytes < dst_cap ? dst_pos + a.chunk_bytes : dst_cap;
            if (k < a.n_chunks && wave == 0 && cl <= (uint32_t)((end - 1) / mat.cols) - (uint32_t)(dst_pos / mat.cols))
                a.partial[k * kPartialSlots + cl] = sum;
        }
    };
    // A chunk that is not decoded leaves empty sums, or their results.
    auto finish_empty = [&]() {
        if (MODE == kModeGemv || MODE == kModeGemvRows) leave_partial_sums(0.0f);
        if (MODE == kModeGemvRows) finish_rows(0.0f);
        if (MODE == kModeGemvW8A8Rows) finish_rows((int32_t)0);
    };

    // ---- raw chunks: the threads of the chunk copy it, eight 16-byte loads in flight per thread
    if (MODE == kModeI8 && CPW == 2) {
        // S = 32: the wavefront's two chunks one after the other, each copied by all 64 lanes with sixteen loads in
        // flight per lane (a wavefront alone on its SIMD has nothing but its own loads to hide a trip to memory behind)
        for (uint32_t h = 0; h < 2; h++) {
            const int from = 32 * (int)h;
            if (!__shfl((int)(active && is_raw), from)) continue;
            const uint64_t off_h = (uint64_t)(uint32_t)__shfl((int)(uint32_t)ent.off, from) |
                                   (uint64_t)(uint32_t)__shfl((int)(uint32_t)(ent.off >> 32), from) << 32;
            const uint32_t raw_h = (uint32_t)__shfl((int)raw, from);
            const uint8_t *p8 = a.blob + off_h;
            uint8_t *d8 = static_cast<uint8_t *>(a.dst) + ((uint64_t)blockIdx.x * CPW + h) * (uint64_t)a.chunk_bytes;
            const uint32_t n16 = raw_h / 16;
            for (uint32_t base = lane; base < n16; base += 16 * 64) {
                u32x4 v[16];
#pragma unroll
                for (int j = 0; j < 16; j++)
                    if (base + j * 64 < n16) v[j] = load16_stream(p8 + 16 * (size_t)(base + j * 64));
#pragma unroll
                for (int j = 0; j < 16; j++)
                    if (base + j * 64 < n16)
                        __builtin_nontemporal_store(v[j], reinterpret_cast<u32x4 *>(d8 + 16 * (size_t)(base + j * 64)));
            }
            for (uint32_t i = n16 * 16 + lane; i < raw_h; i += 64) d8[i] = p8[i];
        }
    } else if (MODE == kModeI8 && active && is_raw) {
        uint8_t *d8 = static_cast<uint8_t *>(a.dst) + dst_pos;
        const uint32_t n16 = raw / 16;
        for (uint32_t base = ct; base < n16; base += 8 * TPC) {
            u32x4 v[8];
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (base + j * TPC < n16) v[j] = load16_stream(payload8 + 16 * (size_t)(base + j * TPC));
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (base + j * TPC < n16)
                    __builtin_nontemporal_store(v[j], reinterpret_cast<u32x4 *>(d8 + 16 * (size_t)(base + j * TPC)));
        }
        for (uint32_t i = n16 * 16 + ct; i < raw; i += TPC) d8[i] = payload8[i];
    }
    if (MODE != kModeI8 && !active) {
        finish_empty();
        return;
    }
    if (MODE == kModeI8 && !huff) {
        leave_record(active ? DC_TRACE_COPIED : DC_TRACE_SKIPPED);
        return;
    }

    // The table is only needed where a chunk of the workgroup is Huffman coded; the condition is the
    // same for every thread that is still here, so the barriers inside are reached together.
    // ---- the code lengths of the header are asked for first, so that they travel while the sub-streams are set up
    uint32_t nib_word = 0;
    if (CODEC == DC_CODEC_HUFFMAN && huff) {
        if (SPL == 8) nib_word = payload[ct];
        else if (SPL == 4) nib_word = reinterpret_cast<const uint16_t *>(payload8)[ct];
        else if (SPL == 2) nib_word = payload8[ct];
        else nib_word = payload8[ct >> 1];
    }

    // ---- sub-stream set-up, first half: the loads (all lanes of a stream set are here together or not at all)
    Region rg;
    Stream st;
    StreamFetch sf;
    if (huff) {
        rg.payload8 = payload8;
        // a 20-byte load may begin in the last bytes of the payload; the blob goes on for DC_BLOB_TAIL_BYTES
        const uint64_t room = a.blob_bytes - ent.off - 20;
        rg.max_off = room < 0xFFFFFFE0ull ? (uint32_t)room : 0xFFFFFFE0u;
        rg.lanes = CPW == 1 ? ~0ull : (sub ? 0xFFFFFFFF00000000ull : 0x00000000FFFFFFFFull);
        rg.next_block = payload[(kFront + 2 * S) / 4 + (CPW == 1 ? wave : 0)] / kBlockBytes;
        if (UNI) rg.next_block = __builtin_amdgcn_readfirstlane(rg.next_block);
        stream_fetch<UNI>(st, rg, reinterpret_cast<const uint16_t *>(payload8)[kFront / 2 + ct], sf);
    }

    const bool build_table = CODEC == DC_CODEC_TANS ? false : CPW == 1 ? huff : (bool)__any(huff);
    if (CODEC == DC_CODEC_TANS && huff) { // (one chunk per workgroup: the same for all of its threads)
        uint32_t *cumq = lds_all + kFrontWords + kTableEntries;
        if (!build_tans_table<S>(payload8, ct, lane, wave, lds_all, tbl_addr, cumq, cumq + 256)) {
            finish_empty();
            return;
        }
    }

    if (build_table) {
        uint32_t *marks = lds_all + sub * kTableEntries;
        constexpr bool SHARED = kFrontWords < CPW * kTableEntries;
        static_assert(!SHARED || (WAVES == 1 && kFrontWords + kTableWords >= CPW * kTableEntries), "room for the marks");
        build_code_table<TPC, WAVES, CPW == 2, SHARED>(SPL == 1 ? (nib_word >> (4 * (ct & 1))) & 15u : nib_word, ct, wave, marks, lds_counts, tbl_addr);
    }

    // ---- sub-stream set-up, second half: the ring is free now
    if (huff) stream_start<CODEC, S, ORDER>(st, sf, ring_lane, tbl_addr);

    const uint32_t round_bytes = 16 * S;
    const uint32_t full_rounds = raw / round_bytes;
    const uint32_t rem = raw - full_rounds * round_bytes;

    if (MODE == kModeI8) {
        uint8_t *d8 = static_cast<uint8_t *>(a.dst) + dst_pos + ct * 16;
        for (uint32_t r = 0; r < full_rounds; r++) {
            uint32_t w[4];
            decode16<S, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, w);
            store16_stream(d8 + (size_t)r * round_bytes, w[0], w[1], w[2], w[3]);
        }
        if (rem) {
            // last, partial round: lanes hold 16, fewer (one lane of the chunk) or no symbols
            const uint32_t start = ct * 16;
            const uint32_t n = rem > start ? (rem - start < 16 ? rem - start : 16) : 0;
            uint8_t *d = d8 + (size_t)full_rounds * round_bytes;
            uint32_t w[4];
            decode16<S, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, w);
            if (n == 16) {
                store16_stream(d, w[0], w[1], w[2], w[3]);
            } else if (n) {
#pragma unroll
                for (uint32_t i = 0; i < 15; i++)
                    if (i < n) d[i] = (uint8_t)(w[i / 4] >> (8 * (i % 4)));
            }
        }
        leave_record(DC_TRACE_DECODED);
        return;
    }

    // ---- fused consumers walk the matrix: group position -> (row, column)
    const uint32_t cols = mat.cols, mat_rows = mat.rows;
    const uint32_t rounds = full_rounds + (rem ? 1 : 0);
    uint64_t pos = dst_pos + ct * 16;
    uint32_t row = (uint32_t)(pos / cols);
    uint32_t col = (uint32_t)(pos - (uint64_t)row * cols);

    if (MODE == kModeBf16) {
        // A lane's 16 values become 32 bytes, so two 16-byte stores of its own values would each
        // write half of every 128-byte line.  Lanes l and l + 16 (the same chunk) trade eight bytes
        // first: afterwards the first store of the wave covers the groups of lanes 0-15 and 32-47
        // completely and the second store those of lanes 16-31 and 48-63, whole lines both.
        //   lane l     (bit 4 clear): w0 w1 = its bytes 0-7,          w2 w3 = bytes 0-7 of lane l + 16
        //   lane l + 16             : w0 w1 = bytes 8-15 of lane l,   w2 w3 = its bytes 8-15
        uint16_t *out = static_cast<uint16_t *>(mat.dst);
        const uint32_t upper = (ct >> 4) & 1u;
        const uint32_t ct_a = ct & ~16u, ct_b = ct_a + 16; // the groups the first and the second store belong to
        const uint64_t pos_a = dst_pos + ct_a * 16, pos_b = dst_pos + ct_b * 16;
        uint32_t row_a = (uint32_t)(pos_a / cols), row_b = (uint32_t)(pos_b / cols);
        uint32_t col_a = (uint32_t)(pos_a - (uint64_t)row_a * cols), col_b = (uint32_t)(pos_b - (uint64_t)row_b * cols);
        auto scale_of = [&](uint32_t row) { return mat.row_scale[row < mat.rows ? row : 0]; };
        auto next_round = [&]() {
            col_a += round_bytes;
            while (col_a >= cols) { col_a -= cols; row_a++; }
            col_b += round_bytes;
            while (col_b >= cols) { col_b -= cols; row_b++; }
        };
        // the 16 values of a round, traded between the lanes, scaled and stored (has_a, has_b: whether the two groups exist)
        auto convert_and_store = [&](const uint32_t w[4], float s_a, float s_b, uint32_t r, bool has_a, bool has_b) {
            // rows of 16 lanes: the odd rows of the first operand change places with the even rows of the second
            const auto x02 = __builtin_amdgcn_permlane16_swap(w[0], w[2], false, false);
            const auto x13 = __builtin_amdgcn_permlane16_swap(w[1], w[3], false, false);
            const uint32_t wa[2] = {x02[0], x13[0]}, wb[2] = {x02[1], x13[1]};
            const uint32_t base = r * round_bytes;
            if (has_a) {
                float f[8];
                word_to_scaled_f32(wa[0], s_a, f);
                word_to_scaled_f32(wa[1], s_a, f + 4);
                store16_stream(out + (pos_a + base + 8 * upper), bf16x2(f[0], f[1]), bf16x2(f[2], f[3]), bf16x2(f[4], f[5]),
                               bf16x2(f[6], f[7]));
            }
            if (has_b) {
                float f[8];
                word_to_scaled_f32(wb[0], s_b, f);
                word_to_scaled_f32(wb[1], s_b, f + 4);
                store16_stream(out + (pos_b + base + 8 * upper), bf16x2(f[0], f[1]), bf16x2(f[2], f[3]), bf16x2(f[4], f[5]),
                               bf16x2(f[6], f[7]));
            }
        };
        if (!huff) {
            // raw chunk: the bytes come straight from the payload
            for (uint32_t r = 0; r < rounds; r++) {
                const uint32_t start = r * round_bytes + ct * 16;
                // the matrix size is a multiple of 16, so a group is whole or absent
                const bool whole = raw >= start + 16;
                const float s_a = scale_of(row_a), s_b = scale_of(row_b);
                uint32_t w[4] = {0, 0, 0, 0};
                if (whole) {
                    const u32x4 v = load16_stream(payload8 + start);
                    w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
                }
                const uint32_t base = r * round_bytes;
                convert_and_store(w, s_a, s_b, r, raw >= base + ct_a * 16 + 16, raw >= base + ct_b * 16 + 16);
                next_round();
            }
            return;
        }
        // Coded chunk.  In the whole rounds every memory access is issued by every lane on every path, in a fixed
        // order (block, block, store, store, scale, scale), so that the wait before a block goes into the ring
        // can count exactly how many younger accesses may stay in flight, the stores among them; the scales of a
        // round are asked for at the end of the round before.
        float s_a = scale_of(row_a), s_b = scale_of(row_b);
        for (uint32_t r = 0; r < full_rounds; r++) {
            uint32_t w[4];
            decode16<S, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, w);
            convert_and_store(w, s_a, s_b, r, true, true);
            next_round();
            s_a = scale_of(row_a);
            s_b = scale_of(row_b);
        }
        if (rem) {
            const uint32_t base = full_rounds * round_bytes;
            uint32_t w[4] = {0, 0, 0, 0};
            decode16<S, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, w);
            convert_and_store(w, s_a, s_b, full_rounds, raw >= base + ct_a * 16 + 16, raw >= base + ct_b * 16 + 16);
        }
        return;
    }

    // The rounds of a raw chunk, four loads of weights in flight: step(whole, its 16 bytes) for every round.
    auto raw_rounds = [&](bool last_whole, auto step) {
        const uint8_t *p = payload8 + ct * 16;
        uint32_t r = 0;
        for (; r + 4 <= full_rounds; r += 4) {
            u32x4 v[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; j++) v[j] = load16_stream(p + (r + j) * round_bytes);
#pragma unroll
            for (uint32_t j = 0; j < 4; j++) step(true, v[j]);
        }
        for (; r < full_rounds; r++) step(true, load16_stream(p + r * round_bytes));
        if (rem) step(last_whole, last_whole ? load16_stream(p + r * round_bytes) : u32x4{0, 0, 0, 0});
    };

    // The coded rounds where the 1024 bytes that a wave decodes in a round never lie in two rows: the wave moves to another row with all
    // of its lanes, so that a round needs no look at the lanes' rows, and a row's end no sorting of them.  The additions are the
    // general walk's, in its order.  13B layer (rows of 5 * 1024 and 13.5 * 1024) 101.5 -> 99.7 us; 4096 columns, 1024 chunks at 256 sub-streams
    // 28.6 -> 27.2, int8 26.5 -> 25.1.  Launches of few wavefronts only take it where rows are whole rounds, which is counted with less (at 64
    // sub-streams 51.6 -> 47.1 and 48.2 -> 45.9; 2 % of it lost with the walk for any rows).
    constexpr uint32_t kSpan = 16 * 64;
    const uint32_t unit = FEW ? round_bytes : kSpan;
    const bool rows_of_spans = (kRows || MODE == kModeGemv) && UNI && huff && cols % unit == 0 && dst_pos % (FEW ? cols : kSpan) == 0 &&
                               raw % (FEW ? cols : kSpan) == 0;
    auto sum_rows_of_spans = [&](auto &mine, auto &acc, uint32_t &col, uint32_t first_row, bool last_whole, auto coded_round) {
        using T = std::remove_reference_t<decltype(acc)>;
        auto end_row = [&](uint32_t slot) {
            const T v = __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lanes_sum(acc)), 63));
            mine += lane == (slot & 63u) ? v : T(0);
            acc = T(0);
        };
        if constexpr (FEW) {
            uint32_t slot = 0, left = cols / round_bytes;
            for (uint32_t r = 0; r < full_rounds; r++)
                coded_round(true, [&]() {
                    if (left == 0) {
                        end_row(slot++);
                        left = cols / round_bytes;
                    }
                    left--;
                    col = left ? col + round_bytes : ct * 16;
                });
            end_row(slot);
        } else {
            uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)col), next_row = (uint32_t)__builtin_amdgcn_readfirstlane((int)row);
            uint32_t cur = next_row;
            uint32_t whole_rows = 0, part = round_bytes; // a round takes the wave this far
            for (; part >= cols; part -= cols) whole_rows++;
            auto enter = [&]() {
                if (next_row != cur) {
                    end_row(cur - first_row);
                    cur = next_row;
                }
                at += part;
                next_row += whole_rows + (at >= cols ? 1u : 0u);
                at -= at >= cols ? cols : 0u;
                col = at + 16 * lane;
            };
            for (uint32_t r = 0; r < full_rounds; r++) coded_round(true, enter);
            if (rem && (bool)__builtin_amdgcn_readfirstlane((int)last_whole)) coded_round(true, enter);
            end_row(cur - first_row);
        }
    };

    // Sums over the waves of the chunk, in wave order, for its first wave.  A wave's ring is its own, and the wave has read
    // the last of it: the totals go there.
    auto over_waves = [&](auto mine) {
        using T = decltype(mine);
        T total = mine;
        if (WAVES > 1) {
            lds_all[wave * kRingStride + lane] = __builtin_bit_cast(uint32_t, mine);
            __syncthreads();
            if (wave == 0) {
                total = T(0);
#pragma unroll
                for (int v = 0; v < WAVES; v++) total += __builtin_bit_cast(T, lds_all[v * kRingStride + lane]);
            }
        }
        return total;
    };

    if (MODE == kModeGemv || MODE == kModeGemvAtomic || MODE == kModeGemvRows) {
        // Partial dot products of the int8 values with x; the row scale is applied once per row by the finish
        // kernel.  A lane keeps the sum of its groups of one row; when some lane of the wave moves to another
        // row, the wave sums its lanes by row.  kModeGemvAtomic: one atomic on y per row the wave holds.
        // Else the sum of the r-th row the chunk touches goes to lane r of the wave (of the chunk's half
        // of it when S = 32), which keeps the wave's total for that row; at the end the waves' totals are
        // added in wave order through LDS and the chunk leaves one sum per row in the workspace.  Every
        // addition then has a fixed place in a fixed order, so the result is the same bits at every run.
        const uint32_t first_row = (uint32_t)(dst_pos / cols);
        const uint16_t *x = mat.x_bf16;
        in_register<UNI>(mat_rows);
        in_register<UNI>(cols);
        in_register<UNI>(x);
        float mine = 0.0f; // this wave's sum for row first_row + cl
        uint32_t cur_row = 0xFFFFFFFFu;
        float acc = 0.0f;
        auto flush = [&]() {
            const uint32_t key = cur_row < mat_rows ? cur_row : 0xFFFFFFFFu;
            if (MODE == kModeGemvAtomic) lanes_add_by_key<CPW == 2, float>(mat.y_accum, key, acc);
            else lanes_add_runs_to_slots<CPW == 2, float>(mine, key, (cur_row - first_row) % LPC + sub * LPC, acc);
            acc = 0.0f;
            cur_row = 0xFFFFFFFFu;
        };
        // An int8 value is a bf16 value exactly: two of them packed, times two values of x as they lie in memory, in one
        // instruction (products exact in fp32, summed in fp32).  The values come straight out of byte 1 of their table
        // entries, without being packed to bytes first, and x is asked for before the group is decoded.
        // Coded and raw chunks have loops of their own: in a loop that can load weights on one path, the compiler waits for
        // every load before it uses the weights, the blocks asked for a moment ago among them (product of 1024 chunks at 64
        // sub-streams, a wavefront a SIMD: 64.4 -> 59.5 us, int8 73.1 -> 56.2; 13B layer at 256: 104.7 -> 101.7; with the
        // single launch where that applies).
        auto enter_row = [&](bool whole) {
            if (__any(whole && row != cur_row && cur_row != 0xFFFFFFFFu)) flush();
            cur_row = whole ? row : cur_row;
            // on to the next round at once: a loop behind the products would keep the first half's from being
            // carried out between the second half's look-ups
            col += round_bytes;
            while (col >= cols) { col -= cols; row++; }
        };
        struct Sixteen { uint32_t x[8]; };
        auto load_x = [&]() -> Sixteen {
            const uint4 *xp = reinterpret_cast<const uint4 *>(x + col); // col + 16 <= cols, group or not
            const uint4 xa = xp[0], xb = xp[1];
            return {{xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w}};
        };
        auto coded_round = [&](bool whole, auto enter) {
            Sixteen xs;
            uint32_t e[8];
            auto products = [&](const uint32_t e[8], uint32_t half, int from, int to) {
                if (whole)
#pragma unroll
                    for (int i = from; i < to; i++)
                        acc = dot2_bf16(bf16x2(byte_f32<1>(e[2 * i]), byte_f32<1>(e[2 * i + 1])), xs.x[4 * half + i], acc);
                if (FEW) in_register<false>(acc);
            };
            auto begin = [&]() {
                xs = load_x();
                enter();
            };
            if constexpr (FEW) {
                uint32_t f[8];
                step_and_decode8<S, 0, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, e, early(begin));
                step_and_decode8<S, 1, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, f, late([&](int i) { products(e, 0, 2 * i, 2 * i + 2); }));
                products(f, 1, 0, 4);
            } else {
                begin();
                step_and_decode8<S, 0, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, e);
                products(e, 0, 0, 4);
                step_and_decode8<S, 1, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, e);
                products(e, 1, 0, 4);
            }
        };
        auto raw_round = [&](bool whole, const u32x4 &w) {
            const Sixteen xs = load_x();
            enter_row(whole);
            if (whole)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    acc = dot2_bf16(bf16x2(byte_f32<0>(w[i]), byte_f32<1>(w[i])), xs.x[2 * i], acc);
                    acc = dot2_bf16(bf16x2(byte_f32<2>(w[i]), byte_f32<3>(w[i])), xs.x[2 * i + 1], acc);
                }
        };
        const bool last_whole = raw >= full_rounds * round_bytes + ct * 16 + 16;
        if (rows_of_spans) {
            sum_rows_of_spans(mine, acc, col, first_row, last_whole, coded_round);
        } else {
            if (huff) {
                for (uint32_t r = 0; r < full_rounds; r++) coded_round(true, [&]() { enter_row(true); });
                if (rem) coded_round(last_whole, [&]() { enter_row(last_whole); });
            } else {
                raw_rounds(last_whole, raw_round);
            }
            flush();
        }
        if (MODE != kModeGemvAtomic) {
            const float total = over_waves(mine);
            leave_partial_sums(total);
            if (MODE == kModeGemvRows) finish_rows(total);
        }
    }

    if (MODE == kModeGemvW8A8 || MODE == kModeGemvW8A8Rows) {
        // The same walk with int8 activations (Eq. 4 of the paper): four v_dot4 per group, exact int32
        // sums, integer atomics (or the lanes' slots, see above), so the result does not depend on the order of the additions.
        const uint32_t first_row = (uint32_t)(dst_pos / cols);
        const int8_t *x = mat.x_i8;
        in_register<UNI>(mat_rows);
        in_register<UNI>(cols);
        in_register<UNI>(x);
        int32_t mine = 0;
        uint32_t cur_row = 0xFFFFFFFFu;
        int32_t acc = 0;
        auto flush = [&]() {
            const uint32_t key = cur_row < mat_rows ? cur_row : 0xFFFFFFFFu;
            if (MODE == kModeGemvW8A8) lanes_add_by_key<CPW == 2, int32_t>(reinterpret_cast<int32_t *>(mat.y_accum), key, acc);
            else lanes_add_runs_to_slots<CPW == 2, int32_t>(mine, key, (cur_row - first_row) % LPC + sub * LPC, acc);
            acc = 0;
            cur_row = 0xFFFFFFFFu;
        };
        auto add_products = [&](bool whole, const uint32_t w[4], const uint4 &x) {
            if (whole) {
                acc = __builtin_amdgcn_sdot4((int)w[0], (int)x.x, acc, false);
                acc = __builtin_amdgcn_sdot4((int)w[1], (int)x.y, acc, false);
                acc = __builtin_amdgcn_sdot4((int)w[2], (int)x.z, acc, false);
                acc = __builtin_amdgcn_sdot4((int)w[3], (int)x.w, acc, false);
            }
        };
        auto load_x = [&]() { return *reinterpret_cast<const uint4 *>(x + col); };
        auto enter_row = [&](bool whole) {
            if (__any(whole && row != cur_row && cur_row != 0xFFFFFFFFu)) flush();
            cur_row = whole ? row : cur_row;
            col += round_bytes;
            while (col >= cols) { col -= cols; row++; }
        };
        auto coded_round = [&](bool whole, auto enter) {
            uint4 xs;
            uint32_t w[4];
            auto begin = [&]() {
                xs = load_x(); // asked for before the group is decoded
                enter();
            };
            if constexpr (FEW) {
                decode16<S, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, w, early(begin));
            } else {
                begin();
                decode16<S, CODEC, ORDER>(st, rg, tbl_addr, ring_lane, w);
            }
            add_products(whole, w, xs);
        };
        auto raw_round = [&](bool whole, const u32x4 &v) {
            const uint4 xs = load_x();
            enter_row(whole);
            const uint32_t w[4] = {v[0], v[1], v[2], v[3]};
            add_products(whole, w, xs);
        };
        const bool last_whole = raw >= full_rounds * round_bytes + ct * 16 + 16;
        if (rows_of_spans) {
            sum_rows_of_spans(mine, acc, col, first_row, last_whole, coded_round);
        } else {
            if (huff) {
                for (uint32_t r = 0; r < full_rounds; r++) coded_round(true, [&]() { enter_row(true); });
                if (rem) coded_round(last_whole, [&]() { enter_row(last_whole); });
            } else {
                raw_rounds(last_whole, raw_round);
            }
            flush();
        }
        if (MODE == kModeGemvW8A8Rows) finish_rows(over_waves(mine));
    }
}

// Blocks of 256 rows of the matrices of a fused GEMV call, matrix after matrix.
struct RowBlocks {
    uint32_t chunk_bytes;
    const float *partial; // the ordered product: kPartialSlots sums per chunk
    uint32_t first_block[DC_MAX_MATRICES]; // no block's number beyond the last matrix
    MatrixArgs mats[DC_MAX_MATRICES];
};
__device__ __forceinline__ uint32_t matrix_of_block(const RowBlocks &rb, uint32_t block)
{
    uint32_t mi = 0;
#pragma unroll
    for (uint32_t i = 1; i < DC_MAX_MATRICES; i++) mi += block >= rb.first_block[i] ? 1u : 0u;
    return mi;
}

__global__ __launch_bounds__(256) void dc_gemv_zero_kernel(RowBlocks rb)
{
    const uint32_t mi = matrix_of_block(rb, blockIdx.x);
    const uint32_t i = (blockIdx.x - rb.first_block[mi]) * 256 + threadIdx.x;
    if (i < rb.mats[mi].rows) rb.mats[mi].y_accum[i] = 0.0f;
}

template <bool W8A8> __global__ __launch_bounds__(256) void dc_gemv_finish_kernel(RowBlocks rb)
{
    const uint32_t mi = matrix_of_block(rb, blockIdx.x);
    const MatrixArgs &m = rb.mats[mi];
    const uint32_t i = (blockIdx.x - rb.first_block[mi]) * 256 + threadIdx.x;
    if (i < m.rows) {
        const float scale = m.row_scale[i];
        if (W8A8) store_row(m, i, scaled_sum(m, scale, reinterpret_cast<const int32_t *>(m.y_accum)[i]));
        else store_row(m, i, scaled_sum(m, scale, m.y_accum[i]));
    }
}

// The ordered product: y_i = scale_i * (sum over the chunks that hold a part of row i, in chunk order, of the
// chunk's sum for the row).  Chunk c of a matrix holds bytes [c*C, c*C + C) of it and keeps the sum of the r-th
// row it touches, row (c*C) div cols + r, in slot r.
__global__ __launch_bounds__(256) void dc_gemv_ordered_finish_kernel(RowBlocks rb)
{
    const uint32_t mi = matrix_of_block(rb, blockIdx.x);
    const MatrixArgs &m = rb.mats[mi];
    const uint32_t i = (blockIdx.x - rb.first_block[mi]) * 256 + threadIdx.x;
    if (i < m.rows) {
        const float scale = m.row_scale[i]; // on its way while the sums are found
        const uint64_t C = rb.chunk_bytes;
        const uint64_t begin = (uint64_t)i * m.cols, last = begin + m.cols - 1;
        const uint64_t c0 = begin / C, c1 = last / C;
        const float *p = rb.partial + (m.first_chunk + c0) * kPartialSlots;
        // chunks after the first begin inside the row: it is the first that they touch.  Two sums are asked for at once.
        const float next = c1 > c0 ? p[kPartialSlots] : 0.0f;
        float sum = p[i - (uint32_t)(c0 * C / m.cols)];
        if (c1 > c0) sum += next;
        for (uint64_t c = c0 + 2; c <= c1; c++) sum += p[(c - c0) * kPartialSlots];
        store_row(m, i, scaled_sum(m, scale, sum));
    }
}

// Batch-1 product on weights that are already decoded: y_i = scale_i * sum_j q_ij x_j, q int8 row-major.
// A workgroup owns kGemvRows consecutive rows; its 256 threads walk the columns 16 bytes a thread
// (4 KiB a workgroup and row), so that x is converted once for all the rows; a weight costs one
// conversion (sign-extending byte select) and one fused multiply-add.
// Bound by latency: rows of more than 4 KiB take several turns, and a turn's loads are issued before the products of the turn
// before (4096 x 11008: 9.9 -> 9.3 us; rows of one turn as before).  Two or eight rows a workgroup: 3 to 30 % slower.
constexpr int kGemvRows = 4;
__global__ __launch_bounds__(256) void dc_gemv_i8_kernel(const uint8_t *__restrict__ q, const float *__restrict__ row_scale,
                                                         uint32_t rows, uint32_t cols, const uint16_t *__restrict__ x_bf16,
                                                         float *__restrict__ y_f32, uint16_t *__restrict__ y_bf16)
{
    __shared__ float part[4][kGemvRows];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t row0 = blockIdx.x * kGemvRows;
    const uint8_t *qr[kGemvRows];
#pragma unroll
    for (int r = 0; r < kGemvRows; r++) {
        const uint32_t row = row0 + r < rows ? row0 + r : rows - 1; // rows past the end repeat the last one
        qr[r] = q + (size_t)row * cols;
    }
    const float scale = row_scale[row0 + (threadIdx.x & 3u) < rows ? row0 + (threadIdx.x & 3u) : row0]; // for the end, where nothing would hide its trip
    float acc[kGemvRows] = {0.0f, 0.0f, 0.0f, 0.0f};
    struct Turn { u32x4 w[kGemvRows]; uint4 xa, xb; };
    auto load = [&](uint32_t c) -> Turn {
        Turn t;
#pragma unroll
        for (int r = 0; r < kGemvRows; r++) t.w[r] = load16_stream(qr[r] + c);
        const uint4 *xp = reinterpret_cast<const uint4 *>(x_bf16 + c);
        t.xa = xp[0];
        t.xb = xp[1];
        return t;
    };
    auto add = [&](const Turn &t) {
        const u32x4 *w = t.w;
        const uint4 xa = t.xa, xb = t.xb;
        const uint32_t xs[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
        float xf[16];
#pragma unroll
        for (int i = 0; i < 8; i++) {
            xf[2 * i] = bf16_bits_to_f32(xs[i] & 0xFFFFu);
            xf[2 * i + 1] = __uint_as_float(xs[i] & 0xFFFF0000u);
        }
#pragma unroll
        for (int r = 0; r < kGemvRows; r++) {
#pragma unroll
            for (int i = 0; i < 4; i++) {
                acc[r] = __builtin_fmaf(byte_f32<0>(w[r][i]), xf[4 * i], acc[r]);
                acc[r] = __builtin_fmaf(byte_f32<1>(w[r][i]), xf[4 * i + 1], acc[r]);
                acc[r] = __builtin_fmaf(byte_f32<2>(w[r][i]), xf[4 * i + 2], acc[r]);
                acc[r] = __builtin_fmaf(byte_f32<3>(w[r][i]), xf[4 * i + 3], acc[r]);
            }
        }
    };
    uint32_t c = threadIdx.x * 16;
    if (c < cols) {
        Turn now = load(c);
        for (c += 4096; c < cols; c += 4096) { // the next turn's loads run while this one's products are formed
            const Turn next = load(c);
            add(now);
            now = next;
        }
        add(now);
    }
    in_register<false>(scale);
#pragma unroll
    for (int r = 0; r < kGemvRows; r++) acc[r] = lanes_sum(acc[r]);
    if (lane == 63) {
#pragma unroll
        for (int r = 0; r < kGemvRows; r++) part[wave][r] = acc[r];
    }
    __syncthreads();
    if (threadIdx.x < kGemvRows && row0 + threadIdx.x < rows) {
        const uint32_t r = threadIdx.x;
        const float total = part[0][r] + part[1][r] + part[2][r] + part[3][r];
        const float y = scale * total;
        y_f32[row0 + r] = y;
        if (y_bf16) y_bf16[row0 + r] = (uint16_t)(bf16x2(y, 0.0f) & 0xFFFFu);
    }
}

// The same product with int8 activations (Eq. 4): y_i = (float(sum_j q_ij xq_j) * scale_i) * x_scale.
// Same decomposition; four v_dot4 per 16 weights, exact int32 sums.
__global__ __launch_bounds__(256) void dc_gemv_w8a8_kernel(const uint8_t *__restrict__ q, const float *__restrict__ row_scale,
                                                           uint32_t rows, uint32_t cols, const int8_t *__restrict__ x_i8,
                                                           float x_scale, float *__restrict__ y_f32,
                                                           uint16_t *__restrict__ y_bf16)
{
    __shared__ int32_t part[4][kGemvRows];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t row0 = blockIdx.x * kGemvRows;
    const uint8_t *qr[kGemvRows];
#pragma unroll
    for (int r = 0; r < kGemvRows; r++) {
        const uint32_t row = row0 + r < rows ? row0 + r : rows - 1; // rows past the end repeat the last one
        qr[r] = q + (size_t)row * cols;
    }
    const float scale = row_scale[row0 + (threadIdx.x & 3u) < rows ? row0 + (threadIdx.x & 3u) : row0]; // for the end, where nothing would hide its trip
    int32_t acc[kGemvRows] = {0, 0, 0, 0};
    struct Turn { u32x4 w[kGemvRows]; uint4 x; };
    auto load = [&](uint32_t c) -> Turn {
        Turn t;
#pragma unroll
        for (int r = 0; r < kGemvRows; r++) t.w[r] = load16_stream(qr[r] + c);
        t.x = *reinterpret_cast<const uint4 *>(x_i8 + c);
        return t;
    };
    auto add = [&](const Turn &t) {
        const uint32_t xs[4] = {t.x.x, t.x.y, t.x.z, t.x.w};
#pragma unroll
        for (int r = 0; r < kGemvRows; r++)
#pragma unroll
            for (int i = 0; i < 4; i++) acc[r] = __builtin_amdgcn_sdot4((int)t.w[r][i], (int)xs[i], acc[r], false);
    };
    uint32_t c = threadIdx.x * 16;
    if (c < cols) {
        Turn now = load(c);
        for (c += 4096; c < cols; c += 4096) { // the next turn's loads run while this one's products are formed (see above)
            const Turn next = load(c);
            add(now);
            now = next;
        }
        add(now);
    }
    in_register<false>(scale);
#pragma unroll
    for (int r = 0; r < kGemvRows; r++)
        acc[r] = __builtin_bit_cast(int32_t, lanes_prefix_sum<false>(__builtin_bit_cast(uint32_t, acc[r]))); // total in lane 63
    if (lane == 63) {
#pragma unroll
        for (int r = 0; r < kGemvRows; r++) part[wave][r] = acc[r];
    }
    __syncthreads();
    if (threadIdx.x < kGemvRows && row0 + threadIdx.x < rows) {
        const uint32_t r = threadIdx.x;
        const int32_t total = part[0][r] + part[1][r] + part[2][r] + part[3][r];
        const float y = ((float)total * scale) * x_scale;
        y_f32[row0 + r] = y;
        if (y_bf16) y_bf16[row0 + r] = (uint16_t)(bf16x2(y, 0.0f) & 0xFFFFu);
    }
}

__global__ __launch_bounds__(256) void dc_copy_kernel(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, uint64_t n16)
{
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

thread_local hipError_t g_last_hip_error = hipSuccess;

int launch_status() { return dc_launch_status(); }

// Kernel arguments every decode launch shares; the trailer is what a blob of these parameters ends with.
void common_args(BytesArgs &a, const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev, uint64_t n_chunks,
                 const dc_params *p)
{
    a.blob = blob_dev;
    a.blob_bytes = blob_bytes;
    a.table = table_dev;
    a.n_chunks = n_chunks;
    a.chunk_bytes = p->chunk_bytes;
    a.trailer[0] = DC_TRAILER_MAGIC;
    a.trailer[1] = DC_FORMAT_ID | (uint32_t)DC_LOOKAHEAD_BITS << 16;
    a.trailer[2] = p->chunk_bytes;
    a.trailer[3] = p->n_streams | p->codec << 16;
}

bool decode_params_ok(const dc_params *p)
{
    if (!p) return false;
    if (p->chunk_bytes < 16 || p->chunk_bytes > DC_MAX_CHUNK_BYTES || p->chunk_bytes % 16) return false;
    if (p->codec == DC_CODEC_TANS) return p->n_streams == 64 || p->n_streams == 128 || p->n_streams == 256;
    if (p->codec != DC_CODEC_HUFFMAN) return false;
    return p->n_streams == 32 || p->n_streams == 64 || p->n_streams == 128 || p->n_streams == 256;
}

// SIMDs of the current device, four to a compute unit, looked up once per device; 0 if the runtime does not say, which is no error of the call.
uint32_t device_simds()
{
    static std::atomic<uint32_t> simds_of_device[kMaxDevices];
    int dev = -1, units = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices) {
        uint32_t n = simds_of_device[dev].load(std::memory_order_relaxed);
        if (n) return n;
        if (hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && units > 0) {
            n = 4u * (uint32_t)units;
            simds_of_device[dev].store(n, std::memory_order_relaxed);
            return n;
        }
    }
    (void)hipGetLastError(); // not to be taken for the launch's
    return 0;
}

// The order of a decoder's work in a launch of `waves` wavefronts.
// For few of them: up to one a SIMD a launch is as long as a lane's chain of look-ups, and these kernels are up to 19 % shorter, the more the
// longer the chunks (4 KiB: as long).  Up to two a SIMD they are 2 to 9 % shorter where half of the chunks are raw and between 2 %
// longer and 7 % shorter where none is; short chunks, in which the set-up counts for more, lose there (4 KiB: 1 to 3 %; bf16 of 16 KiB at
// 128 and 256 sub-streams: 1 to 3 %), and so does the conversion at 32 sub-streams, whose stores are in each other's way (up to 8 %).  At three a
// SIMD, where the wavefronts hide each other's look-ups and the LDS is what they wait for, they are 7 to 17 % longer (products at 32
// sub-streams: up to 10 % shorter where all chunks are coded, up to 4 % longer where half are raw, which the host does not know).
// The second copy of the ring's first words saves address arithmetic and costs a store of 16 bytes a lane and half group.  At 32
// sub-streams the conversion is up to 27 % longer with it (2048 chunks of 64 KiB 120.1, without it 105.4 us), products are up to 5 %
// shorter, bytes up to 7 % shorter up to one wavefront a SIMD and from there on up to 3 % longer.  At 64 and 128 it is worth some
// percent either way: it costs most where the LDS of a compute unit has a wavefront of each SIMD, or two, and less with some raw chunks.
// At 128: 1 to 2 % shorter up to three wavefronts to two SIMDs (product of 512 chunks of 64 KiB 30.8, without it 31.5 us), from there on
// 1 % shorter to 2 % longer.  At 64, bytes: 1 to 3 % shorter up to the same line, but chunks of 16 KiB up to 2.6 % longer from half a
// wavefront a SIMD on (1024 of them 14.4 / 14.0); those of 64 KiB with one a SIMD are as long where all are coded and 2 %
// shorter where half are raw.  The conversion: 1 % either way, mostly shorter (640 chunks 55.2 / 56.1, 1024 55.6 / 55.3).
// Products: up to 2 % shorter up to three wavefronts to four SIMDs, 1 to 2 % longer with one on each (int8 product of 1024 chunks 46.2 / 45.4).
int order_of_work(int mode, uint32_t n_streams, uint64_t waves, uint32_t chunk_bytes, uint32_t simds)
{
    const bool bytes = mode == kModeI8, bf16 = mode == kModeBf16;
    const uint64_t two_a_simd = 2ull * simds;
    if (n_streams == 32) {
        if (bf16) return waves <= simds ? kFew : kMany;
        if (waves <= simds) return kFewAgain;
        return waves > two_a_simd || chunk_bytes < 16384 ? kMany : bytes ? kFew : kFewAgain;
    }
    if (waves > simds && (waves > two_a_simd || chunk_bytes < (bf16 ? 32768u : 16384u))) return kMany;
    if (n_streams == 256) return kFew;
    if (n_streams == 64 && bf16) return kFewAgain;
    const uint64_t again = n_streams == 128 || (bytes && chunk_bytes >= 32768) ? simds * 3ull / 2 : bytes ? simds / 2 : simds * 3ull / 4;
    return waves <= again ? kFewAgain : kFew;
}

template <int S, int MODE> void launch_one(const ArgsOf<MODE> &a, hipStream_t stream)
{
    using G = Geometry<S>;
    const uint32_t grid = (uint32_t)((a.n_chunks + G::kChunksPerWave - 1) / G::kChunksPerWave);
    const int order = order_of_work(MODE, S, grid * (uint64_t)G::kWaves, a.chunk_bytes, device_simds());
    constexpr bool BYTES = MODE == kModeI8, BF16 = MODE == kModeBf16;
    if constexpr (S == 32 ? BYTES || BF16 : S == 64 ? !BF16 : S == 128)
        if (order == kFew) {
            hipLaunchKernelGGL((dc_decode_kernel<S, MODE, DC_CODEC_HUFFMAN, true, false, false>), dim3(grid), dim3(G::kThreads), 0, stream, a);
            return;
        }
    if constexpr (S != 32 || !BF16) // (256 sub-streams: the kernel without the copy)
        if (order != kMany) {
            hipLaunchKernelGGL((dc_decode_kernel<S, MODE, DC_CODEC_HUFFMAN, true>), dim3(grid), dim3(G::kThreads), 0, stream, a);
            return;
        }
    hipLaunchKernelGGL((dc_decode_kernel<S, MODE, DC_CODEC_HUFFMAN>), dim3(grid), dim3(G::kThreads), 0, stream, a);
}

// tANS payloads: S >= 64, one chunk per workgroup
template <int MODE> int launch_tans(const ArgsOf<MODE> &a, uint32_t S, hipStream_t stream)
{
    if (a.n_chunks > 0x7FFFFFFFull) return DC_E_ARG;
    const uint32_t grid = (uint32_t)a.n_chunks;
    switch (S) {
    case 64: hipLaunchKernelGGL((dc_decode_kernel<64, MODE, DC_CODEC_TANS>), dim3(grid), dim3(64), 0, stream, a); break;
    case 128: hipLaunchKernelGGL((dc_decode_kernel<128, MODE, DC_CODEC_TANS>), dim3(grid), dim3(128), 0, stream, a); break;
    case 256: hipLaunchKernelGGL((dc_decode_kernel<256, MODE, DC_CODEC_TANS>), dim3(grid), dim3(256), 0, stream, a); break;
    default: return DC_E_ARG;
    }
    return launch_status();
}

template <int MODE> int launch_decode(const ArgsOf<MODE> &a, uint32_t S, hipStream_t stream, uint32_t codec = DC_CODEC_HUFFMAN)
{
    if (codec == DC_CODEC_TANS) return launch_tans<MODE>(a, S, stream);
    if (a.n_chunks > 0x7FFFFFFFull) return DC_E_ARG;
    switch (S) {
    case 32: launch_one<32, MODE>(a, stream); break;
    case 64: launch_one<64, MODE>(a, stream); break;
    case 128: launch_one<128, MODE>(a, stream); break;
    case 256: launch_one<256, MODE>(a, stream); break;
    default: return DC_E_ARG;
    }
    return launch_status();
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

} // namespace

int dc_launch_status()
{
    g_last_hip_error = hipGetLastError();
    return g_last_hip_error == hipSuccess ? DC_OK : DC_E_HIP;
}


extern "C" int dc_decompress_chunks(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev,
                                    uint64_t n_chunks, const dc_params *params, int8_t *dst_dev, uint64_t dst_cap,
                                    void *hip_stream)
{
    if (!decode_params_ok(params) || !blob_dev || !table_dev || !dst_dev || n_chunks == 0 ||
        blob_bytes < DC_BLOB_TAIL_BYTES || blob_bytes % 16)
        return DC_E_ARG;
    if (params->format != DC_FORMAT_ID) return DC_E_FORMAT;
    if (!aligned16(blob_dev) || !aligned16(dst_dev) || (reinterpret_cast<uintptr_t>(table_dev) & 7u)) return DC_E_ARG;
    if (dst_cap < (n_chunks - 1) * (uint64_t)params->chunk_bytes + 1) return DC_E_CAP;
    BytesArgs a = {};
    common_args(a, blob_dev, blob_bytes, table_dev, n_chunks, params);
    a.dst = dst_dev;
    a.dst_cap = dst_cap;
    return launch_decode<kModeI8>(a, params->n_streams, static_cast<hipStream_t>(hip_stream), params->codec);
}

extern "C" int dc_decompress_chunks_traced(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev,
                                           uint64_t n_chunks, const dc_params *params, int8_t *dst_dev, uint64_t dst_cap,
                                           uint64_t *trace_dev, void *hip_stream)
{
    if (!decode_params_ok(params) || !blob_dev || !table_dev || !dst_dev || !trace_dev || n_chunks == 0 ||
        n_chunks > 0x7FFFFFFFull || blob_bytes < DC_BLOB_TAIL_BYTES || blob_bytes % 16)
        return DC_E_ARG;
    if (params->format != DC_FORMAT_ID) return DC_E_FORMAT;
    if (params->codec != DC_CODEC_HUFFMAN || params->n_streams != 256) return DC_E_ARG;
    if (!aligned16(blob_dev) || !aligned16(dst_dev) || (reinterpret_cast<uintptr_t>(table_dev) & 7u) ||
        (reinterpret_cast<uintptr_t>(trace_dev) & 7u))
        return DC_E_ARG;
    if (dst_cap < (n_chunks - 1) * (uint64_t)params->chunk_bytes + 1) return DC_E_CAP;
    BytesArgs a = {};
    common_args(a, blob_dev, blob_bytes, table_dev, n_chunks, params);
    a.dst = dst_dev;
    a.dst_cap = dst_cap;
    a.trace = trace_dev;
    const dim3 grid((uint32_t)n_chunks), block(Geometry<256>::kThreads);
    if (order_of_work(kModeI8, 256, n_chunks * Geometry<256>::kWaves, a.chunk_bytes, device_simds()) != kMany)
        hipLaunchKernelGGL((dc_decode_kernel<256, kModeI8, DC_CODEC_HUFFMAN, true, true>), grid, block, 0, static_cast<hipStream_t>(hip_stream), a);
    else
        hipLaunchKernelGGL((dc_decode_kernel<256, kModeI8, DC_CODEC_HUFFMAN, false, true>), grid, block, 0, static_cast<hipStream_t>(hip_stream), a);
    return launch_status();
}

namespace {

// Host checks shared by the fused calls, and the kernel arguments built from the matrix list.
int fused_args(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev, uint64_t n_chunks,
               const dc_params *params, const dc_matrix *mats, uint32_t n_mats, int mode, DecodeArgs &a)
{
    if (!decode_params_ok(params) || !blob_dev || !table_dev || !mats || n_mats == 0 || n_mats > DC_MAX_MATRICES ||
        n_chunks == 0 || blob_bytes < DC_BLOB_TAIL_BYTES || blob_bytes % 16)
        return DC_E_ARG;
    if (params->format != DC_FORMAT_ID) return DC_E_FORMAT;
    if (!aligned16(blob_dev) || (reinterpret_cast<uintptr_t>(table_dev) & 7u)) return DC_E_ARG;
    a = DecodeArgs{};
    common_args(a, blob_dev, blob_bytes, table_dev, n_chunks, params);
    a.n_mats = n_mats;
    for (uint32_t &first : a.next_first) first = 0xFFFFFFFFu;
    uint64_t next_chunk = 0;
    for (uint32_t i = 0; i < n_mats; i++) {
        const dc_matrix &m = mats[i];
        if (m.rows == 0 || m.cols == 0 || m.cols % 16 || !m.row_scale_dev) return DC_E_ARG;
        const bool gemv = mode != kModeBf16;
        if (mode == kModeGemv) {
            if (!m.x_bf16_dev || !m.y_accum_dev || m.cols > 16384 || !aligned16(m.x_bf16_dev)) return DC_E_ARG;
        } else if (mode == kModeGemvW8A8) {
            if (!m.x_i8_dev || !m.y_accum_dev || m.cols > 16384 || !aligned16(m.x_i8_dev)) return DC_E_ARG;
        } else {
            if (!m.dst_bf16_dev || !aligned16(m.dst_bf16_dev)) return DC_E_ARG;
        }
        const uint64_t total = (uint64_t)m.rows * m.cols;
        if (!gemv && m.dst_cap_elems < total) return DC_E_CAP;
        // the matrices follow each other in the table, each starting at a chunk of its own
        if (m.first_chunk != next_chunk) return DC_E_ARG;
        next_chunk += (total + params->chunk_bytes - 1) / params->chunk_bytes;
        if (i) a.next_first[i - 1] = (uint32_t)m.first_chunk; // below 2^31, or the launch is refused
        MatrixArgs &k = a.mats[i];
        k.first_chunk = m.first_chunk;
        k.rows = m.rows;
        k.cols = m.cols;
        k.row_scale = m.row_scale_dev;
        k.dst = m.dst_bf16_dev;
        k.x_bf16 = m.x_bf16_dev;
        k.y_accum = m.y_accum_dev;
        k.y_bf16 = m.y_bf16_dev;
        k.x_i8 = m.x_i8_dev;
        k.x_scale = m.x_scale;
    }
    if (next_chunk != n_chunks) return DC_E_ARG;
    return DC_OK;
}

} // namespace

extern "C" int dc_decompress_dequant_bf16_layer(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev,
                                                uint64_t n_chunks, const dc_params *params, const dc_matrix *mats_host,
                                                uint32_t n_mats, void *hip_stream)
{
    DecodeArgs a;
    const int rc = fused_args(blob_dev, blob_bytes, table_dev, n_chunks, params, mats_host, n_mats, kModeBf16, a);
    if (rc != DC_OK) return rc;
    return launch_decode<kModeBf16>(a, params->n_streams, static_cast<hipStream_t>(hip_stream), params->codec);
}

namespace {

// Rows a chunk of chunk_bytes bytes can touch in a matrix with rows of `cols` bytes whose first chunk starts a row.
uint64_t rows_touched_by_a_chunk(uint32_t chunk_bytes, uint32_t cols)
{
    if (chunk_bytes % cols == 0) return chunk_bytes / cols;
    return (chunk_bytes + cols - 1) / cols + 1;
}

// Whether no result of the products lies over something that a decoding workgroup reads or the workspace, which one writes:
// then a workgroup may write results while others are still at work.
bool results_apart(const DecodeArgs &a, const void *workspace, uint64_t workspace_bytes)
{
    struct Range { uintptr_t at; uint64_t n; };
    auto apart = [](Range x, Range y) { return x.at + x.n <= y.at || y.at + y.n <= x.at; };
    auto range = [](const void *p, uint64_t n) { return Range{reinterpret_cast<uintptr_t>(p), p ? n : 0}; };
    for (uint32_t i = 0; i < a.n_mats; i++) {
        const MatrixArgs &out = a.mats[i];
        for (const Range &r : {range(out.y_accum, 4ull * out.rows), range(out.y_bf16, 2ull * out.rows)}) {
            if (!apart(r, range(a.blob, a.blob_bytes)) || !apart(r, range(a.table, a.n_chunks * sizeof(dc_chunk))) ||
                !apart(r, range(workspace, workspace_bytes)))
                return false;
            for (uint32_t j = 0; j < a.n_mats; j++) {
                const MatrixArgs &in = a.mats[j];
                if (!apart(r, range(in.row_scale, 4ull * in.rows)) || !apart(r, range(in.x_bf16, 2ull * in.cols)) ||
                    !apart(r, range(in.x_i8, in.cols)))
                    return false;
            }
        }
    }
    return true;
}

// The product fused into the decode: one launch where the chunks hold whole rows; two where a chunk's rows have a lane each (bf16
// activations); else three: zero y, decode, scale y.
template <int MODE>
int gemv_layer(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev, uint64_t n_chunks,
               const dc_params *params, const dc_matrix *mats_host, uint32_t n_mats, void *workspace_dev,
               uint64_t workspace_bytes, void *hip_stream)
{
    DecodeArgs a;
    int rc = fused_args(blob_dev, blob_bytes, table_dev, n_chunks, params, mats_host, n_mats, MODE, a);
    if (rc != DC_OK) return rc;
    RowBlocks rb = {};
    uint32_t row_blocks = 0;
    for (uint32_t &first : rb.first_block) first = 0xFFFFFFFFu;
    rb.chunk_bytes = params->chunk_bytes;
    bool ordered = MODE == kModeGemv;
    // One launch instead of two or three (4 MiB at 256 sub-streams: 21.6 -> 20.0 us, int8 27.0 -> 19.3) if no row reaches
    // into a second chunk, the chunk's rows have a lane each, and results may be written
    // while other chunks are decoded (a caller may put y in the place of x).  The chunks leave their partial sums in the
    // workspace on this route too: what a call leaves there does not depend on where its results lie.
    bool whole_rows = results_apart(a, workspace_dev, n_chunks * kPartialSlots * sizeof(float));
    for (uint32_t i = 0; i < n_mats; i++) {
        rb.mats[i] = a.mats[i];
        rb.first_block[i] = row_blocks;
        row_blocks += (a.mats[i].rows + 255) / 256;
        // the ordered product keeps a row's sum in the lane of the row's number inside the chunk
        if (rows_touched_by_a_chunk(params->chunk_bytes, a.mats[i].cols) > (params->n_streams < 64 ? params->n_streams : 64))
            ordered = whole_rows = false;
        if (params->chunk_bytes % a.mats[i].cols) whole_rows = false;
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (ordered) {
        // decode leaves one sum per chunk and row in the workspace, the finish kernel adds them in chunk order
        if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & 3u)) return DC_E_ARG;
        if (workspace_bytes / (kPartialSlots * sizeof(float)) < n_chunks) return DC_E_CAP;
        a.partial = static_cast<float *>(workspace_dev);
        if (whole_rows) return launch_decode<kModeGemvRows>(a, params->n_streams, stream, params->codec);
        rb.partial = a.partial;
        rc = launch_decode<kModeGemv>(a, params->n_streams, stream, params->codec);
        if (rc != DC_OK) return rc;
        hipLaunchKernelGGL(dc_gemv_ordered_finish_kernel, dim3(row_blocks), dim3(256), 0, stream, rb);
        return launch_status();
    }
    if (MODE == kModeGemvW8A8 && whole_rows) return launch_decode<kModeGemvW8A8Rows>(a, params->n_streams, stream, params->codec);
    hipLaunchKernelGGL(dc_gemv_zero_kernel, dim3(row_blocks), dim3(256), 0, stream, rb);
    rc = launch_decode<MODE == kModeGemv ? kModeGemvAtomic : MODE>(a, params->n_streams, stream, params->codec);
    if (rc != DC_OK) return rc;
    hipLaunchKernelGGL(dc_gemv_finish_kernel<MODE == kModeGemvW8A8>, dim3(row_blocks), dim3(256), 0, stream, rb);
    return launch_status();
}

} // namespace

extern "C" int dc_decompress_gemv_workspace(uint64_t n_chunks, uint64_t *workspace_bytes)
{
    if (!workspace_bytes || n_chunks == 0 || n_chunks > 0x7FFFFFFFull) return DC_E_ARG;
    *workspace_bytes = n_chunks * kPartialSlots * sizeof(float);
    return DC_OK;
}

extern "C" int dc_decompress_gemv_layer(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev,
                                        uint64_t n_chunks, const dc_params *params, const dc_matrix *mats_host,
                                        uint32_t n_mats, void *workspace_dev, uint64_t workspace_bytes, void *hip_stream)
{
    return gemv_layer<kModeGemv>(blob_dev, blob_bytes, table_dev, n_chunks, params, mats_host, n_mats, workspace_dev,
                                 workspace_bytes, hip_stream);
}

extern "C" int dc_decompress_gemv_w8a8_layer(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev,
                                             uint64_t n_chunks, const dc_params *params, const dc_matrix *mats_host,
                                             uint32_t n_mats, void *hip_stream)
{
    return gemv_layer<kModeGemvW8A8>(blob_dev, blob_bytes, table_dev, n_chunks, params, mats_host, n_mats, nullptr, 0,
                                     hip_stream);
}

extern "C" int dc_decompress_gemv_w8a8(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev,
                                       uint64_t n_chunks, const dc_params *params, const float *row_scale_dev,
                                       uint32_t rows, uint32_t cols, const int8_t *x_i8_dev, float x_scale,
                                       float *y_accum_dev, uint16_t *y_bf16_dev, void *hip_stream)
{
    dc_matrix m = {};
    m.rows = rows;
    m.cols = cols;
    m.row_scale_dev = row_scale_dev;
    m.x_i8_dev = x_i8_dev;
    m.x_scale = x_scale;
    m.y_accum_dev = y_accum_dev;
    m.y_bf16_dev = y_bf16_dev;
    return dc_decompress_gemv_w8a8_layer(blob_dev, blob_bytes, table_dev, n_chunks, params, &m, 1, hip_stream);
}

extern "C" int dc_decompress_dequant_bf16(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev,
                                          uint64_t n_chunks, const dc_params *params, const float *row_scale_dev,
                                          uint32_t rows, uint32_t cols, uint16_t *dst_bf16_dev, uint64_t dst_cap_elems,
                                          void *hip_stream)
{
    dc_matrix m = {};
    m.rows = rows;
    m.cols = cols;
    m.row_scale_dev = row_scale_dev;
    m.dst_bf16_dev = dst_bf16_dev;
    m.dst_cap_elems = dst_cap_elems;
    return dc_decompress_dequant_bf16_layer(blob_dev, blob_bytes, table_dev, n_chunks, params, &m, 1, hip_stream);
}

extern "C" int dc_decompress_gemv(const uint8_t *blob_dev, uint64_t blob_bytes, const dc_chunk *table_dev,
                                  uint64_t n_chunks, const dc_params *params, const float *row_scale_dev, uint32_t rows,
                                  uint32_t cols, const uint16_t *x_bf16_dev, float *y_f32_dev, uint16_t *y_bf16_dev,
                                  void *workspace_dev, uint64_t workspace_bytes, void *hip_stream)
{
    dc_matrix m = {};
    m.rows = rows;
    m.cols = cols;
    m.row_scale_dev = row_scale_dev;
    m.x_bf16_dev = x_bf16_dev;
    m.y_accum_dev = y_f32_dev;
    m.y_bf16_dev = y_bf16_dev;
    return dc_decompress_gemv_layer(blob_dev, blob_bytes, table_dev, n_chunks, params, &m, 1, workspace_dev,
                                    workspace_bytes, hip_stream);
}

extern "C" const char *dc_last_hip_error(void) { return hipGetErrorString(g_last_hip_error); }

extern "C" int dc_gemv_w8a8(const int8_t *q_dev, const float *row_scale_dev, uint32_t rows, uint32_t cols,
                            const int8_t *x_i8_dev, float x_scale, float *y_f32_dev, uint16_t *y_bf16_dev, void *hip_stream)
{
    if (!q_dev || !row_scale_dev || !x_i8_dev || !y_f32_dev || rows == 0 || cols == 0 || cols % 16 || cols > 16384)
        return DC_E_ARG;
    if (!aligned16(q_dev) || !aligned16(x_i8_dev)) return DC_E_ARG;
    const uint32_t blocks = (rows + kGemvRows - 1) / kGemvRows;
    hipLaunchKernelGGL(dc_gemv_w8a8_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       reinterpret_cast<const uint8_t *>(q_dev), row_scale_dev, rows, cols, x_i8_dev, x_scale, y_f32_dev,
                       y_bf16_dev);
    return launch_status();
}

extern "C" int dc_gemv_i8(const int8_t *q_dev, const float *row_scale_dev, uint32_t rows, uint32_t cols,
                          const uint16_t *x_bf16_dev, float *y_f32_dev, uint16_t *y_bf16_dev, void *hip_stream)
{
    if (!q_dev || !row_scale_dev || !x_bf16_dev || !y_f32_dev || rows == 0 || cols == 0 || cols % 16) return DC_E_ARG;
    if (!aligned16(q_dev) || !aligned16(x_bf16_dev)) return DC_E_ARG;
    const uint32_t blocks = (rows + kGemvRows - 1) / kGemvRows;
    hipLaunchKernelGGL(dc_gemv_i8_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       reinterpret_cast<const uint8_t *>(q_dev), row_scale_dev, rows, cols, x_bf16_dev, y_f32_dev,
                       y_bf16_dev);
    return launch_status();
}

extern "C" int dc_device_copy(const void *src_dev, void *dst_dev, uint64_t bytes, void *hip_stream)
{
    if (!src_dev || !dst_dev || bytes == 0 || bytes % 16 || !aligned16(src_dev) || !aligned16(dst_dev)) return DC_E_ARG;
    const uint64_t n16 = bytes / 16;
    // one 16-byte element a thread: measured 6.5 TB/s (read + write) on 6.5 GB, where a grid capped at 32
    // workgroups a compute unit that strides over the buffer reads 4.9
    uint64_t blocks = (n16 + 255) / 256;
    if (blocks > 0x7FFFFFFFull) blocks = 0x7FFFFFFFull;
    hipLaunchKernelGGL(dc_copy_kernel, dim3((uint32_t)blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<const u32x4 *>(src_dev), static_cast<u32x4 *>(dst_dev), n16);
    return launch_status();
}
