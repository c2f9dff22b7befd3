// Device side of libdc_mi355x: chunk compression on the GPU (the compression stage of Section 3.1 of
// the paper; Section 4.2 also reports compression speed).  Three launches, two where chunks are raw or coded
// each by itself:
//   dc_codes_kernel   one workgroup per chunk: byte histogram, length-limited code lengths by
//                     package-merge (same ordering rules as the host compressor, so the lengths are
//                     identical), bits of every sub-stream, size of the Huffman payload;
//   dc_layout_kernel  one workgroup: which chunks stay raw, payload offsets (prefix sum), chunk table (up to
//                     8192 chunks that are raw or coded each by itself, the next kernel does this on the side: own_place);
//   dc_emit_kernel    one workgroup per chunk: header, canonical codes, and the sub-streams written as
//                     16-byte blocks in the order of the format's placement rule.
// For the container's second coder (tANS) dc_tans_model_kernel takes the place of dc_codes_kernel: byte
// histogram, frequencies normalised to 2048 by the format's rule, the states of every value, and every
// sub-stream coded backwards once, which leaves one 96-bit item (fields and width) per eight bytes in the
// workspace; dc_emit_kernel then writes those items forwards where it would write codes.
// The stored format is in include/dc.h.
#include <hip/hip_runtime.h>

#include <mutex>

#include "dc.h"
#include "dc_device.h"

using namespace dcdev;

namespace {

constexpr int kL = DC_MAX_CODE_LEN;
constexpr uint32_t kBlockBits = 8 * DC_BLOCK_BYTES;

struct EncArgs {
    const uint8_t *src;
    uint64_t raw_bytes;
    uint64_t n_chunks;
    uint32_t chunk_bytes;
    uint32_t S;
    uint32_t policy;
    uint32_t block_chunks;
    uint64_t n_raw; // DC_POLICY_RAW_FRACTION: chunks that stay raw
    uint32_t codec;
    bool placed; // the layout kernel has run; else the coder finds the chunks' places
    // workspace
    uint8_t *lens;  // [n_chunks][256] code lengths (Huffman)
    uint32_t *bits; // [n_chunks][S] bits of every sub-stream
    uint32_t *comp; // [n_chunks] bytes of the coded payload
    uint16_t *freq;  // tANS: [n_chunks][256] normalised frequencies
    uint16_t *first; // tANS: [n_chunks][S] first state of every sub-stream
    uint8_t *items;  // tANS: [n_chunks][2 * chunk_bytes], see item_place
    // results
    uint8_t *blob;
    uint64_t blob_cap;
    dc_chunk *table;
    uint64_t *result; // [0] blob bytes needed, [1] 0 or DC_E_CAP as an unsigned value
};

__device__ __forceinline__ uint32_t set_width(uint32_t S) { return S < 64 ? S : 64; }
// bytes of the code description at the start of a payload: 256 code lengths, or 256 frequencies of 12 bits
__device__ __forceinline__ uint32_t front_bytes(uint32_t codec) { return codec == DC_CODEC_TANS ? 384u : 128u; }
__device__ __forceinline__ uint32_t header_bytes(uint32_t S, uint32_t codec = DC_CODEC_HUFFMAN)
{
    return (front_bytes(codec) + 2 * S + 4 * (S / set_width(S)) + 15) / 16 * 16;
}
// A sub-stream of `bits` bits is cut into blocks from its end: bytes, 16-byte blocks, and bytes of the short first block.
__device__ __forceinline__ uint32_t bytes_of(uint32_t bits) { return (bits + 7) / 8; }
__device__ __forceinline__ uint32_t blocks_of(uint32_t bits) { return (bytes_of(bits) + DC_BLOCK_BYTES - 1) / DC_BLOCK_BYTES; }
__device__ __forceinline__ uint32_t head_bytes_of(uint32_t bits) { return bits ? bytes_of(bits) - DC_BLOCK_BYTES * (blocks_of(bits) - 1) : 0; }
__device__ __forceinline__ uint32_t chunk_len(const EncArgs &a, uint64_t k)
{
    const uint64_t lo = k * a.chunk_bytes;
    const uint64_t left = a.raw_bytes - lo;
    return left < a.chunk_bytes ? (uint32_t)left : a.chunk_bytes;
}

// Pairs of codes (at most 22 bits each, their widths in the low bytes of l) joined to the at most 88 bits of half a group.
// some: the first two pairs may have no bits at all.
struct HalfGroup {
    uint32_t w0, w1, w2;
    uint32_t bits; // in the low byte
};
__device__ __forceinline__ HalfGroup joined(const uint32_t p[4], const uint32_t l[4], bool some)
{
    const uint64_t lo = (uint64_t)p[1] << (l[0] & 63u) | p[0], hi = (uint64_t)p[3] << (l[2] & 63u) | p[2];
    const uint32_t m = l[0] + l[1]; // at most 44
    const uint64_t low = lo | hi << (m & 63u);
    const uint32_t high = !some || (m & 0xFFu) ? (uint32_t)(hi >> ((64 - m) & 63u)) : 0u;
    return {(uint32_t)low, (uint32_t)(low >> 32), high, m + l[2] + l[3]};
}

// What the tANS model kernel leaves for the coder: half a group in three words, its width above the 24 bits that the third
// needs.  A chunk's items lie by rounds of its sub-streams' groups, as the coder reads them: four words of every
// group, then the other two (24 bytes a group of the 32 it has in the workspace).  With an item of 32 bits for every two bytes the
// two kernels moved 180 MB of items for 45 MB of bytes; now 135, and the coder does not join them (the call 72.5 -> 68.2 us, of 202 MB
// 321 -> 266).
struct ItemPlace {
    uint64_t first, rest; // bytes from the start of the items
};
__device__ __forceinline__ ItemPlace item_place(uint64_t k, uint32_t chunk_bytes, uint32_t groups, uint32_t S, uint32_t r, uint32_t t)
{
    const uint32_t in_round = groups - r * S < S ? groups - r * S : S;
    const uint64_t round = k * 2 * chunk_bytes + 24 * r * S;
    return {round + 16 * t, round + 16 * in_round + 8 * t};
}

// step(16 bytes) for the groups t, t + 256, ... below n16, four loads in flight (one load at a time left a chunk alone on its
// compute unit waiting for memory sixteen times over: 8 us of the 28 us such a chunk of 64 KiB took in the statistics).
template <typename Step> __device__ __forceinline__ void each_group(const uint8_t *src, uint32_t t, uint32_t n16, Step step)
{
    uint32_t i = t;
    for (; i + 768 < n16; i += 1024) {
        uint32_t at = 16 * i;
        anew(at); // a 32-bit offset each turn, not four pointers carried along
        u32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = *reinterpret_cast<const u32x4 *>(src + (at + 4096 * j));
        keep_order(); // else the last three are asked for once the first has come
#pragma unroll
        for (int j = 0; j < 4; j++) step(v[j]);
    }
    for (; i < n16; i += 256) step(*reinterpret_cast<const u32x4 *>(src + 16 * i));
}

constexpr uint32_t kHistogramPart = 1u << 18; // bytes whose counts fit the fields

// Byte histogram of a chunk by 256 threads.  arena: 4096 words of LDS.  Column c = t mod 32 holds, for every value m of
// the lower seven bits, one word arena[32 m + c] (one column per LDS bank, so the lanes of one update never meet in
// a bank): the bytes with these seven bits in the lower 14 bits of the word, those of them with the eighth bit set above.
// A part of the chunk puts at most 8192 + 15 bytes into a column, so the lower field never carries.  The statistics are bound by the
// vector ALU and by waiting for memory and LDS in turn; laid out like this a byte costs three operations and the update (a
// shift, its address, its increment), where the parity of the value as the choice of the field took five.  With the loads
// and look-ups kept together (each_group, the sub-streams' bits) the kernel takes 76 instead of 81 us on 3088 chunks of 64 KiB,
// the call 159.8 instead of 170.6; 45 MB in chunks of 256 KiB 98 instead of 111.
// Ends with hist[v] valid for all threads.
__device__ __forceinline__ void chunk_histogram(const uint8_t *src, uint32_t raw, uint32_t *arena, uint32_t *hist)
{
    const uint32_t t = threadIdx.x;
    const uint32_t column = lds_address(arena) + 4 * (t & 31u);
    // x: the byte's bit 0 at bit 7
    auto count = [&](uint32_t x) {
        atomicAdd((uint32_t *)(lds_u32 *)(uintptr_t)(column + (x & 0x3F80u)), (x & 0x4000u) | 1u);
    };
    uint32_t sum = 0;
    for (uint32_t from = 0; from < raw; from += kHistogramPart) {
        const uint32_t n = raw - from < kHistogramPart ? raw - from : kHistogramPart;
        for (uint32_t i = t; i < 1024; i += 256) reinterpret_cast<u32x4 *>(arena)[i] = u32x4{0, 0, 0, 0};
        __syncthreads();
        const uint32_t n16 = n / 16;
        each_group(src + from, t, n16, [&](const u32x4 &v) {
#pragma unroll
            for (int w = 0; w < 4; w++) {
                count(v[w] << 7);
                count(v[w] >> 1);
                count(v[w] >> 9);
                count(v[w] >> 17);
            }
        });
        for (uint32_t i = n16 * 16 + t; i < n; i += 256) count((uint32_t)src[from + i] << 7);
        __syncthreads();
        // Threads 2m and 2m + 1 take 16 columns each of the values m and m + 128 and trade their sums; they begin at column m mod 16
        // so that the lanes of a read spread over the banks.
        uint32_t all = 0, upper = 0;
        const uint32_t m = t >> 1;
        uint32_t at = lds_address(arena) + 4 * (32 * m + 16 * (t & 1u) + (m & 15u));
        anew(at);
#pragma unroll
        for (uint32_t i = 0; i < 16; i++) {
            const uint32_t w = lds_load32(at ^ (4 * i));
            all += w & 0x3FFFu;
            upper += w >> 14;
        }
        all += (uint32_t)__builtin_amdgcn_mov_dpp((int)all, 0xB1, 0xF, 0xF, true); // quad_perm 1 0 3 2
        upper += (uint32_t)__builtin_amdgcn_mov_dpp((int)upper, 0xB1, 0xF, 0xF, true);
        sum += (t & 1u) ? upper : all - upper;
        __syncthreads();
    }
    hist[(t >> 1) + 128 * (t & 1u)] = sum;
    __syncthreads();
}

// Bitonic sort of the wave's 64 keys, ascending.  Partners 1, 2 and 8 lanes apart come through the data-parallel primitives.
__device__ __forceinline__ uint32_t wave_sorted(uint32_t k, uint32_t lane)
{
#pragma unroll
    for (uint32_t size = 2; size <= 64; size <<= 1) {
#pragma unroll
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
            uint32_t o;
            if (stride == 1) o = (uint32_t)__builtin_amdgcn_mov_dpp((int)k, 0xB1, 0xF, 0xF, true);       // quad_perm 1 0 3 2
            else if (stride == 2) o = (uint32_t)__builtin_amdgcn_mov_dpp((int)k, 0x4E, 0xF, 0xF, true);  // quad_perm 2 3 0 1
            else if (stride == 8) o = (uint32_t)__builtin_amdgcn_mov_dpp((int)k, 0x128, 0xF, 0xF, true); // rotation by 8 of 16
            else o = (uint32_t)__shfl_xor((int)k, (int)stride);
            const bool smaller = ((lane & size) == 0) == ((lane & stride) == 0); // this lane keeps the smaller key
            k = smaller ? (k < o ? k : o) : (k < o ? o : k);
        }
    }
    return k;
}

// How many of a chunk's leaves (ascending: count << 8 | value) weigh no more than a package.  Weights are put into
// buckets by their exponent and the seven bits behind the first one; for every bucket the number of leaves in the buckets before it is kept.  The
// leaves of the package's own bucket, two as a rule, are looked at together, kAtOnce of them, once halving has left no more; up to a
// weight of 255 all of them count, because there a bucket is one weight.
struct LeafRanks {
    static constexpr uint32_t kBits = 7, kLast = (20 << kBits) + 1; // a bucket heavier than any leaf (a chunk has 2^20 bytes at most)
    static constexpr uint32_t kEntries = 256 * 12;                  // kLast + 2 at least; as many for every thread
    static constexpr uint32_t kAtOnce = 4;                          // leaves behind the last that may be looked at
    uint16_t *lighter;
    const uint32_t *leaves;
    static __device__ __forceinline__ uint32_t bucket(uint32_t weight) // weight: 1 to 2^24
    {
        const uint32_t b = (__float_as_uint((float)weight) >> (23 - kBits)) - (127u << kBits);
        return b < kLast ? b : kLast;
    }
    __device__ __forceinline__ uint32_t not_heavier(uint32_t weight) const
    {
        const uint32_t b = bucket(weight), most = weight << 8 | 0xFFu;
        uint32_t lo = lighter[b], hi = lighter[b + 1];
        lo = weight < 2u << kBits ? hi : lo;
        while (hi - lo > kAtOnce) {
            const uint32_t mid = (lo + hi) / 2;
            if (leaves[mid] <= most) lo = mid + 1;
            else hi = mid;
        }
        uint32_t more = 0; // (behind the bucket's last leaf all are heavier)
#pragma unroll
        for (uint32_t i = 0; i < kAtOnce; i++) more += leaves[lo + i] <= most ? 1u : 0u;
        return lo + more;
    }
};

// Package-merge of few leaves (key: ascending, count << 8 | value; n: 2 to kFewLeavesLoaded), as far as leaves_before[j - 1][m], the leaves among the first
// 2m items of level j.  Thread t owns items 2t and 2t + 1 of a level, the pair that is package t of the next, and searches for the
// number a of leaves among the 2t items before them.  From level to level items get lighter and a falls, by about half as much each
// time, so the search begins that far below the last a and is mostly over after a few steps, after none where there are hardly
// any leaves.  What many leaves take (in the kernel) costs the same whatever their number: the tables of LeafRanks and some
// four trips to LDS a level.  2048 chunks of 4 KiB with it / with this: 2 values 29.7 / 25.4 us, 16 30.2 / 27.1, 64 30.5 / 27.9, 128 31.3 / 30.3; 20 of 64 values 15.08 / 15.13.
// From 65 leaves on, where more than one wave takes part, it is a chunk's trips to LDS against the compute unit's
// work: 64 such chunks of 128 values take 15.4 / 15.9, so that there it is for launches of more than four workgroups a compute unit.
constexpr uint32_t kFewLeaves = 64, kFewLeavesLoaded = 128;
__device__ __forceinline__ void merge_few(const uint32_t *key, uint32_t n, uint32_t (*packages)[512], uint16_t (*leaves_before)[256])
{
    const uint32_t t = threadIdx.x, d = 2 * t;
    uint32_t size = n, a_last = d < n ? d : n;
    if (d + 1 < n) packages[0][t] = (key[d] >> 8) + (key[d + 1] >> 8);
#pragma unroll 1
    for (uint32_t j = 1; j < kL; j++) {
        if (n > 64) {
            __syncthreads();
        } else { // the first wave has them all
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        const uint32_t *packs = packages[(j - 1) & 1];
        const uint32_t npk = size / 2;
        size = n + npk;
        if (d > size) continue;
        // the smallest a with leaf a heavier than package d - 1 - a
        uint32_t a = d > npk ? d - npk : 0, hi = a_last;
        const uint32_t fall = j < 8 ? 256u >> j : 1u;
        uint32_t mid = a + fall < hi ? hi - fall : (a + hi) / 2;
        while (a < hi) {
            if (key[mid] >> 8 <= packs[d - 1 - mid]) a = mid + 1;
            else hi = mid;
            mid = (a + hi) / 2;
        }
        a_last = a;
        leaves_before[j - 1][t] = (uint16_t)a;
        // items d and d + 1
        const uint32_t b = d - a, l0 = key[a] >> 8, l1 = key[a + 1] >> 8, p0 = packs[b], p1 = packs[b + 1];
        const bool leaf0 = a < n && (b >= npk || l0 <= p0);
        const uint32_t a1 = a + (leaf0 ? 1u : 0u), b1 = b + (leaf0 ? 0u : 1u);
        const uint32_t l = leaf0 ? l1 : l0, p = leaf0 ? p0 : p1;
        const bool leaf1 = a1 < n && (b1 >= npk || l <= p);
        if (d + 1 < size) packages[j & 1][t] = (leaf0 ? l0 : p0) + (leaf1 ? l : p);
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void dc_codes_kernel(EncArgs a)
{
    // 16 KiB used twice: first the histogram columns, then the tables of the package-merge.
    __shared__ __attribute__((aligned(64))) uint32_t arena[4096];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t key[256 + LeafRanks::kAtOnce]; // count << 8 | byte value, ascending after the sort; absent values last
    __shared__ uint32_t bought_leaves[kL];
    __shared__ uint8_t len_of[256];
    __shared__ uint32_t sbits[256];
    __shared__ uint32_t area_bytes[4]; // per stream set: whole blocks and short first blocks
    uint32_t *unsorted = arena;                                                          // [256] the waves' sorted keys
    uint32_t(*in_waves)[4][4] = reinterpret_cast<uint32_t(*)[4][4]>(arena);              // [two in turn][limit][wave], see wave_limits
    uint32_t *lighter = arena + 256;                                                     // LeafRanks
    uint32_t(*items)[512] = reinterpret_cast<uint32_t(*)[512]>(arena + 1792);            // packages where they lie among a level's items, two levels in turn
    uint16_t(*leaves_before)[256] = reinterpret_cast<uint16_t(*)[256]>(arena + 2816);    // [kL - 1][256], of level 1 and up
    static_assert(LeafRanks::kEntries / 2 == 1536 && 2816 + (kL - 1) * 128 <= 4096, "one behind the other");

    const uint32_t t = threadIdx.x;
    const uint64_t k = blockIdx.x;
    const uint32_t raw = chunk_len(a, k);
    const uint8_t *src = a.src + k * a.chunk_bytes;

    sbits[t] = 0;
    len_of[t] = 0;
    if (t < 4) area_bytes[t] = 0;
    chunk_histogram(src, raw, arena, hist);

    for (uint32_t i = t; i < (LeafRanks::kEntries / 2 + 1024) / 4; i += 256) reinterpret_cast<u32x4 *>(lighter)[i] = u32x4{0, 0, 0, 0};
    if (t < LeafRanks::kAtOnce) key[256 + t] = ~0u;
    const uint32_t cnt = hist[t];
    const uint32_t n = (uint32_t)__syncthreads_count(cnt != 0);
    const bool few = n <= (a.n_chunks > 1024 ? kFewLeavesLoaded : kFewLeaves);
    // leaves in order of (count, byte value): sorted in the waves first, then every key finds its place among the other
    // three waves' keys
    {
        const uint32_t lane = t & 63u, wave = t >> 6;
        const uint32_t k1 = wave_sorted(cnt ? (cnt << 8 | t) : (0xFF000000u | t), lane); // counts are below 2^24 - 2^16
        unsorted[t] = k1;
        __syncthreads();
        uint32_t place = lane;
#pragma unroll
        for (uint32_t o = 1; o < 4; o++) {
            const uint32_t *other = unsorted + 64 * ((wave + o) & 3u);
            uint32_t below = 0;
#pragma unroll
            for (uint32_t step = 32; step > 0; step >>= 1) below += other[below + step - 1] < k1 ? step : 0u;
            place += below + (other[below] < k1 ? 1u : 0u);
        }
        key[place] = k1;
    }
    __syncthreads();

    if (n == 1) {
        if (t == 0) len_of[key[0] & 0xFFu] = 1;
    } else if (n >= 2 && few) {
        merge_few(key, n, items, leaves_before);
    } else if (n >= 2) {
        // Package-merge: level 0 is the sorted leaves; level j is the leaves merged with the pairs of
        // level j-1, a leaf before a package of equal weight.  leaves_before[j][m] = leaves among the
        // first 2m items of level j (no other numbers are asked for).
        // Thread t makes package t of every level.  The leaves are the same at all levels, so how many of them come before a package is
        // looked up (LeafRanks); the package goes to its place among the items, what is left empty there are the leaves in their
        // order, and a thread finds its next package's two items by counting packages: one barrier a level and four
        // trips to LDS one after the other, where a search for the number of leaves before every second item took some ten.  A chunk alone on
        // its compute unit spends 5.2 us here instead of 6.5, together with seven others 7.0 instead of 8.4; the call 31.8 instead of 32.9 us on 256
        // chunks of 64 KiB, 18.1 instead of 18.9 on 64 of 16 KiB, 146.2 instead of 148.1 on 3088 of 64 KiB.
        const uint32_t lane = t & 63u, wave = t >> 6;
        // How many threads' values are below each of three limits, 1 to 3 times `limit`, wave by wave.
        auto wave_limits = [&](uint32_t (*to)[4], uint32_t v, uint32_t limit) {
            uint32_t count = 0;
#pragma unroll
            for (uint32_t w = 1; w < 4; w++) count = with_lane(count, w, (uint32_t)__popcll(__ballot(v < w * limit)));
            if (lane < 4) to[lane][wave] = count;
        };
        auto below_own = [&](uint32_t (*from)[4]) { // those below this wave's limit
            const u32x4 c = *reinterpret_cast<const u32x4 *>(from[wave]);
            return c[0] + c[1] + c[2] + c[3];
        };
        const LeafRanks ranks = {reinterpret_cast<uint16_t *>(lighter), key};
        {
            const uint32_t own = LeafRanks::bucket(key[t] >> 8), next = t + 1 < n ? LeafRanks::bucket(key[t + 1 < 255 ? t + 1 : 255] >> 8) : ~0u;
            if (t < n && own != next) ranks.lighter[own + 1] = (uint16_t)(t + 1); // the last leaf of its bucket
            wave_limits(in_waves[0], t < n ? own + 1 : ~0u, LeafRanks::kEntries / 4);
        }
        __syncthreads();
        {
            // every bucket without a mark takes the one before it
            constexpr int PER = LeafRanks::kEntries / 256 / 2;
            uint32_t *mine = lighter + PER * t, w[PER], tail = 0;
#pragma unroll
            for (int i = 0; i < PER; i++) {
                w[i] = mine[i];
                tail = w[i] & 0xFFFFu ? w[i] & 0xFFFFu : tail;
                tail = w[i] >> 16 ? w[i] >> 16 : tail;
            }
            uint32_t cur = lanes_last_nonzero_below<false>(tail);
            cur = cur ? cur : below_own(in_waves[0]);
#pragma unroll
            for (int i = 0; i < PER; i++) {
                const uint32_t lo = w[i] & 0xFFFFu ? w[i] & 0xFFFFu : cur;
                cur = w[i] >> 16 ? w[i] >> 16 : lo;
                mine[i] = lo | cur << 16;
            }
        }
        uint32_t size = n;
        uint32_t weight = (key[2 * t < 255 ? 2 * t : 255] >> 8) + (key[2 * t < 254 ? 2 * t + 1 : 255] >> 8);
        __syncthreads();
#pragma unroll 1
        for (int j = 1; j < kL; j++) {
            const uint32_t packages = size / 2;
            size = n + packages;
            uint32_t *level = items[j & 1];
            uint32_t place = ~0u;
            if (t < packages) {
                place = t + ranks.not_heavier(weight);
                level[place] = weight;
            }
            wave_limits(in_waves[j & 1], place, 128);
            __syncthreads();
            uint2 *pair = reinterpret_cast<uint2 *>(level) + t;
            const uint2 v = *pair;
            const uint32_t before = below_own(in_waves[j & 1]);
            *pair = make_uint2(0, 0); // for the level after next
            const uint64_t m0 = __ballot(v.x != 0), m1 = __ballot(v.y != 0);
            uint32_t packs = __builtin_amdgcn_mbcnt_hi((uint32_t)(m0 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m0, before));
            packs = __builtin_amdgcn_mbcnt_hi((uint32_t)(m1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m1, packs));
            const uint32_t a0 = 2 * t - packs, a1 = a0 + (v.x ? 0u : 1u); // the leaves that may be items 2t and 2t + 1
            leaves_before[j - 1][t] = (uint16_t)a0;
            const uint32_t l0 = key[a0 < 255 ? a0 : 255] >> 8, l1 = key[a1 < 255 ? a1 : 255] >> 8;
            weight = (v.x ? v.x : l0) + (v.y ? v.y : l1);
        }
    }
    if (n >= 2) {
        __syncthreads();
        if (t == 0) {
            uint32_t bought = 2 * n - 2;
            for (int j = kL - 1; j >= 0; j--) {
                uint32_t nl = 0;
                if (bought > 0) {
                    nl = j ? leaves_before[j - 1][bought / 2] : bought;
                    bought = 2 * (bought - nl);
                }
                bought_leaves[j] = nl;
            }
        }
        __syncthreads();
        if (t < n) {
            uint32_t depth = 0;
#pragma unroll
            for (int j = 0; j < kL; j++) depth += t < bought_leaves[j];
            len_of[key[t] & 0xFFu] = (uint8_t)depth;
        }
    }
    __syncthreads();
    a.lens[k * 256 + t] = len_of[t];

    // bits of every sub-stream: thread t sees the 16-byte groups t, t + 256, ... which all belong to
    // sub-stream t mod S (S divides 256)
    const uint32_t groups = (raw + 15) / 16;
    uint32_t mine = 0;
    each_group(src, t, raw / 16, [&](const u32x4 &v) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            uint32_t l[8]; // eight look-ups on their way before the first is added
#pragma unroll
            for (int i = 0; i < 8; i++) l[i] = len_of[(v[2 * h + (i >> 2)] >> (8 * (i & 3))) & 0xFFu];
            keep_order();
#pragma unroll
            for (int i = 0; i < 8; i++) mine += l[i];
            anew(mine);
        }
    });
    if (groups > raw / 16 && t == (groups - 1) % 256) // the last group lacks bytes
        for (uint32_t p = 16 * (groups - 1); p < raw; p++) mine += len_of[src[p]];
    if (mine) atomicAdd(&sbits[t % a.S], mine);
    __syncthreads();
    if (t < a.S) {
        a.bits[k * a.S + t] = sbits[t];
        if (sbits[t]) atomicAdd(&area_bytes[t / set_width(a.S)], DC_BLOCK_BYTES * (blocks_of(sbits[t]) - 1) + head_bytes_of(sbits[t]));
    }
    __syncthreads();
    if (t == 0) {
        uint32_t size = header_bytes(a.S);
        for (uint32_t w = 0; w < a.S / set_width(a.S); w++) size += (area_bytes[w] + 15u) & ~15u;
        a.comp[k] = size;
    }
}


// ---------------------------------------------------------------------------------------------
// tANS: frequencies, states, and every sub-stream coded backwards once
// ---------------------------------------------------------------------------------------------

constexpr uint32_t kTansBits = DC_TANS_STATE_BITS;
constexpr uint32_t kTansL = 1u << kTansBits;

// Smallest of the lanes' values, for all lanes.
__device__ __forceinline__ float lanes_smallest(float v)
{
    const uint32_t none = __float_as_uint(__builtin_huge_valf()); // what a lane without a source counts as
#define DC_SMALLEST_STEP(CTRL, MASK)                                                                                     \
    v = __builtin_fminf(__uint_as_float((uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)__float_as_uint(v), CTRL, MASK, 0xF, false)), v);
    DC_SMALLEST_STEP(0x111, 0xF)
    DC_SMALLEST_STEP(0x112, 0xF)
    DC_SMALLEST_STEP(0x114, 0xF)
    DC_SMALLEST_STEP(0x118, 0xF)
    DC_SMALLEST_STEP(0x142, 0xA)
    DC_SMALLEST_STEP(0x143, 0xC)
#undef DC_SMALLEST_STEP
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), 63));
}

// The second half of the normalisation rule by one wavefront; lane l holds counts and frequencies of the values l, l + 64,
// l + 128, l + 192.

// Too few states: `steps` times the value with the largest count / q gains one, the lower value among equals.  No value
// gains twice: with R = raw / 2048, a value whose share is one state or more has count / q >= R before and count / (q + 1) < R
// after, a value that got its one state for being present has count < R, and there are more of the former than steps, which
// are the sum of their shares' fractions less what the others were given.  So the steps go to the `steps` largest ratios, found
// through the smallest of them, bit by bit.  Ratios are below 1024 and two of them differ by 1 / (2048 * 2048) or more, so
// that their fixed-point quotients of 22 bits (grant_key) stand in the same order, and only equal ones are equal.  Four bits a turn, without
// branches, until no more keys are left than steps.
// (One step at a time, a reduction over the lanes each: the whole call 77 us on 688 chunks of 64 KiB and 65 on 1024 of 16 KiB
// where it now takes 69 and 40.)
__device__ __forceinline__ uint32_t grant_key(uint32_t count, uint32_t q, uint32_t raw)
{
    const uint32_t d = q ? q : 1u, high = (count << 11) / d, rest = (count << 11) - high * d;
    return (count << kTansBits) >= raw ? (high << 11) + (rest << 11) / d : 0u;
}
__device__ __forceinline__ void grant_states(const uint32_t key[4], uint32_t q[4], uint32_t steps)
{
    uint32_t last = 0; // the smallest key that gains: the largest that `steps` keys are not below
    uint32_t gain = 0; // how many keys are not below it
#pragma unroll 1
    for (int at = 28; at >= 0 && gain != steps; at -= 4)
#pragma unroll
        for (int j = 3; j >= 0; j--) {
            const uint32_t next = last | 1u << (at + j);
            uint32_t n = 0;
#pragma unroll
            for (int i = 0; i < 4; i++) n += (uint32_t)__popcll(__ballot(key[i] >= next));
            last = n >= steps ? next : last;
            gain = n >= steps ? n : gain;
        }
#pragma unroll
    for (int i = 0; i < 4; i++) steps -= (uint32_t)__popcll(__ballot(key[i] > last)); // what is left for keys equal to it
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const uint64_t m = __ballot(key[i] == last);
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        q[i] += key[i] > last || (key[i] == last && rank < steps) ? 1u : 0u;
        const uint32_t n = (uint32_t)__popcll(m);
        steps -= n < steps ? n : steps;
    }
}

// Too many states: `steps` times the value with q > 1 and the smallest count / (q - 1) loses one, the lower value among equals.
// A value may lose several.  A step is a serial link, so it is kept short: the
// ratios are held as 32-bit quotients, which are within 2^-22 of the ratio (counts and divisors are exact, the
// reciprocal is within one unit of the last place and the product within half of one); the value sought has a quotient
// within 2^-20 of the best one, and where several have, their exact cross products (below 2^31) decide.
// (Cross products of (count, divisor, value) triples through shuffles: 1.4 us a step.)
__device__ __forceinline__ void take_states(const uint32_t c[4], uint32_t q[4], uint32_t steps, uint32_t lane)
{
    auto ratio = [&](uint32_t count, uint32_t freq) -> float {
        return freq >= 2 ? (float)count * __builtin_amdgcn_rcpf((float)(freq - 1)) : __builtin_huge_valf();
    };
    float key[4];
#pragma unroll
    for (int i = 0; i < 4; i++) key[i] = ratio(c[i], q[i]);
    for (; steps > 0; steps--) {
        float mine = key[0];
#pragma unroll
        for (int i = 1; i < 4; i++) mine = __builtin_fminf(key[i], mine);
        const float near = lanes_smallest(mine) * (1.0f + 0x1p-20f);
        uint64_t m[4];
        uint32_t many = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            m[i] = __ballot(key[i] <= near);
            many += (uint32_t)__popcll(m[i]);
        }
        uint32_t value = m[0] ? (uint32_t)__builtin_ctzll(m[0]) : m[1] ? 64u + (uint32_t)__builtin_ctzll(m[1])
                       : m[2] ? 128u + (uint32_t)__builtin_ctzll(m[2]) : 192u + (uint32_t)__builtin_ctzll(m[3] | 1ull << 63);
        if (many != 1) {
            // in ascending order of the values, so that only a strictly better ratio takes over
            uint32_t best_c = 0, best_d = 0;
#pragma unroll
            for (uint32_t i = 0; i < 4; i++)
                for (uint64_t left = m[i]; left; left &= left - 1) {
                    const uint32_t from = (uint32_t)__builtin_ctzll(left);
                    const uint32_t count = (uint32_t)__builtin_amdgcn_readlane((int)c[i], from);
                    const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)q[i], from) - 1;
                    if (best_d == 0 || count * best_d < best_c * d) {
                        best_c = count;
                        best_d = d;
                        value = 64 * i + from;
                    }
                }
        }
#pragma unroll
        for (uint32_t i = 0; i < 4; i++)
            if (value == lane + 64 * i) {
                q[i]--;
                key[i] = ratio(c[i], q[i]);
            }
    }
}

__global__ __launch_bounds__(256) void dc_tans_model_kernel(EncArgs a)
{
    __shared__ __attribute__((aligned(64))) uint32_t arena[4096];   // histogram columns; then marks (u16[2048]) and state_of (u16[2048])
    __shared__ uint32_t hist[256];
    __shared__ uint32_t nq[256];       // normalised frequencies
    __shared__ uint32_t cumq[256];     // first place | frequency << 16
    __shared__ uint32_t step_of[256];  // what a symbol does to X (see below)
    __shared__ uint32_t wave_sum[4];
    __shared__ uint32_t area_bytes[4];
    uint16_t *marks = reinterpret_cast<uint16_t *>(arena);
    uint16_t *state_of = reinterpret_cast<uint16_t *>(arena + 1024); // 2048 + the state of value v numbered q + i at cum[v] + i

    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint64_t k = blockIdx.x;
    const uint32_t raw = chunk_len(a, k);
    const uint8_t *src = a.src + k * a.chunk_bytes;
    const uint32_t S = a.S;

    if (t < 4) area_bytes[t] = 0;
    chunk_histogram(src, raw, arena, hist);

    // ---- frequencies: floor shares, at least one state for a present value, then the difference to 2048
    // settled one state at a time (largest count / frequency gains one; smallest count / (frequency - 1)
    // among frequencies above one loses one; the lower value among equals)
    {
        const uint32_t cnt = hist[t];
        const uint32_t share = (cnt << kTansBits) / raw; // cnt is at most 2^20
        const uint32_t q0 = cnt ? (share ? share : 1u) : 0u;
        nq[t] = q0;
        const uint32_t incl = lanes_prefix_sum<false>(q0);
        if (lane == 63) wave_sum[wave] = incl;
    }
    __syncthreads();
    const int32_t diff = (int32_t)kTansL - (int32_t)(wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3]);
    if (diff > 0) { // the ratios, two divisions each, by all threads
        cumq[t] = grant_key(hist[t], nq[t], raw);
        __syncthreads();
    }
    if (wave == 0) {
        uint32_t c[4], q[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            c[i] = hist[lane + 64 * i];
            q[i] = nq[lane + 64 * i];
        }
        if (diff > 0) {
            uint32_t key[4];
#pragma unroll
            for (int i = 0; i < 4; i++) key[i] = cumq[lane + 64 * i];
            grant_states(key, q, (uint32_t)diff);
        } else if (diff < 0) take_states(c, q, (uint32_t)-diff, lane);
#pragma unroll
        for (int i = 0; i < 4; i++) nq[lane + 64 * i] = q[i];
    }
    for (uint32_t i = t; i < 1024; i += 256) arena[i] = 0; // the marks
    __syncthreads();

    // ---- places: value v owns places cum[v] .. cum[v] + q[v] - 1 of the 2048
    const uint32_t qv = nq[t];
    {
        const uint32_t incl = lanes_prefix_sum<false>(qv);
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        uint32_t cum = incl - qv;
        for (uint32_t w = 0; w < wave; w++) cum += wave_sum[w];
        cumq[t] = cum | qv << 16;
        a.freq[k * 256 + t] = (uint16_t)qv;
        // A symbol's field has nb bits, nb the smallest n with (X >> n) < 2q: X lies in [2048, 4096), so that is
        // n0 = 12 - (bits of 2q - 1), or one more from X = 2q << n0 on, which lies in (2048, 4096] too:
        // nb = (X + ((n0 + 1) << 12) - (2q << n0)) >> 12.  That addend takes 16 bits (n0 is 11 at most), and so does the place of the value's
        // states less q, in bytes and signed: one word, because the look-ups of this table and of the states, at random, keep the LDS
        // busy through the whole chain.
        const uint32_t n0 = (uint32_t)__builtin_clz((2 * qv - 1) | 1u) - (31 - kTansBits);
        step_of[t] = ((((n0 + 1) << 12) - (2 * qv << n0)) & 0xFFFFu) | 2 * (cum - qv) << 16;
        if (qv) {
            marks[cum] = (uint16_t)(t + 1);
            // also at the first place of every later wave of the pass below that the value reaches into
            for (uint32_t p = (cum / 512 + 1) * 512; p < cum + qv; p += 512) marks[p] = (uint16_t)(t + 1);
        }
    }
    __syncthreads();
    // ---- states: place p is state rev11(p); the states of a value in ascending order are numbered q, q + 1, ...
    // Thread t takes places 8t .. 8t + 7; the number of place p among the places a .. e - 1 of its value is q
    // plus, for every set bit i of p, the places of the value that agree with p below bit i and have bit i
    // clear: (e + M - 1 - c) div M - (a + M - 1 - c) div M with M = 2^(i+1), c = p mod 2^i.  The sums over a and e are kept in
    // the halves of one word, which neither additions nor, with a mask, shifts let into each other.
    {
        const uint4 m4 = *reinterpret_cast<const uint4 *>(marks + 8 * t);
        const uint32_t w16[4] = {m4.x, m4.y, m4.z, m4.w};
        uint32_t tail = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t lo = w16[i] & 0xFFFFu, hi = w16[i] >> 16;
            tail = lo ? lo : tail;
            tail = hi ? hi : tail;
        }
        uint32_t cur = lanes_last_nonzero_below<false>(tail);
        uint32_t first[8], span[8], sum[8], most = 0;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const uint32_t m = (i & 1) ? w16[i / 2] >> 16 : w16[i / 2] & 0xFFFFu;
            cur = m ? m : cur;
            const uint32_t cq = cumq[(cur - 1) & 255u];
            first[i] = cq & 0xFFFFu;
            span[i] = cq + (cq << 16);
            sum[i] = 0;
            most = cq > most ? cq : most;
        }
        // A bit counts only where the value has more places than the bit's weight (of 2^b places in a row no two agree below bit b), so
        // the most frequent value of the wave ends the count; of the lowest three it is known which are set.  (All eleven bits of all
        // places, then those that count in a loop with a branch a thread, then as here, with the ratios above by one wave, by all threads always, where
        // they are asked for: 66 chunks of 8 KiB 15.6 / 15.9 / 15.4 us, of one value 13.4 / 14.2 / 13.9; 2048 of 4 KiB 33.4 / 33.8 / 32.4.)
        auto both = [](uint32_t v) { return v << 16 | v; };
        auto halved = [&](uint32_t v, uint32_t by) { return v >> by & both(0xFFFFu >> by); };
#pragma unroll
        for (uint32_t b = 0; b < 3; b++)
#pragma unroll
            for (uint32_t i = 0; i < 8; i++)
                if (i >> b & 1u) sum[i] += halved(span[i] + both((2u << b) - 1 - (i & ((1u << b) - 1))), b + 1);
#pragma unroll
        for (uint32_t i = 0; i < 8; i++) span[i] -= both(i);
#pragma unroll
        for (uint32_t b = 3; b < kTansBits; b++) {
            if (!__any(most >> 16 > 1u << b)) break;
            const uint32_t from = both((2u << b) - 1 - 8 * (t & ((1u << (b - 3)) - 1)));
            const uint32_t mask = t >> (b - 3) & 1u ? both(0xFFFFu >> (b + 1)) : 0u;
#pragma unroll
            for (int i = 0; i < 8; i++) sum[i] += (span[i] + from) >> (b + 1) & mask;
        }
#pragma unroll
        for (int i = 0; i < 8; i++)
            state_of[(first[i] + (sum[i] >> 16) - (sum[i] & 0xFFFFu)) & (kTansL - 1)] = (uint16_t)(kTansL + (__brev(8 * t + i) >> (32 - kTansBits)));
    }
    __syncthreads();

    // ---- every sub-stream coded from its last symbol to its first: X = 2048; per symbol the smallest n with
    // (X >> n) < 2q, the field X mod 2^n, then X = 2048 + the state of the value numbered X >> n.  The fields of half a group
    // are joined as the coder wants them (joined), and land in the workspace where it reads them (item_place).
    // This is one serial chain per lane, few wavefronts to a SIMD: everything that does not depend on X (the bytes of the
    // next group, what the 16 values do to X) is loaded before the chain needs it, and a link of the chain is four
    // operations and one look-up of the next state (40 us for 688 chunks of 64 KiB when the field's width was worked out
    // from the frequency inside the chain, 22 now, of which the
    // 1.4 KiB a wavefront and round that go to and from memory are the larger part).
    const uint32_t groups = (raw + 15) / 16;
    if (t < S) {
        const uint32_t my_groups = t < groups ? (groups - t + S - 1) / S : 0;
        const uint32_t states = lds_address(state_of);
        uint32_t X = kTansL, bits = 0;
        uint32_t w[4] = {0, 0, 0, 0};
        uint32_t step[16];
        auto step_at = [&](const uint32_t b[4], int i) { return step_of[(b[i >> 2] >> (8 * (i & 3))) & 0xFFu]; };
        auto load_group = [&](uint32_t r) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(src + 16 * (t + r * S));
            w[0] = v[0]; w[1] = v[1]; w[2] = v[2]; w[3] = v[3];
        };
        // Codes a group, the bytes from the n-th on absent.  What its bytes do to X is in `step`, the bytes of group r - 1 are in w; those of group
        // r - 2 are loaded, and what those of r - 1 do is looked up, while the chain waits for its states (looked up ahead of the chain, sixteen at a
        // time: 688 chunks of 64 KiB 66.6 instead of 65.8 us, 45 MB in chunks of 256 KiB 112.9 instead of 109.7, at 128 sub-streams 76.0 instead of 75.1).
        auto code_group = [&](uint32_t r, uint32_t n, bool whole) {
            const uint32_t before[4] = {w[0], w[1], w[2], w[3]};
            if (r > 1) load_group(r - 2);
            uint32_t p[8], l[8];
#pragma unroll
            for (int j = 7; j >= 0; j--) {
                uint32_t field = 0, width = 0;
#pragma unroll
                for (int i = 2 * j + 1; i >= 2 * j; i--) {
                    if (whole || (uint32_t)i < n) {
                        const uint32_t nb = (X + (step[i] & 0xFFFFu)) >> 12;
                        field = field << nb | __builtin_amdgcn_ubfe(X, 0u, nb);
                        width += nb;
                        X = lds_load16(states + (uint32_t)((int32_t)step[i] >> 16) + 2 * (X >> nb));
                    }
                    step[i] = step_at(before, i);
                }
                p[j] = field;
                l[j] = width;
            }
            const HalfGroup h0 = joined(p, l, true), h1 = joined(p + 4, l + 4, true);
            bits += h0.bits + h1.bits;
            const ItemPlace at = item_place(k, a.chunk_bytes, groups, S, r, t);
            *reinterpret_cast<u32x4 *>(a.items + at.first) = u32x4{h0.w0, h0.w1, h0.w2 | h0.bits << 24, h1.w0};
            *reinterpret_cast<uint2 *>(a.items + at.rest) = make_uint2(h1.w1, h1.w2 | h1.bits << 24);
        };
        uint32_t r = my_groups;
        if (r) {
            const uint32_t lo = 16 * (t + (r - 1) * S);
            const uint32_t n = raw - lo < 16 ? raw - lo : 16; // only a stream's last group may lack bytes
            w[0] = w[1] = w[2] = w[3] = 0;
            for (uint32_t i = 0; i < n; i++) w[i >> 2] |= (uint32_t)src[lo + i] << (8 * (i & 3u));
#pragma unroll
            for (int i = 0; i < 16; i++) step[i] = step_at(w, i);
            if (r > 1) load_group(r - 2);
            code_group(--r, n, false);
        }
        while (r > 0) code_group(--r, 16, true);
        if (my_groups) bits += kTansBits;
        a.first[k * S + t] = (uint16_t)(X - kTansL);
        a.bits[k * S + t] = bits;
        if (bits) atomicAdd(&area_bytes[t / set_width(S)], DC_BLOCK_BYTES * (blocks_of(bits) - 1) + head_bytes_of(bits));
    }
    __syncthreads();
    if (t == 0) {
        uint32_t size = header_bytes(S, DC_CODEC_TANS);
        for (uint32_t w = 0; w < S / set_width(S); w++) size += (area_bytes[w] + 15u) & ~15u;
        a.comp[k] = size;
    }
}

// Gain of coding a chunk (raw size less coded payload size) as an unsigned key in the same order.
__device__ __forceinline__ uint32_t gain_key(uint32_t raw, uint32_t coded)
{
    return raw - coded + 0x80000000u; // both are below 2^24
}
__device__ __forceinline__ uint32_t gain_key(const EncArgs &a, uint64_t k) { return gain_key(chunk_len(a, k), a.comp[k]); }

// Whether chunk k stays raw under the policies that look at the chunk alone.
__device__ __forceinline__ bool stays_raw(const EncArgs &a, uint32_t k, uint32_t raw, uint32_t coded)
{
    if (a.policy == DC_POLICY_AUTO) return coded >= raw;
    return a.policy == DC_POLICY_BLOCK_LAST && k % a.block_chunks != a.block_chunks - 1;
}
// What follows the payloads (`bytes` of them), and the result words.
__device__ __forceinline__ void close_blob(const EncArgs &a, uint64_t bytes)
{
    const bool fits = bytes + DC_BLOB_TAIL_BYTES <= a.blob_cap;
    a.result[0] = bytes + DC_BLOB_TAIL_BYTES;
    a.result[1] = fits ? 0 : (uint64_t)(int64_t)DC_E_CAP;
    if (!fits) return;
    // the closing bytes: zeros, then the trailer (magic number, format id and look-ahead, chunk size,
    // sub-streams and coder); the blob is 16-byte aligned and so is `bytes`
    uint32_t *closing = reinterpret_cast<uint32_t *>(a.blob + bytes);
    for (int i = 0; i < (DC_BLOB_TAIL_BYTES - DC_TRAILER_BYTES) / 4; i++) closing[i] = 0;
    uint32_t *trailer = closing + (DC_BLOB_TAIL_BYTES - DC_TRAILER_BYTES) / 4;
    trailer[0] = DC_TRAILER_MAGIC;
    trailer[1] = DC_FORMAT_ID | (uint32_t)DC_LOOKAHEAD_BITS << 16;
    trailer[2] = a.chunk_bytes;
    trailer[3] = a.S | a.codec << 16;
}

// Which chunks stay raw.  DC_POLICY_RAW_FRACTION: the n_raw chunks of lowest gain, lower index first
// among equal gains, i.e. the chunks with key < threshold and the first `equal_raw` chunks with
// key == threshold.
struct RawRule {
    uint32_t threshold;
    uint32_t equal_raw;
};

constexpr uint32_t kLayoutThreads = 1024;
constexpr uint32_t kLayoutTile = 4 * kLayoutThreads; // chunks a pass of the layout kernel looks at

// Sum of v over the threads before this one, and over all of them (`total`).  waves: 16 words of LDS, free again after the
// next barrier that the caller issues.
__device__ __forceinline__ uint32_t threads_prefix_sum(uint32_t v, uint32_t *waves, uint32_t &total)
{
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t incl = lanes_prefix_sum<false>(v);
    if (lane == 63) waves[wave] = incl;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (uint32_t w = 0; w < kLayoutThreads / 64; w++) {
        const uint32_t c = waves[w];
        before += w < wave ? c : 0u;
        total += c;
    }
    return before + incl - v;
}

// One workgroup, because offsets are sums over all chunks before.  Bound by latency: it works through the payload sizes
// in tiles of 4096 chunks, four consecutive ones a thread, so that a tile costs one trip to memory and two barriers (a
// thread with a run of chunks of its own, read one by one, took 13.7 us for 3088 chunks; this takes 5).  Sizes are summed in units
// of 16 bytes: a tile's fit 32 bits.
__global__ __launch_bounds__(kLayoutThreads) void dc_layout_kernel(EncArgs a)
{
    __shared__ uint32_t digit_count[256];
    __shared__ uint32_t waves[2][kLayoutThreads / 64];
    __shared__ uint32_t sel_prefix, sel_rank;
    const uint32_t t = threadIdx.x;
    const bool by_gain = a.policy == DC_POLICY_RAW_FRACTION && a.n_raw > 0;

    RawRule rule = {0, 0};
    if (by_gain) {
        // Radix select, most significant byte first: the key of rank n_raw - 1 in ascending order.
        if (t == 0) {
            sel_prefix = 0;
            sel_rank = (uint32_t)(a.n_raw - 1);
        }
        for (int shift = 24; shift >= 0; shift -= 8) {
            if (t < 256) digit_count[t] = 0;
            __syncthreads();
            const uint32_t prefix = sel_prefix;
            for (uint64_t k = t; k < a.n_chunks; k += kLayoutThreads) {
                const uint32_t key = gain_key(a, k);
                if (shift == 24 || ((key ^ prefix) >> (shift + 8)) == 0) atomicAdd(&digit_count[(key >> shift) & 0xFFu], 1u);
            }
            __syncthreads();
            if (t < 64) {
                // the digit in which the rank lies: four digits a lane, counts of the lanes before
                uint32_t c[4], sum = 0;
#pragma unroll
                for (int i = 0; i < 4; i++) sum += c[i] = digit_count[4 * t + i];
                uint32_t before = lanes_prefix_sum<false>(sum) - sum;
                const uint32_t rank = sel_rank;
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (uint32_t i = 0; i < 4; i++) {
                    if (rank >= before && rank - before < c[i]) {
                        sel_prefix = prefix | (4 * t + i) << shift;
                        sel_rank = rank - before;
                    }
                    before += c[i];
                }
            }
            __syncthreads();
        }
        rule.threshold = sel_prefix;
        rule.equal_raw = sel_rank + 1;
    }

    uint64_t run = 0;       // bytes of the payloads of the tiles before
    uint32_t run_equal = 0; // chunks of exactly the threshold in them
    for (uint64_t tile = 0; tile < a.n_chunks; tile += kLayoutTile) {
        const uint64_t k0 = tile + 4 * t;
        uint32_t coded[4] = {0, 0, 0, 0};
        if (k0 + 4 <= a.n_chunks) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(a.comp + k0);
#pragma unroll
            for (int i = 0; i < 4; i++) coded[i] = v[i];
        } else {
            for (uint32_t i = 0; i < 4; i++)
                if (k0 + i < a.n_chunks) coded[i] = a.comp[k0 + i];
        }
        uint32_t raw[4], key[4], equal = 0;
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            raw[i] = k0 + i < a.n_chunks ? chunk_len(a, k0 + i) : 0u;
            key[i] = gain_key(raw[i], coded[i]);
            equal += by_gain && raw[i] && key[i] == rule.threshold;
        }
        uint32_t equal_total = 0;
        if (by_gain) equal = run_equal + threads_prefix_sum(equal, waves[0], equal_total);
        uint32_t size[4], sum = 0; // in units of 16 bytes
        bool is_raw[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            bool keep = stays_raw(a, (uint32_t)(k0 + i), raw[i], coded[i]); // n_chunks < 2^31
            if (by_gain) keep = key[i] != rule.threshold ? key[i] < rule.threshold : equal++ < rule.equal_raw;
            is_raw[i] = keep;
            size[i] = raw[i] ? (keep ? (raw[i] + 15u) / 16 : coded[i] / 16) : 0u;
            sum += size[i];
        }
        uint32_t total;
        uint64_t off = run + 16ull * threads_prefix_sum(sum, waves[1], total);
#pragma unroll
        for (uint32_t i = 0; i < 4; i++) {
            if (!raw[i]) continue;
            dc_chunk e;
            e.off = off;
            e.comp_bytes = 16 * size[i];
            e.raw_bytes_flags = raw[i] | (is_raw[i] ? DC_CHUNK_RAW : 0u);
            a.table[k0 + i] = e;
            off += e.comp_bytes;
        }
        run += 16ull * total;
        run_equal += equal_total;
        __syncthreads();
    }
    if (t == 0) close_blob(a, run);
}

// The layout without a launch of its own, where every chunk is raw or coded by itself: chunk k's workgroup adds up the sizes of the
// chunks before it (they come out of the L2), writes the chunk's table entry, and the last one closes the blob.  The launch takes 5 us and
// leaves a gap; the sums take more the more chunks there are.  With the launch and without, replays of a graph: 64 chunks of
// 16 KiB 24.3 and 21.6 us, 3072 of 64 KiB 152.3 and 147.1, 8192 of 16 KiB 144.9 and 140.6, of 4 KiB at 64 sub-streams (a quarter of the
// threads) 92.6 and 90.6, with tANS 101.6 and 97.2; 12 288 of 16 KiB 212.0 and 216.8.  Blocks of one or two chunks (BLOCK_LAST) have as
// many sizes to add: one trip to memory after the other they took 10 and 4 % longer than with the launch at 8192 chunks of 4 KiB and 64
// sub-streams, with all asked for in batches 5 and 2 % less.  sums: a word for every wave.
constexpr uint64_t kOwnLayoutChunks = 8192;
template <int THREADS> __device__ __forceinline__ dc_chunk own_place(const EncArgs &a, uint32_t k, uint32_t *sums)
{
    const uint32_t t = threadIdx.x;
    uint32_t sum = 0; // in units of 16 bytes; all chunks before this one are whole
    if (a.policy == DC_POLICY_BLOCK_LAST && a.block_chunks > 1) { // (blocks of one chunk: all are coded)
        // the last of every block_chunks chunks is coded; eight sizes are asked for at once
        const uint32_t blocks = k / a.block_chunks;
        if (t == 0) sum = (k - blocks) * (a.chunk_bytes / 16);
        const uint32_t *p = a.comp + (a.block_chunks - 1);
        uint32_t b = t;
        for (; b + 7 * THREADS < blocks; b += 8 * THREADS) {
            uint32_t v[8];
#pragma unroll
            for (uint32_t i = 0; i < 8; i++) v[i] = p[(b + i * THREADS) * a.block_chunks];
            keep_order();
#pragma unroll
            for (uint32_t i = 0; i < 8; i++) sum += v[i] / 16;
        }
        for (; b < blocks; b += THREADS) sum += p[b * a.block_chunks] / 16;
    } else {
        const uint32_t most = a.policy == DC_POLICY_AUTO ? a.chunk_bytes : 0xFFFFFFFFu; // what a chunk takes at most
        auto add = [&](uint32_t v) { sum += (v < most ? v : most) / 16; };
        uint32_t j = 4 * t;
        for (; j + 4 * THREADS + 4 <= k; j += 8 * THREADS) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(a.comp + j), w = *reinterpret_cast<const u32x4 *>(a.comp + j + 4 * THREADS);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                add(v[i]);
                add(w[i]);
            }
        }
        for (; j < k; j += 4 * THREADS) // (the sizes' array is padded to 256 bytes)
        {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(a.comp + j);
#pragma unroll
            for (uint32_t i = 0; i < 4; i++)
                if (j + i < k) add(v[i]);
        }
    }
    sum = (uint32_t)__builtin_amdgcn_readlane((int)lanes_prefix_sum<false>(sum), 63);
    if (THREADS > 64) {
        if ((t & 63u) == 0) sums[t >> 6] = sum;
        __syncthreads();
        sum = 0;
#pragma unroll
        for (int w = 0; w < THREADS / 64; w++) sum += sums[w];
    }
    const uint32_t raw = chunk_len(a, k), coded = a.comp[k];
    const bool keep = stays_raw(a, k, raw, coded);
    dc_chunk e;
    e.off = 16ull * sum;
    e.comp_bytes = keep ? (raw + 15u) & ~15u : coded;
    e.raw_bytes_flags = raw | (keep ? DC_CHUNK_RAW : 0u);
    if (t == 0) {
        a.table[k] = e;
        if (k + 1 == a.n_chunks) close_blob(a, e.off + e.comp_bytes);
    }
    return e;
}

// One sub-stream while it is written.  The coder keeps step with the decoder it writes for: the placement rule gives block
// f its place when a decoder would ask for it, 3 to 5 blocks before its bits are coded, and the place waits in a queue
// in LDS until the block is full.  The words of the block at the position and the next lie in LDS too.  Positions and block counts are
// kept times 8: bits 8-10 of a position are then the slot of its word as they stand.
struct Coder {
    uint32_t pos;   // 8 * (position in bits, from where block 0 would start)
    uint32_t asked; // 1024 * (blocks that have their place)
};

constexpr uint32_t kPlaces = 8; // places a lane's queue holds; at most 520 bits, 5 blocks, are placed beyond the position
constexpr uint32_t kWords = 8;  // words of a lane: two blocks

// Bound by the issue of vector instructions where the chip is full (four workgroups a compute unit instead of eight cost 7 %), by the trips
// to LDS and memory of a round where it is not.  So a round is free of branches (but for two around a stream's first block), its reads
// stand together ahead of what needs them, and the block at the position lies in LDS: kept in registers, selecting, merging and carrying
// over its words took 24 of the 90 vector operations of half a group, against 14 of 66 and six LDS accesses more.  3088 chunks of 64 KiB
// 77 -> 72 us, 45 MB in chunks of 256 KiB with the statistics 98 -> 83, 256 chunks of 64 KiB at 32 sub-streams with them 129 -> 107.
template <int THREADS, int CODEC> __global__ __launch_bounds__(THREADS) void dc_emit_kernel(EncArgs a)
{
    constexpr int WAVES = THREADS / 64;
    constexpr bool TANS = CODEC == DC_CODEC_TANS;
    constexpr uint32_t kFront = TANS ? 384 : 128; // code description at the start of a payload
    __shared__ __attribute__((aligned(2048))) uint32_t places[WAVES * kPlaces * 64]; // the lanes' queues: payload offsets
    __shared__ __attribute__((aligned(2048))) uint32_t words[WAVES * kWords * 64];   // the lanes' words
    __shared__ uint32_t book[256];                                                  // length | bit-reversed code << 16
    __shared__ uint32_t set_bytes[WAVES], place_sums[WAVES];
    __shared__ uint32_t len_count[4][kL + 1]; // [64 byte values][code length]

    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    const uint64_t k = blockIdx.x;
    const uint32_t S = a.S;
    // Asked for ahead of the chunk's place: the code lengths of the byte values t, t + THREADS, ... and the bits of the lane's
    // stream.  (Trips to memory one after the other and codes numbered in loops over the lengths were 10 of the 34 us of a workgroup's life.)
    constexpr int kValues = 256 / THREADS;
    uint32_t len[kValues];
    if (!TANS)
#pragma unroll
        for (int i = 0; i < kValues; i++) len[i] = a.lens[k * 256 + t + i * THREADS];
    const bool has_stream = t < S;
    const uint32_t stream_bits = has_stream ? a.bits[k * S + t] : 0;
    dc_chunk ent = a.placed ? a.table[k] : own_place<THREADS>(a, (uint32_t)k, place_sums);
    // The entry is the same in all lanes, which the compiler does not see: left in vector registers it makes every store through the window
    // below a loop over the window's values (a round 169 vector and 29 scalar instructions instead of 157 and 18, 3088 chunks of 64 KiB 78.3 us
    // instead of 74.9 in a trace, 688 with tANS 21.0 instead of 19.9).
    auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    ent.off = (uint64_t)uniform((uint32_t)(ent.off >> 32)) << 32 | uniform((uint32_t)ent.off);
    ent.comp_bytes = uniform(ent.comp_bytes);
    ent.raw_bytes_flags = uniform(ent.raw_bytes_flags);
    const uint32_t raw = ent.raw_bytes_flags & ~DC_CHUNK_RAW;
    if (ent.off + ent.comp_bytes + DC_BLOB_TAIL_BYTES > a.blob_cap) return; // the caller's blob is too small
    const uint8_t *src = a.src + k * a.chunk_bytes;
    uint8_t *out = a.blob + ent.off;

    if (ent.raw_bytes_flags & DC_CHUNK_RAW) {
        const uint32_t n16 = raw / 16;
        for (uint32_t base = t; base < n16; base += 4 * THREADS) { // four loads in flight per thread
            u32x4 v[4];
#pragma unroll
            for (uint32_t j = 0; j < 4; j++)
                if (base + j * THREADS < n16) v[j] = load16_stream(src + 16 * (size_t)(base + j * THREADS));
#pragma unroll
            for (uint32_t j = 0; j < 4; j++)
                if (base + j * THREADS < n16)
                    __builtin_nontemporal_store(v[j], reinterpret_cast<u32x4 *>(out + 16 * (size_t)(base + j * THREADS)));
        }
        if (t < 16 && n16 * 16 < raw) out[n16 * 16 + t] = n16 * 16 + t < raw ? src[n16 * 16 + t] : 0;
        return;
    }

    // ---- header: code lengths (tANS: frequencies, two of 12 bits in three bytes), blocks of every sub-stream,
    // region offsets
    if (TANS) {
        for (uint32_t i = t; i < 128; i += THREADS) {
            const uint32_t two = a.freq[k * 256 + 2 * i] | (uint32_t)a.freq[k * 256 + 2 * i + 1] << 12;
            out[3 * i] = (uint8_t)two;
            out[3 * i + 1] = (uint8_t)(two >> 8);
            out[3 * i + 2] = (uint8_t)(two >> 16);
        }
    } else {
#pragma unroll
        for (int i = 0; i < kValues; i++) { // eight lengths to a word, put together by the lanes that hold them
            uint32_t x = len[i] << (4 * (t & 7u));
            x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true); // quad_perm 1 0 3 2
            x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true); // quad_perm 2 3 0 1
            x |= (uint32_t)__shfl_xor((int)x, 4);
            if ((t & 7u) == 0) *reinterpret_cast<uint32_t *>(out + (t + i * THREADS) / 2) = x;
        }
    }
    const uint32_t nb = blocks_of(stream_bits), hb = head_bytes_of(stream_bits);
    const uint32_t pad = nb ? DC_BLOCK_BYTES - hb : 0; // bytes that block 0 of the stream lacks at its front
    if (has_stream) reinterpret_cast<uint16_t *>(out + kFront)[t] = (uint16_t)(nb | (hb ? (hb - 1) << 12 : 0));
    // the area of a stream set: its whole blocks, then the short first blocks, lane after lane
    const uint32_t whole_incl = lanes_prefix_sum<false>(nb ? nb - 1 : 0);
    const uint32_t heads_incl = lanes_prefix_sum<false>(hb);
    const uint32_t whole_total = (uint32_t)__builtin_amdgcn_readlane((int)whole_incl, 63);
    const uint32_t heads_total = (uint32_t)__builtin_amdgcn_readlane((int)heads_incl, 63);
    uint32_t rank[kValues];
    if (!TANS)
#pragma unroll
        for (int i = 0; i < kValues; i++) {
            uint32_t count = 0;
            rank[i] = 0;
#pragma unroll
            for (uint32_t l = 1; l <= (uint32_t)kL; l++) {
                const uint64_t m = __ballot(len[i] == l);
                const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                rank[i] = len[i] == l ? below : rank[i];
                count = lane == l ? (uint32_t)__popcll(m) : count;
            }
            if (lane <= (uint32_t)kL) len_count[wave + i * WAVES][lane] = count;
        }
    if (lane == 63) set_bytes[wave] = (DC_BLOCK_BYTES * whole_total + heads_total + 15u) & ~15u;
    __syncthreads();
    const uint32_t hdr = header_bytes(S, CODEC);
    const uint32_t n_sets = S / set_width(S);
    uint32_t region = hdr; // first byte of this wave's area
    for (uint32_t w = 0; w < wave; w++) region += set_bytes[w];
    if (lane == 0 && wave < n_sets) reinterpret_cast<uint32_t *>(out + kFront + 2 * S)[wave] = region;
    const uint32_t heads_at = region + DC_BLOCK_BYTES * whole_total;                  // the heads of the set, padded to 16 ...
    const uint32_t heads_padded = set_bytes[wave] - DC_BLOCK_BYTES * whole_total; // ... take this many bytes
    for (uint32_t i = kFront + 2 * S + 4 * n_sets + t; i < hdr; i += THREADS) out[i] = 0;

    // ---- canonical codes: numbered in order of (length, byte value).  Before the barrier a wave has ranked its values among those of
    // equal length in the same 64; behind it lane l has the counts of length l, and every shorter code of length m stands
    // for 2^(l - m) codes of length l that come first: a prefix sum over the lanes, aligned to the longest code.
    if (!TANS) {
        uint32_t count[4], total = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
            count[b] = lane <= (uint32_t)kL ? len_count[b][lane] : 0u;
            total += count[b];
        }
        const uint32_t longest = lane <= (uint32_t)kL ? kL - lane : 0u; // how far a code of this length is aligned up
        const uint32_t first = (lanes_prefix_sum<false>(total << longest) - (total << longest)) >> longest;
#pragma unroll
        for (int i = 0; i < kValues; i++) {
            uint32_t base = first;
#pragma unroll
            for (int b = 0; b < 3; b++) base += (uint32_t)b < wave + i * WAVES ? count[b] : 0u;
            const uint32_t code = rank[i] + (uint32_t)__shfl((int)base, (int)len[i]);
            book[t + i * THREADS] = len[i] ? len[i] | (__brev(code) >> ((32 - len[i]) & 31u)) << 16 : 0u;
        }
    }
    __syncthreads();
    // (A set whose sub-streams hold nothing has no part in what follows: of a chunk of 512 bytes the first of 256 sub-streams' four waves codes
    // all, and 8192 such chunks took 5 %, with tANS 11 % longer when the other three went through its rounds as well.)
    if (!has_stream || whole_total + heads_total == 0) return;

    // ---- the sub-stream of this lane
    const uint32_t groups = (raw + 15) / 16;
    const uint32_t rounds = (groups + S - 1) / S;
    const uint32_t full_rounds = raw / (16 * S); // rounds in which every lane has a whole group
    const uint32_t places_lane = lds_address(places + wave * (kPlaces * 64) + lane);
    const uint32_t words_lane = lds_address(words + wave * (kWords * 64) + lane);
    uint32_t next_place = region;
    const uint32_t end_blocks = 8 * kBlockBits * nb;
    // the stream starts behind the `pad` bytes that block 0 lacks; block 0 is among the heads and takes no place
    Coder c = {64 * pad, nb ? 8 * kBlockBits : 0};
    *(lds_u32 *)(uintptr_t)places_lane = StoreWindow::kNowhere;
#pragma unroll
    for (int i = 0; i < 4; i++) *(lds_u32 *)(uintptr_t)(words_lane + 256 * i) = 0; // nothing before the stream's first bit
    u32x4 head = {0, 0, 0, 0};

    // One carrying out of the placement rule.  Every lane writes; one that asks for no block writes where its next place will go
    // (the queue is longer than what is ever placed, so nothing that is still needed lies there).
    auto place = [&]() {
        const uint32_t bound = c.pos + 8 * DC_LOOKAHEAD_BITS;
        const bool want = c.asked < (bound < end_blocks ? bound : end_blocks);
        const uint64_t m = __ballot(want);
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        *(lds_u32 *)(uintptr_t)(((c.asked >> 2) & 256 * (kPlaces - 1)) | places_lane) = next_place + rank * DC_BLOCK_BYTES;
        c.asked += want ? 8 * kBlockBits : 0u;
        next_place += (uint32_t)__popcll(m) * DC_BLOCK_BYTES;
    };
    // What the last half group has completed: block 0 is kept for the heads, any other goes to its place.  The store is issued
    // in any case, for a lane without a complete block outside the window: with a store on some paths only, the wait for the
    // next round's bytes was one for all stores as well.
    const StoreWindow window(out, ent.comp_bytes);
    struct Done {
        uint32_t words; // where the block's words lie
        uint32_t place;
        uint64_t first; // the lanes whose block 0 it is
    } done = {words_lane, StoreWindow::kNowhere, 0};
    // What LDS holds for the next half group: the word that the last bit coded lies in, and the place of the block at the position.
    struct Held {
        uint32_t word, place;
    };
    auto slot_of_word = [&](uint32_t k) { return (lds_u32 *)(uintptr_t)(((c.pos - 8 + 256 * k) & 256 * (kWords - 1)) | words_lane); };
    auto held = [&]() -> Held { return {*slot_of_word(0), lds_load32(((c.pos >> 2) & 256 * (kPlaces - 1)) | places_lane)}; };
    auto completed = [&](bool complete, uint32_t place) { // the block at the position
        done.words = (c.pos & 0x400u) | words_lane;
        done.place = complete ? place : StoreWindow::kNowhere;
        done.first = __ballot(complete && c.pos < 8 * kBlockBits);
    };
    auto hand_over = [&](const u32x4 &v) {
        window.store16(done.place, v);
        if (done.first) {
            keep_order(); // a branch that is hardly ever taken, not four selections
            if (done.first >> lane & 1u) head = v;
        }
    };
    auto done_words = [&]() { return u32x4{lds_load32(done.words), lds_load32(done.words + 256), lds_load32(done.words + 512), lds_load32(done.words + 768)}; };
    // Appends n <= 96 bits, n in the low byte of `bits`.  What the word that the last bit lies in holds is shifted up to its end and goes
    // before the new bits, which then only shift down into their words; a full word is shifted by nothing and written once more.
    auto append = [&](const Held &h, uint32_t w0, uint32_t w1, uint32_t w2, uint32_t bits) {
        const uint32_t up = 0u - (c.pos >> 3); // shifts read the low 5 bits
        *slot_of_word(0) = __builtin_amdgcn_alignbit(w0, h.word << (up & 31u), up);
        *slot_of_word(1) = __builtin_amdgcn_alignbit(w1, w0, up);
        *slot_of_word(2) = __builtin_amdgcn_alignbit(w2, w1, up);
        *slot_of_word(3) = w2 >> (up & 31u);
        const uint32_t end = c.pos + ((bits & 0xFFu) << 3);
        completed((end ^ c.pos) >= 8 * kBlockBits, h.place);
        c.pos = end;
    };

    // what a round codes of this lane's stream: the group's 16 bytes; tANS: its items
    u32x4 in = {0, 0, 0, 0};
    uint2 in_rest = {0, 0};
    auto load_items = [&](uint32_t r) {
        const ItemPlace at = item_place(k, a.chunk_bytes, groups, S, r, t);
        in = *reinterpret_cast<const u32x4 *>(a.items + at.first);
        in_rest = *reinterpret_cast<const uint2 *>(a.items + at.rest);
    };
    auto load_group = [&](uint32_t r) -> uint32_t { // returns the bytes of it that exist
        const uint32_t lo = 16 * (t + r * S);
        const uint32_t in_n = lo < raw ? (raw - lo < 16 ? raw - lo : 16) : 0;
        if (TANS) {
            // the model kernel has left items for every byte of a group, empty ones for bytes that do not exist
            if (in_n) load_items(r);
            else in = u32x4{0, 0, 0, 0}, in_rest = make_uint2(0, 0);
        } else if (in_n == 16) {
            in = *reinterpret_cast<const u32x4 *>(src + lo);
        } else {
            in = u32x4{0, 0, 0, 0};
            for (uint32_t i = 0; i < in_n; i++) in[i >> 2] |= (uint32_t)src[lo + i] << (8 * (i & 3u));
        }
        return in_n;
    };
    auto load_whole_group = [&](uint32_t r) {
        if (TANS) load_items(r);
        else in = *reinterpret_cast<const u32x4 *>(src + 16 * (t + r * S));
    };
    // Codes half a group, at most 88 bits: codes are joined to pairs (22 bits), fours (44) and eights.  In the loop below nothing
    // depends on another lane or on how far the stream has come, so all lanes do the same work at every step.
    auto code_half = [&](const u32x4 &now, const uint2 &rest, uint32_t half, uint32_t n, bool whole) {
        // what depends on the position is read from LDS ahead of the codes
        const u32x4 last = done_words();
        const Held h = held();
        keep_order();
        place();
        HalfGroup g;
        if (TANS) {
            hand_over(last);
            g = half ? HalfGroup{now[3], rest.x, rest.y, 0} : HalfGroup{now[0], now[1], now[2], 0};
            g.bits = g.w2 >> 24;
            g.w2 &= 0xFFFFFFu;
        } else {
            uint32_t p[4], l[4]; // pairs, and their bits in the low byte (shifts read no more than that)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const uint32_t w = now[2 * half + i / 2] >> (16 * (i & 1));
                uint32_t e0 = book[w & 0xFFu], e1 = book[(w >> 8) & 0xFFu];
                if (!whole) {
                    e0 = 2u * i < n ? e0 : 0u;
                    e1 = 2u * i + 1 < n ? e1 : 0u;
                }
                p[i] = (e0 >> 16) | (e1 >> 16) << (e0 & 31u);
                l[i] = e0 + e1;
            }
            hand_over(last);
            g = joined(p, l, !whole);
        }
        append(h, g.w0, g.w1, g.w2, g.bits);
    };

    // step 0 is carried out five times, the first of which takes block 0; a tANS stream opens with its first state, which a
    // decoder reads before the fifth
    for (int pass = 1; pass < 4; pass++) place();
    if (TANS) append(held(), t < groups ? a.first[k * S + t] : 0u, 0, 0, t < groups ? DC_TANS_STATE_BITS : 0u);
    if (full_rounds) load_whole_group(0);
    in_register<false>(in); // so that the wait in the loop is for the turn before and not for the first one's
    if (TANS) in_register<false>(in_rest.x);
    for (uint32_t r = 0; r < full_rounds; r++) {
        const u32x4 now = in;
        const uint2 rest = in_rest;
        load_whole_group(r + 1 < full_rounds ? r + 1 : r);
        code_half(now, rest, 0, 8, true);
        keep_order(); // the second half's addresses are not worked out ahead: registers for eight wavefronts a SIMD
        code_half(now, rest, 1, 8, true);
    }
    if (rounds > full_rounds) { // the chunk's last groups: some lanes have none, one may have a part of one
        const uint32_t n = load_group(full_rounds);
        code_half(in, in_rest, 0, n, false);
        code_half(in, in_rest, 1, n > 8 ? n - 8 : 0, false);
    }
    hand_over(done_words());
    // the last block, unless its last bit was the stream's (the zero bits that fill the last byte are not coded)
    completed(c.pos % (8 * kBlockBits) != 0, held().place);
    hand_over(done_words());

    // ---- the heads of the set: put together where the wave's queues were, once all of its lanes have read the last of
    // their queues, then written with whole 16-byte stores, the padding of the area included.  A lane's block 0 goes, its first
    // `pad` bytes zero, to the place where those bytes would begin: shifted to words, five of them, and added to the
    // cleared area (16 bytes before it for the first lane's).  Byte by byte it took 170 of the wave's 2900 vector operations.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint32_t stage = lds_address(places + wave * (kPlaces * 64));
    typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
    *(lds_u32x4 *)(uintptr_t)(stage + 16 * lane) = u32x4{0, 0, 0, 0};
    if (lane < 2) *(lds_u32x4 *)(uintptr_t)(stage + 16 * (set_width(S) + lane)) = u32x4{0, 0, 0, 0};
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    {
        const uint32_t at = 16 + heads_incl - hb - pad, up = 8 * (at & 3u);
        const uint32_t h[6] = {0, head[0], head[1], head[2], head[3], 0};
#pragma unroll
        for (uint32_t i = 0; i < 5; i++)
            atomicAdd((uint32_t *)(lds_u32 *)(uintptr_t)(stage + (at & ~3u) + 4 * i),
                     (uint32_t)((((uint64_t)h[i + 1] << 32 | h[i]) << up) >> 32));
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (uint32_t o = DC_BLOCK_BYTES * lane; o < heads_padded; o += DC_BLOCK_BYTES * 64)
        *reinterpret_cast<u32x4 *>(out + heads_at + o) = *(lds_u32x4 *)(uintptr_t)(stage + 16 + o);
}

template <int THREADS> void launch_emit(const EncArgs &a, hipStream_t stream)
{
    if (a.codec == DC_CODEC_TANS)
        hipLaunchKernelGGL((dc_emit_kernel<THREADS, DC_CODEC_TANS>), dim3((uint32_t)a.n_chunks), dim3(THREADS), 0, stream, a);
    else
        hipLaunchKernelGGL((dc_emit_kernel<THREADS, DC_CODEC_HUFFMAN>), dim3((uint32_t)a.n_chunks), dim3(THREADS), 0, stream, a);
}

bool enc_params_ok(const dc_params *p)
{
    if (!p) return false;
    if (p->chunk_bytes < 16 || p->chunk_bytes > DC_MAX_CHUNK_BYTES || p->chunk_bytes % 16) return false;
    if (p->n_streams != 32 && p->n_streams != 64 && p->n_streams != 128 && p->n_streams != 256) return false;
    if (p->codec == DC_CODEC_TANS ? p->n_streams < 64 : p->codec != DC_CODEC_HUFFMAN) return false;
    if (p->policy == DC_POLICY_BLOCK_LAST) return p->block_chunks != 0;
    if (p->policy == DC_POLICY_RAW_FRACTION) return p->raw_fraction >= 0.0f && p->raw_fraction <= 1.0f;
    return p->policy == DC_POLICY_ALL_HUFF || p->policy == DC_POLICY_AUTO;
}

uint64_t align256(uint64_t x) { return (x + 255) & ~255ull; }

} // namespace

extern "C" int dc_compress_chunks_dev_workspace(uint64_t raw_bytes, const dc_params *params, uint64_t *workspace_bytes)
{
    if (!enc_params_ok(params) || raw_bytes == 0 || !workspace_bytes) return DC_E_ARG;
    if (params->format != DC_FORMAT_ID) return DC_E_FORMAT;
    const uint64_t nc = (raw_bytes + params->chunk_bytes - 1) / params->chunk_bytes;
    *workspace_bytes = align256(nc * 256) + align256(nc * params->n_streams * 4) + align256(nc * 4);
    // tANS: the frequencies, the first states and the items besides.  Of the 32 bytes for every group of 16 the items take 24 (item_place); the
    // size stays what callers have set aside, and what the fixed workspace below refuses stays refused.
    if (params->codec == DC_CODEC_TANS)
        *workspace_bytes += align256(nc * 512) + align256(nc * params->n_streams * 2) + align256(nc * params->chunk_bytes * 2);
    return DC_OK;
}

namespace {

// The two or three launches of the compression, with the workspace (code lengths, sub-stream sizes and payload
// sizes between them) wherever the caller of this function has it.
int compress_chunks_on_stream(const int8_t *src_dev, uint64_t raw_bytes, const dc_params *params, uint8_t *blob_dev,
                              uint64_t blob_cap, dc_chunk *table_dev, uint64_t table_cap, void *workspace_dev,
                              uint64_t workspace_bytes, uint64_t *result_dev, void *hip_stream)
{
    uint64_t need = 0;
    if (const int rc = dc_compress_chunks_dev_workspace(raw_bytes, params, &need)) return rc;
    if (!src_dev || !blob_dev || !table_dev || !workspace_dev || !result_dev) return DC_E_ARG;
    if ((reinterpret_cast<uintptr_t>(src_dev) & 15u) || (reinterpret_cast<uintptr_t>(blob_dev) & 15u) ||
        (reinterpret_cast<uintptr_t>(table_dev) & 7u) || (reinterpret_cast<uintptr_t>(workspace_dev) & 15u) ||
        (reinterpret_cast<uintptr_t>(result_dev) & 7u))
        return DC_E_ARG;
    const uint64_t nc = (raw_bytes + params->chunk_bytes - 1) / params->chunk_bytes;
    if (nc > 0x7FFFFFFFull) return DC_E_ARG;
    if (workspace_bytes < need || table_cap < nc) return DC_E_CAP;
    EncArgs a = {};
    a.src = reinterpret_cast<const uint8_t *>(src_dev);
    a.raw_bytes = raw_bytes;
    a.n_chunks = nc;
    a.chunk_bytes = params->chunk_bytes;
    a.S = params->n_streams;
    a.policy = params->policy;
    a.block_chunks = params->block_chunks;
    a.n_raw = 0;
    if (params->policy == DC_POLICY_RAW_FRACTION) {
        a.n_raw = (uint64_t)((double)params->raw_fraction * (double)nc + 0.5);
        if (a.n_raw > nc) a.n_raw = nc;
    }
    uint8_t *ws = static_cast<uint8_t *>(workspace_dev);
    a.lens = ws;
    a.bits = reinterpret_cast<uint32_t *>(ws + align256(nc * 256));
    a.comp = reinterpret_cast<uint32_t *>(ws + align256(nc * 256) + align256(nc * a.S * 4));
    a.codec = params->codec;
    if (a.codec == DC_CODEC_TANS) {
        uint8_t *more = ws + align256(nc * 256) + align256(nc * a.S * 4) + align256(nc * 4);
        a.freq = reinterpret_cast<uint16_t *>(more);
        a.first = reinterpret_cast<uint16_t *>(more + align256(nc * 512));
        a.items = more + align256(nc * 512) + align256(nc * a.S * 2);
    }
    a.blob = blob_dev;
    a.blob_cap = blob_cap;
    a.table = table_dev;
    a.result = result_dev;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (a.codec == DC_CODEC_TANS) hipLaunchKernelGGL(dc_tans_model_kernel, dim3((uint32_t)nc), dim3(256), 0, stream, a);
    else hipLaunchKernelGGL(dc_codes_kernel, dim3((uint32_t)nc), dim3(256), 0, stream, a);
    // (The layout kernel has read all sizes when it writes; a workgroup of the coder writes its entry, its payload and, the last one, the
    // result words while others still add sizes up.)
    auto over_workspace = [&](const void *p, uint64_t bytes) {
        const uintptr_t at = reinterpret_cast<uintptr_t>(p), w = reinterpret_cast<uintptr_t>(workspace_dev);
        return at < w + need && w < at + bytes;
    };
    a.placed = nc > kOwnLayoutChunks || a.n_raw > 0 || over_workspace(result_dev, 16) || over_workspace(blob_dev, blob_cap) ||
               over_workspace(table_dev, nc * sizeof(dc_chunk));
    if (a.placed) hipLaunchKernelGGL(dc_layout_kernel, dim3(1), dim3(kLayoutThreads), 0, stream, a);
    switch (a.S) {
    case 32:
    case 64: launch_emit<64>(a, stream); break;
    case 128: launch_emit<128>(a, stream); break;
    default: launch_emit<256>(a, stream); break;
    }
    return dc_launch_status();
}

} // namespace

extern "C" int dc_compress_chunks_dev(const int8_t *src_dev, uint64_t raw_bytes, const dc_params *params,
                                      uint8_t *blob_dev, uint64_t blob_cap, dc_chunk *table_dev, uint64_t table_cap,
                                      void *workspace_dev, uint64_t workspace_bytes, uint64_t *result_dev,
                                      void *hip_stream)
{
    return compress_chunks_on_stream(src_dev, raw_bytes, params, blob_dev, blob_cap, table_dev, table_cap, workspace_dev,
                                     workspace_bytes, result_dev, hip_stream);
}

// ---- the same call for callers that cannot allocate: the workspace is a fixed array in device memory

// Workspace of dc_compress_chunks_dev_static.  One copy per GPU that runs the library, held until the
// process ends.  In host code this name only stands for the array: its address on the current device comes
// from hipGetSymbolAddress (static_scratch below), and only that address is handed to kernels.
static __device__ __align__(256) uint8_t scratch[DC_STATIC_SCRATCH_BYTES];

namespace {

std::mutex g_scratch_lock;
void *g_scratch_of_device[kMaxDevices]; // address of `scratch` on every device that has asked for it

// Address of the workspace array on the current device (looked up once per device), or null with the HIP
// status noted for dc_last_hip_error().
void *static_scratch()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        dc_launch_status();
        return nullptr;
    }
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_of_device[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            dc_launch_status();
            return nullptr;
        }
        g_scratch_of_device[dev] = p;
    }
    return g_scratch_of_device[dev];
}

} // namespace

extern "C" int dc_compress_chunks_dev_static(const int8_t *src_dev, uint64_t raw_bytes, const dc_params *params,
                                             uint8_t *blob_dev, uint64_t blob_cap, dc_chunk *table_dev,
                                             uint64_t table_cap, uint64_t *result_dev, void *hip_stream)
{
    uint64_t need = 0;
    if (const int rc = dc_compress_chunks_dev_workspace(raw_bytes, params, &need)) return rc;
    if (need > DC_STATIC_SCRATCH_BYTES) return DC_E_CAP; // the input is beyond what the fixed workspace serves
    void *ws = static_scratch();
    if (!ws) return DC_E_HIP;
    return compress_chunks_on_stream(src_dev, raw_bytes, params, blob_dev, blob_cap, table_dev, table_cap, ws,
                                     DC_STATIC_SCRATCH_BYTES, result_dev, hip_stream);
}
