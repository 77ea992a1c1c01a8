// Device side of libentro: segment-parallel Huffman decode for gfx950 with
// fused dequantisation and a fused batch-1 matrix-vector product.
//
// EntroLLM ("Segmentation for parallel Huffman decoding", Fig. 3) cuts the
// encoded parameter space into segments with known boundaries and decodes
// them independently; here a segment is a fixed number of symbols and one
// GPU lane owns one segment, so a workgroup of W lanes decodes W consecutive
// segments of one tensor with one shared set of lookup tables in LDS.
// Launches over few segments let several lanes share one (k_shared, below).
//
// Data flow of the decode / dequant kernels, per lane:
//   HBM --128-byte lines (GEMV: 64)--> registers --between output blocks--> 128-byte ring in LDS
//   ring --three dwords--> 63-bit window --14 bits--> first-level table (LDS,
//   16-bit entries: length | symbol) --shift by the entry--> next code ...
//   four symbols --one aligned dword--> the lane's row of the wave's LDS tile
//   tile rows --dequantise / pack, row-wise--> HBM,
// so that every global store instruction of a wave covers whole rows (the GEMV
// has no tile: a lane multiplies its four symbols into x as they come).  All 64
// lanes of a wave decode in step, four symbols per window: no lane waits for
// another, nothing is written to LDS at an odd address, and a flush happens
// after a fixed number of groups.  The symbol loop has no branch per lookup; a
// lane that meets a code too long for the first-level table stops moving for the
// rest of its group, and the wave then finishes that group for it with the
// second-level table or a canonical search.
#include "entro.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <numeric>
#include <string>
#include <type_traits>
#include <vector>

// Partial sums of entro_decode_gemv_static: two floats per segment.  Every GPU the library runs on holds
// its own copy of this array until the process ends.  In host code the name stands for the symbol only;
// the array's address on a device comes from hipGetSymbolAddress (static_scratch below).
static __device__ __align__(256) float scratch[2 * ENTRO_STATIC_GEMV_MAX_SEGMENTS];

namespace {

constexpr int kL1 = 14;                  // stream bits that index the first-level table
constexpr uint32_t kL1Mask = (1u << kL1) - 1u;
constexpr int kL2Cap = 512;              // second-level entries (all long prefixes together)
constexpr int kL2MaxBits = 6;            // the second level resolves codes of up to kL1 + 6 = 20 bits
constexpr int kL2MaxPrefixes = 32;       // more long prefixes than this: second level unused (32 blocks of 16 fill it)
constexpr int kSingleBits = 9;             // pair tables: index bits of the table of single codes
constexpr int kSmallBits = 10;           // index bits that the first level is searched for; longer codes are filled in afterwards
constexpr uint32_t kUnit = 64;           // segments a wavefront decodes at a time: one per lane
constexpr int kGroup = 4;                // symbols per ring read: 63 valid bits >= 4 * 14
constexpr uint32_t kTailShift = 4;       // a stretch's last round is drawn with lanes up to 2^this times finer
constexpr int kTripGroups = 4;           // ring reads between two checks of the ring's fill
constexpr int kScalarProbes = 2;         // scalar reader: symbols per 64-bit load, 33 valid bits >= 2 * kL1
constexpr int kRingBits = 1024;          // a lane's ring: two 64-byte lines (eight 16-byte blocks)
constexpr int kRingDwords = kRingBits / 32 + 2;   // and two mirror dwords
constexpr int kRing2Bits = 512;          // the short ring: four blocks
constexpr int kRing2Dwords = kRing2Bits / 32 + 2;
constexpr int kGroupBits = kGroup * kL1;           // most stream bits a group takes through the first level
constexpr int kTripBits = (kTripGroups - 1) * kGroupBits + 64;   // a trip's last ring read ends this far past its start
constexpr uint32_t kMaxChunkSymbols = 1u << 20;
static_assert(kGroup * kL1 <= 63 && kGroup == 4, "a group packs four symbol bytes into one dword");

// What the kernels read about one tensor.  Lives in kernel arguments (single
// tensor calls) or in the workspace table (batched calls).
struct DevTensor {
    const uint8_t *stream;
    const uint64_t *offsets;
    void *out;
    const uint16_t *x;
    float *partials;            // GEMV: head/tail partial sums, 2 per segment
    const uint16_t *sub;        // entry points inside the segments: stream bits of every piece (or null)
    void *tables;               // batched launches: the tensor's lookup tables as k_tables left them
    uint64_t n;
    uint32_t stream_bytes;
    uint32_t chunk_symbols;     // symbols one lane decodes: a piece, where the tensor has entry points or they are found on the way, else a segment
    uint32_t n_chunks;          // and how many of those the tensor has
    uint32_t sub_shift;         // log2 of lanes per segment (0: a lane takes a whole segment; sub null: they find their starts themselves)
    uint32_t sub_merge;         // log2 of the pieces of the entry-point table that one lane takes
    uint32_t rows;
    uint32_t cols;
    uint32_t bits;
    float scale;
    int32_t zero_point;
    uint32_t max_len;
    uint32_t need_fix;
    uint32_t row_lanes;         // GEMV: lanes per matrix row where a wavefront sums its rows by itself (0: not so)
    uint32_t fine;              // batched launches: index of the same tensor's description with finer lanes (0: none)
    uint32_t fine_shift;        // log2 of how many of those lanes make one of this description's
    uint32_t fix_symbols;       // GEMV: symbols per pair of partial sums: a lane's, or a unit's where lanes share segments
    uint32_t share_shift;       // k_shared*: log2 of the lanes that share a segment (or piece)
    uint32_t share_per;         // segments of a unit, at most 64 >> share_shift (0: the tensor does not go there)
    uint32_t share_units;       // units of the tensor
    uint32_t flat_len;          // k_single on a code of nearly one length: the least length,
    uint32_t flat_last[3];      // and the last value, of 32 stream bits in code order, that begins with a code of up to flat_len + 0, 1, 2 bits
    uint32_t *fine_index;       // k_fine: where the chains of every lane begin (workspace)
    uint32_t fine_len;          // symbols of a lane, a multiple of 8 up to 64 (0: the tensor does not go there)
    uint32_t fine_first;        // of them its first chain's
    uint32_t fine_n;            // lanes of the tensor
    uint32_t fine_pieces;       // pieces of chunk_symbols symbols in a unit of 64 lanes
    uint32_t fine_rows;         // how rows come about: kFineRow, kFineUnits, kFineParts
    uint32_t fine_units;        // units that a wavefront takes one after the other: a row's, or one
    uint32_t fine_quanta;       // how many of those the tensor has
    uint32_t fine_item;         // and how many of them are a work item
    uint8_t len[256];
};

struct WorkItem {
    uint32_t tensor;
    uint32_t first;             // first segment (main kernels) or first row (second-stage sum)
};

// The P modes are the byte, fp32 and bf16 outputs and the GEMV of launches whose tensors all hold
// 4-bit symbols: they decode two symbols per lookup, like the packed output.
// The W modes are the GEMV on wide tables (8-bit symbols, zero-point within [-1, 256]): gemv_direct2.
enum Mode { kModeU8 = 0, kModeU4 = 1, kModeF32 = 2, kModeBF16 = 3, kModeGemvF32 = 4, kModeGemvBF16 = 5,
            kModeU8P = 6, kModeF32P = 7, kModeBF16P = 8, kModeGemvF32P = 9, kModeGemvBF16P = 10,
            kModeGemvF32W = 11, kModeGemvBF16W = 12 };
constexpr bool gemv_f32(int mode) { return mode == kModeGemvF32 || mode == kModeGemvF32P || mode == kModeGemvF32W; }
constexpr bool is_gemv(int mode) {
    return gemv_f32(mode) || mode == kModeGemvBF16 || mode == kModeGemvBF16P || mode == kModeGemvBF16W;
}
constexpr bool wide_gemv(int mode) { return mode == kModeGemvF32W || mode == kModeGemvBF16W; }
// the output format of a mode
constexpr int base_mode(int mode) { return mode == kModeU8P ? kModeU8 : mode == kModeF32P ? kModeF32 : mode == kModeBF16P ? kModeBF16 : mode; }

// Per output mode: symbols of a lane that one flush takes, bytes of its tile row
// (one per table lookup: a symbol, or two 4-bit symbols already packed), waves
// per workgroup (what fits into the 160 KB of LDS), tile bytes one lane consumes
// per flush pass (a 16-byte store for all but fp32) and bytes that a row becomes
// in memory.  The host glue sizes its launches with the same numbers.  The GEMV
// has no tile (only spb, the symbols between two ring refills, and waves count).
template <int MODE> struct Cfg;
template <> struct Cfg<kModeU8> { static constexpr int spb = 64, row = 64, waves = 14, piece = 16, out_row = 64; };
template <> struct Cfg<kModeU4> { static constexpr int spb = 128, row = 64, waves = 14, piece = 16, out_row = 64; };
template <> struct Cfg<kModeF32> { static constexpr int spb = 64, row = 64, waves = 16, piece = 8, out_row = 256; };
template <> struct Cfg<kModeBF16> { static constexpr int spb = 64, row = 64, waves = 16, piece = 8, out_row = 128; };
template <> struct Cfg<kModeGemvF32> { static constexpr int spb = 64, row = 64, waves = 14, piece = 8, out_row = 0; };
template <> struct Cfg<kModeGemvBF16> { static constexpr int spb = 64, row = 64, waves = 14, piece = 8, out_row = 0; };
template <> struct Cfg<kModeGemvF32P> { static constexpr int spb = 128, row = 64, waves = 14, piece = 8, out_row = 0; };
template <> struct Cfg<kModeGemvBF16P> { static constexpr int spb = 128, row = 64, waves = 14, piece = 8, out_row = 0; };
template <> struct Cfg<kModeGemvF32W> { static constexpr int spb = 64, row = 64, waves = 16, piece = 8, out_row = 0; };
template <> struct Cfg<kModeGemvBF16W> { static constexpr int spb = 64, row = 64, waves = 16, piece = 8, out_row = 0; };
template <> struct Cfg<kModeU8P> { static constexpr int spb = 128, row = 64, waves = 14, piece = 16, out_row = 128; };
template <> struct Cfg<kModeF32P> { static constexpr int spb = 128, row = 64, waves = 14, piece = 8, out_row = 512; };
template <> struct Cfg<kModeBF16P> { static constexpr int spb = 128, row = 64, waves = 14, piece = 8, out_row = 256; };
// Packed 4-bit output decodes two symbols per lookup, and so do the P modes.
template <int MODE> constexpr bool kPairMode = MODE == kModeU4 || MODE == kModeU8P || MODE == kModeF32P || MODE == kModeBF16P ||
                                               MODE == kModeGemvF32P || MODE == kModeGemvBF16P;

// Lookup tables of one workgroup (LDS).
// Entry (16 bits): bits 0..5 the code's length, bits 8..15 its symbol, so that an
// entry serves as a 64-bit shift amount as it stands.
// First level: indexed by the next kL1 stream bits.  A zero length marks a prefix
// whose code is longer than kL1 bits (a lane that looks one up does not move);
// the whole low byte is zero then, bits 8..10 are the depth of the prefix's block
// in the second level (7: it has none) and bits 11..15 the block's start in units
// of sixteen entries.
// Second level: per long prefix a block indexed by the following `depth` stream
// bits; zero there sends the lane to the canonical search
// (first / cnt / offs / sorted).
// Pair tables (packed 4-bit output): a first-level entry holds the next TWO codes
// where both fit into the kL1 index bits, their lengths added up and the two
// symbols packed the way the output wants them (first one in the low nibble); a
// zero entry otherwise.  There is no second level then; lut2 starts with a
// table of single codes up to kSingleBits long instead, for what the pair table
// leaves out and for the element-by-element paths.
struct alignas(16) TablesTail {
    uint16_t lut2[kL2Cap];
    uint32_t cnt[ENTRO_MAX_CODE_LEN + 2];
    uint32_t first[ENTRO_MAX_CODE_LEN + 2];
    uint32_t offs[ENTRO_MAX_CODE_LEN + 2];
    uint32_t pdepth[kL2MaxPrefixes];     // per long prefix: bits its second-level block resolves
    uint32_t pbase[kL2MaxPrefixes];      // and where the block starts (a multiple of 16)
    uint32_t first_prefix;               // smallest kL1-bit prefix of a long code; 2^kL1 if level 2 is unused
    uint32_t long_start;                 // the same, but kept when level 2 is unused
    uint32_t pad[2];
    uint8_t sorted[256];
};
// E: the first level's entry.  16 bits: as described above.  32 bits (the GEMV's wide tables): the same in the
// low half and, in the high half, the value the symbol contributes, ready for use: bf16(symbol - zero_point),
// which is exact (an integer of at most 256 in magnitude), so that the product needs neither a conversion
// nor a subtraction per symbol.  A window that is to index 32-bit entries carries two stale low bits.
template <class E>
struct alignas(16) TablesT : TablesTail {
    static constexpr uint32_t stale = sizeof(E) == 2 ? 1u : 2u;
    E lut[1 << kL1];
};
using Tables = TablesT<uint16_t>;
using Tables32 = TablesT<uint32_t>;

// Per-wave LDS: the lanes' stream rings and their output rows.
// The ring is stored dword-major (dword d of lane l at d * 64 + l): whatever
// dword each lane reads, lane l stays on bank l % 32.  A tile row holds the ROW
// symbol bytes a lane decodes between two flushes.  Rows have no padding; row r
// is rotated by tile_rot(r) dwords instead, which spreads over all banks both
// the writes (all lanes write the same dword of their rows at the same time) and
// the row-wise reads of the flush.
template <int ROW>
struct alignas(256) WaveMem {
    static constexpr int row_dwords = ROW / 4;
    static_assert(row_dwords == 16 || row_dwords == 32, "the rotation below is made for these");
    uint32_t ring[kRing2Dwords * 64];
    uint32_t tile[64 * row_dwords];
    // rows of 16 dwords alternate between the two halves of the 32 banks, so pairs of rows share a rotation
    static __device__ __forceinline__ uint32_t tile_rot(uint32_t row) { return row_dwords == 16 ? row >> 1 : row; }
    // where dword j of row `row` lives
    static __device__ __forceinline__ uint32_t tile_at(uint32_t row, uint32_t j) {
        return row * row_dwords + ((j + tile_rot(row)) & (row_dwords - 1));
    }
};

// Per-wave LDS of the kernels that use the short ring: 64 bytes of stream per lane and rows of 32
// symbol bytes.  Row r is rotated by 2 * ((r >> 2) & 3) dwords, which keeps its dword pairs aligned
// and spreads rows four apart (which start on the same bank) over the banks.
struct alignas(256) WaveMem2 {
    static constexpr int row_dwords = 8;
    uint32_t ring[18 * 64];
    uint32_t tile[64 * row_dwords];
    static __device__ __forceinline__ uint32_t tile_at(uint32_t row, uint32_t j) {
        return row * row_dwords + ((j + 2u * ((row >> 2) & 3u)) & (row_dwords - 1));
    }
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef const u32x4 __attribute__((address_space(1))) *global_u4_ptr;
typedef u32x4 __attribute__((address_space(1))) *global_u4_wptr;
typedef u32x2 __attribute__((address_space(1))) *global_u2_wptr;
typedef const uint64_t __attribute__((address_space(1))) *global_u64_ptr;
typedef const uint16_t __attribute__((address_space(1))) *global_u16_ptr;
// LDS pointers with the address space spelled out: the accesses compile to plain
// ds_ instructions with 32-bit addresses
typedef volatile uint32_t __attribute__((address_space(3))) *lds_v32;
typedef const uint32_t __attribute__((address_space(3))) *lds_p32;

__device__ __forceinline__ uint32_t bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

__device__ __forceinline__ float dequant(uint32_t sym, int32_t z, float s) {
    return static_cast<float>(static_cast<int32_t>(sym) - z) * s;
}

__device__ __forceinline__ uint32_t pack_entry(uint32_t sym, uint32_t len) { return len | (sym << 8); }
__device__ __forceinline__ uint32_t entry_len(uint32_t e) { return e & 0x3fu; }
__device__ __forceinline__ uint32_t entry_sym(uint32_t e) { return (e >> 8) & 0xffu; }

// The eight 4-bit symbols of four pair bytes, one per byte, in order.
__device__ __forceinline__ void unpack_nibbles(uint32_t d, uint32_t &lo, uint32_t &hi) {
    const uint32_t even = d & 0x0f0f0f0fu, odd = (d >> 4) & 0x0f0f0f0fu;   // symbols 0, 2, 4, 6 and 1, 3, 5, 7
    lo = __builtin_amdgcn_perm(odd, even, 0x05010400u);
    hi = __builtin_amdgcn_perm(odd, even, 0x07030602u);
}

__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Tables that a launch's preparation has built, from memory into LDS by the whole workgroup of WG lanes: every lane asks for
// its 16-byte pieces at once.
// (In a loop each step waited for its piece, four or five times the way to the L2 and back.)  Measured, loop -> now: step over
// 32 layers of 4-bit products 4086 -> 4036 us; launches of longer stretches do not notice (24-layer set to bytes 804).
template <uint32_t BYTES, uint32_t WG>
__device__ __forceinline__ void copy_tables(void *dst, const void *src) {
    static_assert(BYTES % 16 == 0, "16-byte pieces");
    constexpr uint32_t N = BYTES / 16u, STEPS = (N + WG - 1u) / WG;
    u32x4 v[STEPS];
#pragma unroll
    for (uint32_t i = 0; i < STEPS; ++i) {
        const uint32_t j = i * WG + threadIdx.x;
        v[i] = ((global_u4_ptr)src)[j < N ? j : N - 1u];
    }
#pragma unroll
    for (uint32_t i = 0; i < STEPS; ++i) {
        const uint32_t j = i * WG + threadIdx.x;
        if (j < N) static_cast<u32x4 *>(dst)[j] = v[i];
    }
}

// Canonical code tables and both lookup levels, built from the 256 (or 16)
// code lengths by the whole workgroup of WG >= 256 lanes (four waves hold the
// symbols).  `wcnt` is scratch of 4 * 33 words.
// A small launch waits for this, so little in it is serial: one wavefront turns the counts
// into the canonical tables with its lanes as the lengths (running sums by DPP), and
// the first level is resolved for kSmallBits index bits only, copied to the indexes that end in
// the same bits, and searched bit by bit for the few indexes that start with a longer code.
// Pair tables resolve every index, with two reads of the small table of single codes.
// L2 false: without the second level (k_shared goes to the canonical tables for the codes that its table does not hold).
// 4096 x 4096 without entry points to bf16 32.8 -> 31.9 us, its product 31.3 -> 30.5, 2048 x 2048 to bytes 24.5 -> 23.8.
// Measured as the whole call: one tensor of 2048 symbols to fp32 33.6 -> 22.0 us, 4 M symbols to
// bytes 42.6 -> 30.6 us, against a search over all 14 lengths for every index.
template <int WG, bool PAIR, bool L2 = true, class TB>
__device__ __forceinline__ void build_tables(const DevTensor &t, TB &tb, uint32_t *wcnt) {
    static_assert(WG >= 256, "one lane per symbol");
    constexpr uint32_t kLens = ENTRO_MAX_CODE_LEN + 1;
    typedef std::remove_reference_t<decltype(tb.lut[0])> Entry;
    const uint32_t tid = threadIdx.x;
    const uint32_t wave = tid >> 6;
    const uint32_t max_len = t.max_len;
    const uint32_t l = tid < 256 ? t.len[tid] : 0u;
    if constexpr (L2) {
        if (tid < kL2MaxPrefixes) tb.pdepth[tid] = 0;
        for (uint32_t i = tid; i < kL2Cap; i += WG) tb.lut2[i] = 0;
    }
    // symbols of each length per wave, and every symbol's place among those of its length in its wave
    uint32_t rank = 0;
    if (tid < 256) {
        // one step for each length that occurs among the wavefront's symbols
        if ((tid & 63u) < kLens) wcnt[wave * kLens + (tid & 63u)] = 0;
        wave_sync_lds();
        uint64_t open = __builtin_amdgcn_ballot_w64(l != 0);
        while (open) {
            const uint32_t b = __builtin_amdgcn_readlane(l, static_cast<uint32_t>(__builtin_ctzll(open)));
            const uint64_t m = __builtin_amdgcn_ballot_w64(l == b);
            if (l == b) rank = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
            if ((tid & 63u) == 0) wcnt[wave * kLens + b] = static_cast<uint32_t>(__builtin_popcountll(m));
            open &= ~m;
        }
    }
    __syncthreads();
    if (tid < 64) {
        // lane b: the symbols of length b, those of the lengths below and the first code of length b
        const uint32_t b = tid;
        const uint32_t mine = b >= 1 && b <= max_len ? wcnt[b] + wcnt[kLens + b] + wcnt[2 * kLens + b] + wcnt[3 * kLens + b] : 0u;
        // Code space taken by the shorter codes, in units of 2^-32 (Kraft's inequality keeps it within 33 bits): the first code of
        // length b is its upper b bits.  Both sums over the lanes in front by DPP (lanes 0 to 33: rows of sixteen, then the row
        // totals); one length after the other, with each length's count read from its lane, they took 1.3 us.
        const uint32_t sh = b <= ENTRO_MAX_CODE_LEN ? ENTRO_MAX_CODE_LEN - b : 0u;
        const uint64_t space = static_cast<uint64_t>(mine) << sh;
        uint64_t upto = space;
        uint32_t below = mine;
        auto in_front = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
            constexpr int C = decltype(ctrl)::value, R = decltype(rows)::value;
            const uint32_t lo = __builtin_amdgcn_update_dpp(0u, static_cast<uint32_t>(upto), C, R, 0xf, true);
            const uint32_t hi = __builtin_amdgcn_update_dpp(0u, static_cast<uint32_t>(upto >> 32), C, R, 0xf, true);
            below += __builtin_amdgcn_update_dpp(0u, below, C, R, 0xf, true);
            upto += (static_cast<uint64_t>(hi) << 32) | lo;
        };
        typedef std::integral_constant<int, 0xf> AllRows;
        in_front(std::integral_constant<int, 0x111>{}, AllRows{});                      // row_shr:1, 2, 4, 8
        in_front(std::integral_constant<int, 0x112>{}, AllRows{});
        in_front(std::integral_constant<int, 0x114>{}, AllRows{});
        in_front(std::integral_constant<int, 0x118>{}, AllRows{});
        in_front(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast:15, :31
        in_front(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
        const uint32_t first = static_cast<uint32_t>((upto - space) >> sh) << (b == ENTRO_MAX_CODE_LEN + 1 ? 1u : 0u), off = below - mine;
        if (b <= ENTRO_MAX_CODE_LEN + 1) {
            tb.cnt[b] = mine;
            tb.first[b] = first;
            tb.offs[b] = off;
        }
        // canonical codes grow with length, so the long codes own the kL1-bit prefixes from the
        // first long code's on
        const uint64_t longer = __builtin_amdgcn_ballot_w64(mine != 0 && b > static_cast<uint32_t>(kL1));
        uint32_t long_start = 1u << kL1;
        if (longer) {
            const uint32_t b0 = static_cast<uint32_t>(__builtin_ctzll(longer));
            long_start = __builtin_amdgcn_readlane(first, b0) >> (b0 - kL1);
        }
        if (tid == 0) {
            tb.long_start = long_start;
            tb.first_prefix = (1u << kL1) - long_start > static_cast<uint32_t>(kL2MaxPrefixes) ? 1u << kL1 : long_start;
        }
    }
    __syncthreads();
    uint32_t code = 0;
    const uint32_t first_prefix = tb.first_prefix;
    const bool have_l2 = L2 && !PAIR && first_prefix < (1u << kL1);
    if (l) {
        for (uint32_t w = 0; w < wave; ++w) rank += wcnt[w * kLens + l];
        code = tb.first[l] + rank;
        tb.sorted[tb.offs[l] + rank] = static_cast<uint8_t>(tid);
        if (l > kL1 && have_l2) atomicMax(&tb.pdepth[(code >> (l - kL1)) - first_prefix], l - kL1);
    }
    __syncthreads();
    if (tid < 64 && have_l2) {
        // every long prefix (one lane each) gets a block of 2^min(depth, cap) entries; lower the cap until all fit
        const uint32_t n_prefix = (1u << kL1) - first_prefix;
        const uint32_t depth = tid < n_prefix ? tb.pdepth[tid] : 0u;
        uint32_t cap = kL2MaxBits, d = 0, upto = 0;
        for (;; --cap) {
            d = depth < cap ? depth : cap;
            const uint32_t size = tid < n_prefix ? (d < 4 ? 16u : 1u << d) : 0u;
            upto = size;                                     // inclusive prefix sum of the blocks' sizes
#pragma unroll
            for (uint32_t m = 1; m < static_cast<uint32_t>(kL2MaxPrefixes); m <<= 1) {
                const uint32_t y = __shfl_up(upto, m, 64);
                upto += tid >= m ? y : 0u;
            }
            const uint32_t total = __builtin_amdgcn_readlane(upto, kL2MaxPrefixes - 1);
            upto -= size;
            if (total <= static_cast<uint32_t>(kL2Cap) || cap == 0) break;
        }
        if (tid < n_prefix) {
            tb.pdepth[tid] = d;
            tb.pbase[tid] = upto;
        }
    }
    __syncthreads();
    // second level: every long symbol fills the slots of its block that start with its code
    if (l > kL1 && have_l2) {
        const uint32_t extra = l - kL1;
        const uint32_t prefix = code >> extra;
        const uint32_t depth = tb.pdepth[prefix - first_prefix];
        const uint32_t base = tb.pbase[prefix - first_prefix];
        if (extra <= depth) {
            const uint16_t e = static_cast<uint16_t>(pack_entry(tid, l));
            const uint32_t suffix = code & ((1u << extra) - 1u);
            const uint32_t rev = __brev(suffix) >> (32 - extra);
            for (uint32_t i = rev; i < (1u << depth); i += (1u << extra)) tb.lut2[base + i] = e;
        }
        // longer codes keep the zero entry: canonical search
    }
    // The code of LO to HI bits that the first HI bits of `v` (code order) start with: its length (0: none) and its
    // place among the sorted symbols.  The limits sit in scalar registers.
    uint32_t fb[kL1 + 1], cb[kL1 + 1], ob[kL1 + 1];
#pragma unroll
    for (int b = 1; b <= kL1; ++b) {
        fb[b] = __builtin_amdgcn_readfirstlane(tb.first[b]);
        cb[b] = __builtin_amdgcn_readfirstlane(tb.cnt[b]);
        ob[b] = __builtin_amdgcn_readfirstlane(tb.offs[b]);
    }
    auto search = [&](auto lo_tag, auto hi_tag, uint32_t v, uint32_t &idx) __attribute__((always_inline)) {
        constexpr int LO = decltype(lo_tag)::value, HI = decltype(hi_tag)::value;
        uint32_t len = 0;
        idx = 0;
#pragma unroll
        for (int b = LO; b <= HI; ++b) {
            const uint32_t d = (v >> (HI - b)) - fb[b];
            const bool hit = d < cb[b];                       // at most one length matches
            len = hit ? static_cast<uint32_t>(b) : len;
            idx = hit ? ob[b] + d : idx;
        }
        return len;
    };
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, kL1> Full;
    if constexpr (PAIR) {
        // single codes of up to kSingleBits bits; zero: longer, or no code at all
        typedef std::integral_constant<int, kSingleBits> Single;
        typedef std::integral_constant<int, kSingleBits + 1> Longer;
        for (uint32_t i = tid; i < (1u << kSingleBits); i += WG) {
            uint32_t idx;
            const uint32_t len = search(One{}, Single{}, __brev(i) >> (32 - kSingleBits), idx);
            tb.lut2[i] = static_cast<uint16_t>(len ? pack_entry(tb.sorted[idx], len) : 0u);
        }
        __syncthreads();
        const uint32_t long_start = tb.long_start;
        // the code at the start of these kL1 index bits: out of that table, or a longer one by search (0: none)
        auto one = [&](uint32_t bits14) __attribute__((always_inline)) {
            uint32_t e = tb.lut2[bits14 & ((1u << kSingleBits) - 1u)];
            if (e == 0) {
                uint32_t idx;
                const uint32_t len = search(Longer{}, Full{}, __brev(bits14) >> (32 - kL1), idx);
                if (len) e = pack_entry(tb.sorted[idx], len);
            }
            return e;
        };
        for (uint32_t i = tid; i < (1u << kL1); i += WG) {
            // the first code (an index that starts no code moves one bit and gives symbol 0), then the code
            // that the remaining index bits spell (zeros behind them), if they hold all of it
            uint32_t a = one(i);
            if (a == 0 && (__brev(i) >> (32 - kL1)) < long_start) a = pack_entry(0, 1);
            uint32_t e = 0;
            if (a) {
                const uint32_t b = one(i >> entry_len(a));
                const uint32_t both = entry_len(a) + entry_len(b);
                if (b && both <= static_cast<uint32_t>(kL1)) e = pack_entry(entry_sym(a) | (entry_sym(b) << 4), both);
            }
            tb.lut[i] = static_cast<Entry>(e);
        }
    } else {
        typedef std::integral_constant<int, kSmallBits> Small;
        typedef std::integral_constant<int, kSmallBits + 1> Longer;
        auto entry_of = [&](uint32_t idx, uint32_t len) __attribute__((always_inline)) {
            uint32_t e = pack_entry(tb.sorted[idx], len);
            if constexpr (sizeof(Entry) == 4)           // wide entry: the centred symbol as bf16 in the high half
                e |= __float_as_uint(static_cast<float>(static_cast<int32_t>(tb.sorted[idx]) - t.zero_point)) & 0xffff0000u;
            return e;
        };
        for (uint32_t i = tid; i < (1u << kSmallBits); i += WG) {
            uint32_t idx;
            const uint32_t len = search(One{}, Small{}, __brev(i) >> (32 - kSmallBits), idx);
            tb.lut[i] = static_cast<Entry>(len ? entry_of(idx, len) : 0u);
        }
        __syncthreads();
        // sixteen bytes at a time to all indexes with the same low bits (those of longer codes are filled in below)
        constexpr uint32_t kSmallVecs = sizeof(Entry) << (kSmallBits - 4), kVecs = sizeof(Entry) << (kL1 - 4);
        u32x4 *vecs = reinterpret_cast<u32x4 *>(tb.lut);
        for (uint32_t j = kSmallVecs + tid; j < kVecs; j += WG) vecs[j] = vecs[j & (kSmallVecs - 1u)];
        __syncthreads();
        // codes of up to kSmallBits bits own the index values (in code order) in front of this one
        const uint32_t long_start = tb.long_start;
        for (uint32_t v = ((fb[kSmallBits] + cb[kSmallBits]) << (kL1 - kSmallBits)) + tid; v < (1u << kL1); v += WG) {
            uint32_t idx;
            const uint32_t len = search(Longer{}, Full{}, v, idx);
            // no match: the start of a longer code (the entry says where its second-level block is),
            // or, where a lone symbol leaves half of the code space unused, of none: symbol 0, one bit
            uint32_t e = pack_entry(0, 1);
            if (v >= long_start) {
                e = 7u << 8;
                if (L2 && v >= first_prefix) e = (tb.pdepth[v - first_prefix] << 8) | ((tb.pbase[v - first_prefix] >> 4) << 11);
            }
            if (len) e = entry_of(idx, len);
            tb.lut[__brev(v) >> (32 - kL1)] = static_cast<Entry>(e);
        }
    }
    __syncthreads();
}

// Canonical search over the lengths from `from` on.  `window` holds the next 32
// stream bits, first bit in bit 0.
__device__ __noinline__ uint32_t decode_canonical(const TablesTail &tb, uint32_t window, uint32_t from, uint32_t max_len) {
    const uint32_t v = __brev(window);
    for (uint32_t l = from; l <= max_len; ++l) {
        const uint32_t d = (v >> (32 - l)) - tb.first[l];
        if (d < tb.cnt[l]) return pack_entry(tb.sorted[tb.offs[l] + d], l);
    }
    return pack_entry(0, 1);        // not a code (corrupt stream): keep moving
}

// The code at the start of `window`, which the first level answered with the
// miss entry `miss`: second level (needs kL1 + kL2MaxBits valid bits).  Zero if
// the code is longer still.
__device__ __forceinline__ uint32_t lookup_l2(const TablesTail &tb, uint32_t miss, uint32_t window) {
    const uint32_t depth = (miss >> 8) & 7u;
    if (depth > static_cast<uint32_t>(kL2MaxBits)) return 0;
    return tb.lut2[(((miss >> 11) << 4) + __builtin_amdgcn_ubfe(window, kL1, depth)) & (kL2Cap - 1)];
}

// The same with the canonical search behind it; `window` holds the next 32 stream bits.
__device__ __forceinline__ uint32_t decode_long(const TablesTail &tb, uint32_t miss, uint32_t window, uint32_t max_len) {
    uint32_t e = lookup_l2(tb, miss, window);
    if (__builtin_expect(e == 0, 0)) e = decode_canonical(tb, window, kL1 + 1, max_len);
    return e;
}

// Pair tables: the single code at the start of `window` (the next 32 stream bits).
__device__ __forceinline__ uint32_t single_entry(const TablesTail &tb, uint32_t window, uint32_t max_len) {
    uint32_t e = tb.lut2[window & ((1u << kSingleBits) - 1u)];
    if (__builtin_expect(e == 0, 0)) e = decode_canonical(tb, window, kSingleBits + 1, max_len);
    return e;
}

// Stream bit at which a lane's piece k starts: the segment's offset, plus the lengths of the pieces in
// front of it in the same segment where the tensor has entry points inside its segments.
__device__ __forceinline__ uint64_t seg_start(const DevTensor &t, uint32_t k) {
    const uint32_t sh = t.sub_shift;
    const global_u64_ptr offsets = (global_u64_ptr)t.offsets;
    if (sh == 0) return offsets[k];
    const uint32_t c = k >> sh;
    const uint32_t before = (k - (c << sh)) << t.sub_merge;          // pieces of the segment in front of the lane's
    const global_u16_ptr sb = (global_u16_ptr)t.sub + (static_cast<uint64_t>(c) << (sh + t.sub_merge));
    const uint64_t base = offsets[c];
    // All fifteen are asked for at once, the segment's first entry in the place of those that the lane does not need: loads
    // under a condition each came back one after the other.  Measured, before -> now: 24-layer set to bytes 831 -> 799 us,
    // phi3-shaped 4-bit set to nibbles 882 -> 857, one layer of seven tensors validated and launched to bf16 194 -> 190, steps
    // over 32 layers of 8-bit products 6205 -> 6098 and of 4-bit products 4167 -> 4036.
    uint32_t len[ENTRO_MAX_SUB_PER_CHUNK - 1], add = 0;
#pragma unroll
    for (uint32_t i = 0; i + 1 < ENTRO_MAX_SUB_PER_CHUNK; ++i) len[i] = sb[i < before ? i : 0u];
#pragma unroll
    for (uint32_t i = 0; i + 1 < ENTRO_MAX_SUB_PER_CHUNK; ++i) add += i < before ? len[i] : 0u;
    return base + add;
}

// ---------------------------------------------------------------- scalar reader
// Reads straight from global memory, one symbol per lookup; used for segments
// whose size does not fit the row path and for shorter last segments.

// 64 stream bits starting at the dword that holds absolute stream bit `pos`,
// shifted so that bit pos is bit 0: at least 33 valid bits.  The read is
// clamped to the last 8 bytes of the (padded) stream.
__device__ __forceinline__ uint64_t load_bits(const uint8_t *stream, uint64_t pos, uint32_t last_off) {
    uint32_t off = static_cast<uint32_t>(pos >> 5) << 2;
    off = off < last_off ? off : last_off;
    const uint32_t *w = reinterpret_cast<const uint32_t *>(stream + off);
    const uint64_t v = static_cast<uint64_t>(w[0]) | (static_cast<uint64_t>(w[1]) << 32);
    return v >> (static_cast<uint32_t>(pos) & 31u);
}

struct ScalarReader {
    const uint8_t *stream;
    uint32_t last_off;   // stream_bytes - 8
    uint64_t pos;        // absolute stream bit
    uint64_t buf;
};

// The next symbol's entry from the scalar reader; r.buf must hold kL1 valid bits.
// With pair tables the table of single codes answers.
template <bool PAIR, class TB>
__device__ __forceinline__ uint32_t next_entry(ScalarReader &r, const TB &tb, uint32_t max_len) {
    uint32_t e = PAIR ? tb.lut2[static_cast<uint32_t>(r.buf) & ((1u << kSingleBits) - 1u)]
                      : tb.lut[static_cast<uint32_t>(r.buf) & kL1Mask];
    if (__builtin_expect(entry_len(e) == 0, 0)) {
        const uint32_t window = static_cast<uint32_t>(load_bits(r.stream, r.pos, r.last_off));
        e = PAIR ? decode_canonical(tb, window, kSingleBits + 1, max_len) : decode_long(tb, e, window, max_len);
        r.pos += entry_len(e);
        r.buf = load_bits(r.stream, r.pos, r.last_off);
    } else {
        r.buf >>= entry_len(e);
        r.pos += entry_len(e);
    }
    return e;
}

// ---------------------------------------------------------------- entry points found on the way
// Small launches on a tensor in long segments that carries no entry points (k_single with FIND; t.sub is null and
// t.sub_shift is the log2 of a segment's pieces).  A lane per segment leaves most of the device idle there, and the time is one lane's
// serial chain of lookups.  So 2^sub_shift lanes share a segment: each takes an equal stretch of its bits and decodes
// from a guessed bit, Huffman codes falling into step with the true code boundaries within a few codes.  Then a lane
// whose neighbour ended elsewhere than it began goes again from there, up to the first code boundary that it met the
// first time; from there on nothing changes but the count of its codes.  Lane 0 of a segment starts at a true
// boundary, so once all of them agree every start is true, whatever the data.  The lanes' symbol counts then say where
// each piece of chunk_symbols symbols begins, and the ordinary block path decodes the pieces.
// Data that does not fall into step (a run of one symbol inside a segment), data whose bits are spread too unevenly
// and offset tables that do not fit the stream show by the number of codes that they take: the wavefront then gives the
// search up, and the block path decodes its segments with one lane each, as it does without the search.
constexpr uint32_t kMarkBits = 256;      // stream bits from a lane's guess on in which its first pass marks the codes' starts
                                         // (of 211 000 lanes on weights 14 met one only behind 128 bits, none behind 192)

// What a wavefront of the decode kernels works on: lane l takes the symbols [(first + l) * symbols, + symbols) of the
// tensor, as long as first + l < end.
struct Unit {
    uint32_t first, end, symbols;
};

// At least 57 stream bits from absolute bit `pos` on (clamped to the padded stream's last 8 bytes): four lookups.
__device__ __forceinline__ uint64_t load_bits57(const DevTensor &t, uint64_t pos) {
    uint64_t off = pos >> 3;
    const uint64_t last = t.stream_bytes - 8u;
    off = off < last ? off : last;
    uint64_t v;
    __builtin_memcpy(&v, t.stream + off, 8);
    return v >> (static_cast<uint32_t>(pos) & 7u);
}

// Length of the code at the start of `w` (at least kL1 valid bits), which lies at absolute bit `pos`; moves w behind it.
template <bool PAIR, class TB>
__device__ __forceinline__ uint32_t step_code(const DevTensor &t, const TB &tb, uint64_t pos, uint64_t &w) {
    const uint32_t e = PAIR ? tb.lut2[static_cast<uint32_t>(w) & ((1u << kSingleBits) - 1u)] : tb.lut[static_cast<uint32_t>(w) & kL1Mask];
    uint32_t len = entry_len(e);
    if (__builtin_expect(len == 0, 0)) {
        const uint32_t window = static_cast<uint32_t>(load_bits57(t, pos));
        len = entry_len(PAIR ? decode_canonical(tb, window, kSingleBits + 1, t.max_len) : decode_long(tb, e, window, t.max_len));
        w = load_bits57(t, pos + len);
    } else {
        w >>= len;
    }
    return len;
}

// Stream bit at which the lane's piece of the unit starts (0: the lane has none).  Where the search is given up the unit
// becomes the same stretch of the tensor with a lane per segment.  `ring` is the wavefront's ring memory, not in use yet.
template <bool PAIR, class TB>
__device__ __forceinline__ uint64_t find_start(const DevTensor &t, const TB &tb, lds_v32 ring, Unit &u) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t sh = t.sub_shift, parts = 1u << sh, part = lane & (parts - 1u);
    const uint32_t S = u.symbols;
    const uint32_t seg = (u.first + lane) >> sh;                 // (a wavefront holds whole segments: parts <= 64)
    const bool live = (seg << sh) < u.end;
    uint64_t base = 0;
    uint32_t nsym = 0, span = 0;                                 // the segment's symbols and bits
    if (live) {
        const uint64_t whole = static_cast<uint64_t>(S) << sh, left = t.n - seg * whole;
        nsym = static_cast<uint32_t>(left < whole ? left : whole);
        base = t.offsets[seg];
        const uint64_t end = t.offsets[seg + 1], most = static_cast<uint64_t>(nsym) * ENTRO_MAX_CODE_LEN;
        const uint64_t bits = end > base ? end - base : 0;
        span = static_cast<uint32_t>(bits < most ? bits : most);
    }
    // the lane's stretch, in bits from the segment's start
    const uint32_t guess = static_cast<uint32_t>((static_cast<uint64_t>(span) * part) >> sh);
    const uint32_t limit = static_cast<uint32_t>((static_cast<uint64_t>(span) * (part + 1u)) >> sh);
    // bit b of dword d: a code of the first pass starts at guess + 32 * d + b
    const lds_v32 marks = ring + 64 + lane;
    auto mark_at = [&](uint32_t rel) __attribute__((always_inline)) { return (uint32_t __attribute__((address_space(3))) *)(marks + (rel >> 5) * 64u); };
#pragma unroll
    for (uint32_t d = 0; d < kMarkBits / 32u; ++d) marks[d * 64u] = 0;
    // first pass, four codes a trip: at most an eighth of the segment's symbols, where that is more than a quarter above
    // a piece's own (weights take up to 1.23 times a piece's symbols, 4-bit ones 1.39 times with 32 and 64 pieces)
    const uint32_t whole = S << sh, room = S + S / 4u + 16u;
    uint32_t upto = guess, count = 0;
    for (uint32_t trips = (whole / 8u > room ? whole / 8u : room) / 4u; trips != 0 && __builtin_amdgcn_ballot_w64(upto < limit) != 0; --trips) {
        if (upto < limit) {
            uint64_t w = load_bits57(t, base + upto);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (upto < limit) {
                    const uint32_t rel = upto - guess;
                    if (rel < kMarkBits) __hip_atomic_fetch_or(mark_at(rel), 1u << (rel & 31u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    upto += step_code<PAIR>(t, tb, base + upto, w);
                    ++count;
                }
        }
    }
    // rounds until every lane starts where its neighbour ended (one as a rule, as many as lanes at the most): together at
    // most 64 codes or, in long segments, one of 32 (the slowest lane of a wavefront takes up to 36 on weights)
    const uint32_t first_upto = upto, first_count = count;
    uint32_t from = guess, trips = (whole / 32u > 64u ? whole / 32u : 64u) / 4u;
    bool agreed = __builtin_amdgcn_ballot_w64(upto < limit) == 0;
    while (agreed) {
        const uint32_t before = __shfl_up(upto, 1, 64);
        const uint32_t want = part == 0 ? 0u : before;           // (never in front of the guess: the neighbour passed its limit)
        const bool todo = live && want != from;
        from = want;
        if (__builtin_amdgcn_ballot_w64(todo) == 0) break;
        uint32_t pos = want, steps = 0;
        bool on = todo && pos < limit, joined = false;
        for (; trips != 0 && __builtin_amdgcn_ballot_w64(on) != 0; --trips) {
            if (on) {
                uint64_t w = load_bits57(t, base + pos);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (on) {
                        const uint32_t rel = pos - guess;
                        joined = rel < kMarkBits && ((*(lds_v32)mark_at(rel) >> (rel & 31u)) & 1u) != 0;
                        if (!joined) {
                            pos += step_code<PAIR>(t, tb, base + pos, w);
                            ++steps;
                        }
                        on = !joined && pos < limit;
                    }
            }
        }
        agreed = __builtin_amdgcn_ballot_w64(on) == 0;
        if (todo) {
            upto = joined ? first_upto : pos;
            count = steps;
            if (joined) {
                // the first pass's codes from the common start on
                const uint32_t rel = pos - guess;
                count += first_count;
#pragma unroll
                for (uint32_t d = 0; d < kMarkBits / 32u; ++d) {
                    const uint32_t below = d < (rel >> 5) ? ~0u : d == (rel >> 5) ? (1u << (rel & 31u)) - 1u : 0u;
                    count -= static_cast<uint32_t>(__builtin_popcount(marks[d * 64u] & below));
                }
            }
        }
    }
    uint32_t sum = count;                                        // symbols up to the end of the lane's stretch
    for (uint32_t m = 1; m < parts; m <<= 1) {
        const uint32_t y = __shfl_up(sum, m, 64);
        sum += part >= m ? y : 0u;
    }
    const uint32_t total = __shfl(sum, static_cast<int>(lane | (parts - 1u)), 64);
    if (!agreed || __builtin_amdgcn_ballot_w64(total < nsym) != 0) {
        u.symbols = S << sh;
        u.first >>= sh;
        const uint32_t segments = (u.end + parts - 1u) >> sh, mine = u.first + (64u >> sh);
        u.end = segments < mine ? segments : mine;
        const uint32_t k = u.first + lane;
        return k < u.end ? t.offsets[k] : 0;
    }
    uint32_t idx = sum - count;
    const uint32_t stop = sum < nsym ? sum : nsym;
    uint32_t slot = (idx + S - 1u) / S;                          // next piece to start at or behind symbol idx
    while (slot * S < stop) {
        uint64_t w = load_bits57(t, base + from);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (idx == slot * S && idx < stop) {
                ring[lane - part + slot] = from;
                ++slot;
            }
            from += step_code<PAIR>(t, tb, base + from, w);
            ++idx;
        }
    }
    wave_sync_lds();
    const uint64_t start = u.first + lane < u.end ? base + ring[lane] : 0;
    wave_sync_lds();
    return start;
}

// The tensor's lanes of full length as far as the unit goes (which ends early only where a search was given up), and the
// symbols of the shorter last one, if the unit goes that far.
template <bool FIND>
__device__ __forceinline__ uint32_t full_lanes(const DevTensor &t, const Unit &u) {
    const uint32_t n_full = static_cast<uint32_t>(t.n / u.symbols);
    return FIND && u.end < n_full ? u.end : n_full;
}
template <bool FIND>
__device__ __forceinline__ uint32_t tail_symbols(const DevTensor &t, const Unit &u, uint32_t n_full) {
    if (FIND && u.end == n_full) return 0;
    return static_cast<uint32_t>(t.n - static_cast<uint64_t>(n_full) * u.symbols);
}

// Where the lane's part of a unit starts in the stream: found, where the tensor has been cut without entry points.
template <int MODE, bool FIND, class TB>
__device__ __forceinline__ uint64_t lane_start(const DevTensor &t, const TB &tb, lds_v32 ring, Unit &u) {
    if constexpr (FIND) return find_start<kPairMode<MODE>>(t, tb, ring, u);
    const uint32_t k = u.first + (threadIdx.x & 63u);
    return k < u.end ? seg_start(t, k) : 0;
}

template <int MODE> struct OutTraits;
template <> struct OutTraits<kModeU8> { static constexpr int ebits = 8; };
template <> struct OutTraits<kModeU4> { static constexpr int ebits = 4; };
template <> struct OutTraits<kModeF32> { static constexpr int ebits = 32; };
template <> struct OutTraits<kModeBF16> { static constexpr int ebits = 16; };
template <> struct OutTraits<kModeU8P> { static constexpr int ebits = 8; };
template <> struct OutTraits<kModeF32P> { static constexpr int ebits = 32; };
template <> struct OutTraits<kModeBF16P> { static constexpr int ebits = 16; };

// nsym symbols, element by element: the stream from absolute bit `pos` on holds the tensor's symbols
// first_sym, first_sym + 1, ... (first_sym is even for packed 4-bit output).
template <int MODE, class TB>
__device__ void decode_scalar_from(const DevTensor &t, const TB &tb, uint64_t pos, uint64_t first_sym, uint32_t nsym) {
    ScalarReader r;
    r.stream = t.stream;
    r.last_off = t.stream_bytes - 8u;
    r.pos = pos;
    r.buf = 0;
    const uint32_t max_len = t.max_len;
    const int32_t z = t.zero_point;
    const float s = t.scale;
    uint8_t *out8 = static_cast<uint8_t *>(t.out);
    uint32_t pending = 0;     // low nibble waiting for its partner (packed 4-bit)
    for (uint32_t i = 0; i < nsym; ++i) {
        if (i % kScalarProbes == 0) r.buf = load_bits(r.stream, r.pos, r.last_off);
        const uint32_t sym = entry_sym(next_entry<kPairMode<MODE>>(r, tb, max_len));
        const uint64_t idx = first_sym + i;
        constexpr int OUT = base_mode(MODE);
        if (OUT == kModeU8) out8[idx] = static_cast<uint8_t>(sym);
        if (OUT == kModeU4) {
            if (idx & 1) out8[idx >> 1] = static_cast<uint8_t>(pending | ((sym & 0xfu) << 4));
            else pending = sym & 0xfu;
        }
        if (OUT == kModeBF16) reinterpret_cast<uint16_t *>(t.out)[idx] = static_cast<uint16_t>(bf16_bits(dequant(sym, z, s)));
        if (OUT == kModeF32) reinterpret_cast<float *>(t.out)[idx] = dequant(sym, z, s);
    }
    if (MODE == kModeU4 && (nsym & 1)) out8[(first_sym + nsym - 1) >> 1] = static_cast<uint8_t>(pending);
}

// All nsym symbols of segment k, element by element.
template <int MODE, class TB>
__device__ void decode_scalar(const DevTensor &t, const TB &tb, uint32_t k, uint32_t nsym) {
    decode_scalar_from<MODE>(t, tb, seg_start(t, k), static_cast<uint64_t>(k) * t.chunk_symbols, nsym);
}

// ------------------------------------------------------------------ ring reader
// The long ring (gemv_direct, i.e. the GEMV of tensors that do not fit the wide tables; the
// other kernels use the short ring below).  Each lane keeps up to 128 bytes of its segment
// in a ring in LDS (eight 16-byte blocks, block j in slot j & 7) and the line that follows
// the ring's contents in registers: a lane asks memory for a whole line at a time (LB
// blocks; gemv_direct takes 64 bytes).  Dwords
// 32 and 33 of the lane's ring mirror dwords 0 and 1, so a three-dword read
// starting in the last ring dwords needs no wrap.
// Positions are bits relative to line 0, the line in which the segment starts.  The lane tracks q = p - 1, p being its position: a window read at bit
// q carries one stale low bit, which makes bits 1..14 the first-level table's
// byte offset of the code that starts at p.
// Registers move into the ring only between blocks of output (ring_topup), two
// blocks at a time, at the point where the wave's previous stores have long been
// written: a wait for the line then does not wait for stores.  A lane whose codes
// are so long that the ring runs dry in between loads its ring afresh.
// LB: blocks per line, 8 (128 bytes) or 4 (64 bytes).
template <int LB>
struct RingReader {
    static_assert(LB == 4 || LB == 8, "a line is a half or a whole 128-byte memory line");
    static constexpr uint32_t line_bytes = 16u * LB;
    const uint8_t *stream;
    lds_v32 ring;          // this lane's dword 0; dword d is ring[d * 64]
    uint32_t start64;      // byte offset of line 0 (a multiple of the line size)
    uint32_t last_blk;     // stream_bytes - 16
    uint32_t q;            // p - 1
    uint32_t end;          // the ring holds the stream up to here; a multiple of 256, at most kRingBits past p's block
    u32x4 nx[LB];          // the line at `end`; its pairs of blocks in front of `end` are in the ring already
};

__device__ __forceinline__ u32x4 load_block(const uint8_t *stream, uint32_t off, uint32_t last_blk) {
    off = off < last_blk ? off : last_blk;
    return *(global_u4_ptr)(stream + off);
}

// Line `line` into the registers; blocks past the end of the stream repeat its
// last block (nothing decodes them).
template <int LB>
__device__ __forceinline__ void load_line(RingReader<LB> &r, uint32_t line) {
    const uint32_t base = r.start64 + line * RingReader<LB>::line_bytes;
#pragma unroll
    for (int i = 0; i < LB; ++i) r.nx[i] = load_block(r.stream, base + 16u * i, r.last_blk);
}

// Block `blk` (16 bytes, counted from line 0) into its slot.
template <int LB>
__device__ __forceinline__ void ring_store(RingReader<LB> &r, uint32_t blk, const u32x4 v) {
    const uint32_t slot = blk & 7u;
    lds_v32 dst = r.ring + slot * 256u;
    dst[0] = v.x; dst[64] = v.y; dst[128] = v.z; dst[192] = v.w;
    if (slot == 0) { r.ring[32 * 64] = v.x; r.ring[33 * 64] = v.y; }
}

// Fill the ring with the 128 bytes from the 64-byte half line that holds absolute
// stream bit `pos` on, and ask for the line that holds what comes next (with
// 128-byte lines and p in the second half of line 0 that is line 1, whose first
// half is in the ring then).  RARE: the loads are a loop, to stay small where
// this is inlined into paths that hardly ever run.
template <bool RARE, int LB>
__device__ __forceinline__ void ring_fill(RingReader<LB> &r, uint64_t pos) {
    r.start64 = static_cast<uint32_t>(pos >> 3) & ~(RingReader<LB>::line_bytes - 1u);
    r.q = static_cast<uint32_t>(pos - (static_cast<uint64_t>(r.start64) << 3)) - 1u;
    const uint32_t first = ((r.q + 1u) >> 9) * 4u;                  // first block of the half line that holds p
    r.end = kRingBits + first * 128u;
    if (RARE) {
#pragma unroll 1
        for (uint32_t b = 0; b < 8; ++b) ring_store(r, first + b, load_block(r.stream, r.start64 + 16u * (first + b), r.last_blk));
    } else {
#pragma unroll
        for (uint32_t b = 0; b < 8; ++b) ring_store(r, first + b, load_block(r.stream, r.start64 + 16u * (first + b), r.last_blk));
    }
    load_line(r, r.end / (128u * LB));
}

template <int LB>
__device__ __forceinline__ void ring_load(RingReader<LB> &r, uint64_t pos) { ring_fill<false>(r, pos); }

// A ring read at q takes the dword that holds bit q and the two after it: it
// stays inside the ring's contents while q + 64 < end.
template <int LB>
__device__ __forceinline__ bool ring_short(const RingReader<LB> &r, uint32_t ahead) { return r.q + ahead + 64u >= r.end; }

// Rare: a lane whose codes are so long that the ring ran dry starts it afresh at p.
template <int LB>
__device__ __forceinline__ void ring_reload(RingReader<LB> &r) {
    ring_fill<true>(r, (static_cast<uint64_t>(r.start64) << 3) + r.q + 1u);
}

// Move what the registers hold into the blocks p has left behind, two blocks at
// a time while two slots are free; after the line's last pair, ask for the next
// line.
template <int LB>
__device__ __forceinline__ void ring_topup(RingReader<LB> &r) {
    const uint32_t pblk = ((r.q + 1u) >> 7) << 7;                    // start of the block that holds p
#pragma unroll
    for (uint32_t pair = 0; pair < LB / 2; ++pair) {
        if (((r.end >> 8) & (LB / 2 - 1u)) == pair && r.end - pblk <= kRingBits - 256u) {
            ring_store(r, r.end >> 7, r.nx[2 * pair]);
            ring_store(r, (r.end >> 7) + 1u, r.nx[2 * pair + 1]);
            r.end += 256u;
            if (pair == LB / 2 - 1) load_line(r, r.end / (128u * LB));
        }
    }
}

// The stream from bit q = p - 1 on: 63 valid bits above the stale one.
template <int LB>
__device__ __forceinline__ uint64_t ring_read(const RingReader<LB> &r) {
    // a plain (not volatile) pointer: the compiler may fetch two of the dwords with one instruction
    const lds_p32 src = (lds_p32)(r.ring + ((r.q >> 5) & 31u) * 64u);
    const uint32_t w0 = src[0], w1 = src[64], w2 = src[128];
    const uint32_t lo = __builtin_amdgcn_alignbit(w1, w0, r.q);     // uses q & 31
    const uint32_t hi = __builtin_amdgcn_alignbit(w2, w1, r.q);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// ------------------------------------------------------------- short ring reader
// The same reader with half the LDS, for the kernels whose wavefront count is what limits them
// (a lane's chain of dependent table lookups is bound by LDS latency, so the number of lanes a
// compute unit keeps decoding is its throughput, and LDS is what limits that number): a ring of
// four 16-byte blocks per lane (block j in slot j & 3, dwords 16 and 17 mirror dwords 0 and 1)
// and registers moving into the ring after every 32 symbols instead of 64.  The registers still
// hold a whole 128-byte line (asking memory for 64 bytes at a time reads every line twice).  Block
// i of a line goes to slot i & 3, so the moves are four statically addressed steps, each taken by
// the lanes whose next block belongs into that slot and whose slot is free.  A lane asks for its
// next line when the last block of the current one has moved; it is used from the next boundary
// on, one wait for the whole wavefront.
struct Ring2 {
    const uint8_t *stream;
    lds_v32 ring;          // this lane's dword 0; dword d is ring[d * 64]
    uint32_t start64;      // byte offset of line 0 (a multiple of 128)
    uint32_t last_blk;     // stream_bytes - 16
    uint32_t stale;        // stale low bits of a window: 1 for tables of 16-bit entries, 2 for 32-bit entries
    uint32_t q;            // p - stale, in bits from line 0
    uint32_t end;          // the ring holds the stream up to here; a multiple of 128, at most kRing2Bits past p's block
    u32x4 nx[8];           // the line that holds block end >> 7
};

template <int SLOT>
__device__ __forceinline__ void ring2_store(Ring2 &r, const u32x4 v) {
    lds_v32 dst = r.ring + SLOT * 256;
    dst[0] = v.x; dst[64] = v.y; dst[128] = v.z; dst[192] = v.w;
    if (SLOT == 0) { r.ring[16 * 64] = v.x; r.ring[17 * 64] = v.y; }
}

__device__ __forceinline__ void ring2_load_line(Ring2 &r, uint32_t line) {
    const uint32_t base = r.start64 + line * 128u;
#pragma unroll
    for (int i = 0; i < 8; ++i) r.nx[i] = load_block(r.stream, base + 16u * i, r.last_blk);
}

// Fill the ring with the four blocks from the one that holds absolute stream bit `pos` on and ask
// for the line that holds the block after them (line 0 again, if they end inside it).
template <bool RARE>
__device__ __forceinline__ void ring2_fill(Ring2 &r, uint64_t pos) {
    r.start64 = static_cast<uint32_t>(pos >> 3) & ~127u;
    r.q = static_cast<uint32_t>(pos - (static_cast<uint64_t>(r.start64) << 3)) - r.stale;
    const uint32_t first = (r.q + r.stale) >> 7;                     // 0..7
    r.end = (first + 4u) * 128u;
    if (RARE) {
#pragma unroll 1
        for (uint32_t b = first; b < first + 4u; ++b) {
            const u32x4 v = load_block(r.stream, r.start64 + 16u * b, r.last_blk);
            lds_v32 dst = r.ring + (b & 3u) * 256u;
            dst[0] = v.x; dst[64] = v.y; dst[128] = v.z; dst[192] = v.w;
            if ((b & 3u) == 0) { r.ring[16 * 64] = v.x; r.ring[17 * 64] = v.y; }
        }
    } else {
        u32x4 v[4];
#pragma unroll
        for (uint32_t b = 0; b < 4; ++b) v[b] = load_block(r.stream, r.start64 + 16u * (first + b), r.last_blk);
#pragma unroll
        for (uint32_t b = 0; b < 4; ++b) {
            lds_v32 dst = r.ring + ((first + b) & 3u) * 256u;
            dst[0] = v[b].x; dst[64] = v[b].y; dst[128] = v[b].z; dst[192] = v[b].w;
            if (((first + b) & 3u) == 0) { r.ring[16 * 64] = v[b].x; r.ring[17 * 64] = v[b].y; }
        }
    }
    ring2_load_line(r, r.end >> 10);
}

__device__ __forceinline__ bool ring_short(const Ring2 &r, uint32_t ahead) { return r.q + ahead + 64u >= r.end; }

__device__ __forceinline__ void ring_reload(Ring2 &r) {
    ring2_fill<true>(r, (static_cast<uint64_t>(r.start64) << 3) + r.q + r.stale);
}

template <int J>
__device__ __forceinline__ void ring2_step(Ring2 &r, uint32_t pblk, bool &wants_line) {
    if (((r.end >> 7) & 3u) == J && r.end - pblk <= kRing2Bits - 128u) {
        const bool upper = (r.end >> 9) & 1u;                        // the line's second half
        u32x4 v;
        v.x = upper ? r.nx[J + 4].x : r.nx[J].x;
        v.y = upper ? r.nx[J + 4].y : r.nx[J].y;
        v.z = upper ? r.nx[J + 4].z : r.nx[J].z;
        v.w = upper ? r.nx[J + 4].w : r.nx[J].w;
        ring2_store<J>(r, v);
        r.end += 128u;
        if (J == 3 && upper) wants_line = true;
    }
}

// Between two half blocks of output: registers into the slots p has left behind, then the request for the
// next line by the lanes whose registers are used up.
__device__ __forceinline__ void ring2_topup(Ring2 &r) {
    const uint32_t pblk = ((r.q + r.stale) >> 7) << 7;
    bool wants_line = false;
    ring2_step<0>(r, pblk, wants_line);
    ring2_step<1>(r, pblk, wants_line);
    ring2_step<2>(r, pblk, wants_line);
    ring2_step<3>(r, pblk, wants_line);
    if (wants_line) ring2_load_line(r, r.end >> 10);
}

__device__ __forceinline__ uint64_t ring_read(const Ring2 &r) {
    const lds_p32 src = (lds_p32)(r.ring + ((r.q >> 5) & 15u) * 64u);
    const uint32_t w0 = src[0], w1 = src[64], w2 = src[128];
    const uint32_t lo = __builtin_amdgcn_alignbit(w1, w0, r.q);
    const uint32_t hi = __builtin_amdgcn_alignbit(w2, w1, r.q);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// The first-level entry at this byte offset (an index shifted left by the table's number of stale bits).
template <class TB>
__device__ __forceinline__ uint32_t lut_at(const TB &tb, uint32_t byte_off) {
    typedef std::remove_const_t<std::remove_reference_t<decltype(tb.lut[0])>> E;
    return *reinterpret_cast<const E *>(reinterpret_cast<const char *>(tb.lut) + byte_off);
}

// The rest of a group for the lanes that met a code longer than kL1 bits.  e0..e3
// are the group's entries (from the long code on they all are its miss entry),
// w is the window as it stopped in front of the long code, `packed` the symbols in
// front of it (and junk behind).  The long code comes out of the second level
// with the bits still in the window (at least 63 - 3 * 14 of them; it needs 20)
// or, failing that, out of the canonical search; the symbols behind it are
// looked up one by one, each with a window of its own.
// With pair tables a miss is a pair that the index bits do not hold in full: its
// two codes, and whatever pair after it misses again, come from the table of
// single codes, every one with a window of its own.
template <bool PAIR, class Reader, class TB>
__device__ __forceinline__ uint32_t careful_group(Reader &r, const TB &tb, uint32_t max_len, uint32_t e0,
                                                  uint32_t e1, uint32_t e2, uint32_t e3, uint64_t w, uint32_t packed) {
    const uint32_t l0 = entry_len(e0), l1 = entry_len(e1), l2 = entry_len(e2);
    const uint32_t at = l0 == 0 ? 0u : l1 == 0 ? 1u : l2 == 0 ? 2u : 3u;     // place of the long code
    r.q += l0 + l1 + l2;                                                   // its entries add nothing
    if constexpr (PAIR) {
        packed = __builtin_amdgcn_ubfe(packed, 0, 8u * at);
#pragma unroll 1
        for (uint32_t i = at; i < static_cast<uint32_t>(kGroup); ++i) {
            if (ring_short(r, 0)) ring_reload(r);
            uint32_t e = lut_at(tb, static_cast<uint32_t>(ring_read(r)) & (kL1Mask << TB::stale));
            if (entry_len(e) == 0) {
                const uint32_t a = single_entry(tb, static_cast<uint32_t>(ring_read(r) >> TB::stale), max_len);
                r.q += entry_len(a);
                if (ring_short(r, 0)) ring_reload(r);
                const uint32_t b = single_entry(tb, static_cast<uint32_t>(ring_read(r) >> TB::stale), max_len);
                r.q += entry_len(b);
                e = ((entry_sym(a) & 0xfu) | ((entry_sym(b) & 0xfu) << 4)) << 8;
            } else {
                r.q += entry_len(e);
            }
            packed |= entry_sym(e) << (8u * i);
        }
        if (ring_short(r, kTripBits - 64)) ring_reload(r);
        return packed;
    }
    uint32_t e = lookup_l2(tb, e3, static_cast<uint32_t>(w >> TB::stale));
    if (__builtin_expect(e == 0, 0)) {
        if (ring_short(r, 0)) ring_reload(r);
        e = decode_canonical(tb, static_cast<uint32_t>(ring_read(r) >> TB::stale), kL1 + 1, max_len);
    }
    packed = __builtin_amdgcn_ubfe(packed, 0, 8u * at) | (entry_sym(e) << (8u * at));
    r.q += entry_len(e);
    if (at < static_cast<uint32_t>(kGroup) - 1u) {
        // the symbols behind it: one fresh window holds them all unless another long code turns up
        if (ring_short(r, 0)) ring_reload(r);
        uint64_t wi = ring_read(r);
#pragma unroll
        for (uint32_t i = 1; i < static_cast<uint32_t>(kGroup); ++i) {
            if (i > at) {
                e = lut_at(tb, static_cast<uint32_t>(wi) & (kL1Mask << TB::stale));
                if (__builtin_expect(entry_len(e) == 0, 0)) {
                    if (ring_short(r, 0)) ring_reload(r);
                    wi = ring_read(r);
                    e = decode_long(tb, e, static_cast<uint32_t>(wi >> TB::stale), max_len);
                    r.q += entry_len(e);
                    if (ring_short(r, 0)) ring_reload(r);
                    wi = ring_read(r);
                } else {
                    wi >>= entry_len(e);
                    r.q += entry_len(e);
                }
                packed |= entry_sym(e) << (8u * i);
            }
        }
    }
    // the groups that follow in this trip count on the usual margin
    if (ring_short(r, kTripBits - 64)) ring_reload(r);
    return packed;
}

// One group: a fresh window and kGroup table lookups without a branch; every
// entry is the shift amount that moves the window to the next code.  A lane that
// meets a code longer than kL1 bits stops moving (its later lookups see the same
// bits and give the same entry of length zero); if the wave has such a lane, the
// rest of its group is decoded with more care.  Returns the group's four symbols,
// first one lowest.
template <bool PAIR, class Reader, class TB>
__device__ __forceinline__ uint32_t ring_group(Reader &r, const TB &tb, uint32_t max_len) {
    uint64_t w = ring_read(r);
    const uint32_t e0 = lut_at(tb, static_cast<uint32_t>(w) & (kL1Mask << TB::stale));
    w >>= (e0 & 63u);
    const uint32_t e1 = lut_at(tb, static_cast<uint32_t>(w) & (kL1Mask << TB::stale));
    w >>= (e1 & 63u);
    const uint32_t e2 = lut_at(tb, static_cast<uint32_t>(w) & (kL1Mask << TB::stale));
    w >>= (e2 & 63u);
    const uint32_t e3 = lut_at(tb, static_cast<uint32_t>(w) & (kL1Mask << TB::stale));
    // byte 1 of each entry, in order
    uint32_t packed = __builtin_amdgcn_perm(e1, e0, 0x0c0c0501u) | __builtin_amdgcn_perm(e3, e2, 0x05010c0cu);
    uint32_t q_next = r.q + ((e0 + e1 + e2 + e3) & 0xffu);            // lengths add up in the low byte (<= 56)
    const bool miss = (e3 & 0xffu) == 0;                              // a miss entry's low byte is zero
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(miss) != 0, 0)) {
        if (miss) {
            packed = careful_group<PAIR>(r, tb, max_len, e0, e1, e2, e3, w, packed);
            q_next = r.q;
        }
    }
    r.q = q_next;
    return packed;
}

// A trip of ring_groups for a code whose lengths lie within four neighbouring ones, none above kL1 bits, all of its space taken
// (flat_code): where the next code begins follows from three comparisons, so the lookups, which give the symbols, are not part of
// the chain, and the next window is asked for before a group's symbols are waited for.
// For launches that are one lane's chain and little else: one tensor of 2048 symbols, a lane per piece of 256, to fp32 20.5 -> 19.0 us.
__device__ __forceinline__ void ring_trip_flat(Ring2 &r, const Tables &tb, const DevTensor &t, uint32_t (&four)[kTripGroups]) {
    uint64_t w = ring_read(r);
#pragma unroll
    for (int g = 0; g < kTripGroups; ++g) {
        uint32_t e[4], q = r.q;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            e[i] = lut_at(tb, static_cast<uint32_t>(w) & (kL1Mask << Tables::stale));
            const uint32_t v = __brev(static_cast<uint32_t>(w)) << Tables::stale;
            const uint32_t l = t.flat_len + (v > t.flat_last[0] ? 1u : 0u) + (v > t.flat_last[1] ? 1u : 0u) + (v > t.flat_last[2] ? 1u : 0u);
            w >>= l;
            q += l;
        }
        r.q = q;
        if (g + 1 < kTripGroups) w = ring_read(r);
        __builtin_amdgcn_sched_barrier(0);
        four[g] = __builtin_amdgcn_perm(e[1], e[0], 0x0c0c0501u) | __builtin_amdgcn_perm(e[3], e[2], 0x05010c0cu);
    }
}

// ring_group on wide tables, for the GEMV: returns the four symbols' values (symbol - zero_point as bf16, two per
// dword, first one lowest) instead of the symbols.
template <class Reader>
__device__ __forceinline__ u32x2 ring_group_wide(Reader &r, const Tables32 &tb, uint32_t max_len, float zf) {
    constexpr uint32_t kMask = kL1Mask << Tables32::stale;
    uint64_t w = ring_read(r);
    const uint32_t e0 = lut_at(tb, static_cast<uint32_t>(w) & kMask);
    w >>= (e0 & 63u);
    const uint32_t e1 = lut_at(tb, static_cast<uint32_t>(w) & kMask);
    w >>= (e1 & 63u);
    const uint32_t e2 = lut_at(tb, static_cast<uint32_t>(w) & kMask);
    w >>= (e2 & 63u);
    const uint32_t e3 = lut_at(tb, static_cast<uint32_t>(w) & kMask);
    // the high halves of the entries, in order
    u32x2 vals = {__builtin_amdgcn_perm(e1, e0, 0x07060302u), __builtin_amdgcn_perm(e3, e2, 0x07060302u)};
    uint32_t q_next = r.q + ((e0 + e1 + e2 + e3) & 0xffu);
    const bool miss = (e3 & 0xffu) == 0;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(miss) != 0, 0)) {
        if (miss) {
            const uint32_t packed = careful_group<false>(r, tb, max_len, e0, e1, e2, e3, w,
                                                         __builtin_amdgcn_perm(e1, e0, 0x0c0c0501u) | __builtin_amdgcn_perm(e3, e2, 0x05010c0cu));
            // the same values by arithmetic: an integer of at most 256 in magnitude is a bf16 as it stands
            const uint32_t v0 = __float_as_uint(static_cast<float>(packed & 0xffu) - zf) >> 16;
            const uint32_t v1 = __float_as_uint(static_cast<float>((packed >> 8) & 0xffu) - zf) & 0xffff0000u;
            const uint32_t v2 = __float_as_uint(static_cast<float>((packed >> 16) & 0xffu) - zf) >> 16;
            const uint32_t v3 = __float_as_uint(static_cast<float>(packed >> 24) - zf) & 0xffff0000u;
            vals = u32x2{v0 | v1, v2 | v3};
            q_next = r.q;
        }
    }
    r.q = q_next;
    return vals;
}

template <int MODE, class TB>
__device__ __forceinline__ void gemv_segment(const DevTensor &t, const TB &tb, uint32_t k);

// Decode the kUnit segments from wave_first on, one per lane of this wavefront,
// SPB symbols per lane at a time into the wave's
// LDS tile (one row of symbol bytes per lane; all lanes move in step, four
// symbols per group), then consume the tile row-wise: write it out in the output
// type, so that every store instruction covers whole rows.
template <int MODE, bool FIND = false>
__device__ __forceinline__ void decode_rows(const DevTensor &t, const Tables &tb, WaveMem<Cfg<MODE>::row> *wms,
                                            uint32_t wave_first) {
    static_assert(!is_gemv(MODE), "the GEMV has a kernel of its own");
    constexpr bool PAIR = kPairMode<MODE>;
    constexpr int SPB = Cfg<MODE>::spb;                   // symbols of a lane per block
    constexpr int ROW = Cfg<MODE>::row;                   // bytes they make in the tile
    constexpr int OUT_ROW = Cfg<MODE>::out_row;
    constexpr uint32_t PIECE = Cfg<MODE>::piece;          // tile bytes one lane consumes per pass
    constexpr uint32_t LPR = ROW / PIECE;                 // lanes that consume one row
    constexpr uint32_t RPI = 64 / LPR;                    // rows per pass
    constexpr uint32_t EBITS = OutTraits<MODE>::ebits;
    constexpr int TRIPS = ROW / (kGroup * kTripGroups);
    static_assert(ROW % (kGroup * kTripGroups) == 0, "a row is a whole number of trips");
    static_assert(SPB == (PAIR ? 2 : 1) * ROW, "one tile byte per lookup");
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = threadIdx.x >> 6;
    WaveMem<ROW> &wm = wms[wave];
    if (wave_first >= t.n_chunks) return;
    Unit u = {wave_first, t.n_chunks, t.chunk_symbols};
    uint64_t tail_pos = lane_start<MODE, FIND>(t, tb, (lds_v32)wm.ring, u);   // where the symbols behind the lane's last whole block start
    wave_first = u.first;
    const uint32_t C = u.symbols;
    const uint32_t blocks_total = C / SPB;
    const uint32_t k = wave_first + lane;
    uint32_t nsym = 0;
    if (k < u.end) {
        const uint64_t left = t.n - static_cast<uint64_t>(k) * C;
        nsym = left < C ? static_cast<uint32_t>(left) : C;
    }
    // A shorter last lane takes the row path for its whole blocks and the scalar path for the
    // rest.  The lane moves on with the others past its own end; what it decodes there is not stored.
    const uint32_t my_blocks = nsym / SPB;
    Ring2 r;
    r.stale = Tables::stale;
    r.stream = t.stream;
    r.last_blk = t.stream_bytes - 16u;
    r.ring = (lds_v32)(wm.ring + lane);
    // a lane without a full segment decodes the start of the stream along with the others; nothing of it is stored
    ring2_fill<false>(r, tail_pos);
    const uint64_t bytes_per_chunk = (static_cast<uint64_t>(C) * EBITS) >> 3;
    // the unit's lanes of full length end here, and whole blocks of the shorter last one, if it is among them
    const uint32_t n_full = full_lanes<FIND>(t, u);
    const uint32_t tail_blocks = tail_symbols<FIND>(t, u, n_full) / SPB;
    // a wave that holds only the shorter last segment stops after its blocks
    const uint32_t wave_blocks = wave_first < n_full ? blocks_total : tail_blocks;
    // where the first row this lane serves in a flush pass begins; the passes are RPI rows apart
    uint8_t *const row0 = static_cast<uint8_t *>(t.out) + (wave_first + lane / LPR) * bytes_per_chunk;
    const uint32_t max_len = t.max_len;
    const float zf = static_cast<float>(t.zero_point);    // exact: the host rejects |z| > 2^24
    const float scale = t.scale;
    lds_v32 tile = (lds_v32)wm.tile;

    // integer outputs whose blocks make 64 bytes per row: the even block's pieces, kept for the odd block's flush
    constexpr bool HOLD = OUT_ROW == 64;
    u32x4 held[HOLD ? 64 / RPI : 1];
    bool held_full[HOLD ? 64 / RPI : 1];
    for (uint32_t bs = 0; bs < wave_blocks; ++bs) {
#pragma unroll 1
        for (int trip = 0; trip < TRIPS; ++trip) {
            if (__builtin_expect(ring_short(r, kTripBits - 64), 0)) ring_reload(r);
#pragma unroll
            for (int g = 0; g < kTripGroups; ++g)
                tile[WaveMem<ROW>::tile_at(lane, trip * kTripGroups + g)] = ring_group<PAIR>(r, tb, max_len);
            // the short ring is topped up after every eight groups
            if (trip & 1) ring2_topup(r);
        }
        if (bs + 1 == my_blocks) tail_pos = (static_cast<uint64_t>(r.start64) << 3) + r.q + r.stale;
        wave_sync_lds();
#pragma unroll
        for (uint32_t it = 0; it < 64 / RPI; ++it) {
            const uint32_t rr = it * RPI + lane / LPR;
            const uint32_t piece = lane % LPR;
            const uint32_t kk = wave_first + rr;
            // the row has this block: always in a full segment, up to tail_blocks in the shorter last one
            const bool full = kk < n_full || (kk == n_full && bs < tail_blocks);
            uint8_t *dst = row0 + static_cast<uint64_t>(it) * (RPI * bytes_per_chunk) + static_cast<uint64_t>(bs) * OUT_ROW;
            // Store k of the pass writes the bytes [k * LPR * 16, (k + 1) * LPR * 16) of the row's
            // piece of this block, 16 per lane, so that every store instruction covers whole
            // stretches of memory; the lane fetches the tile bytes that become its 16 bytes.
            constexpr int OUT = base_mode(MODE);
            constexpr uint32_t SYMS = OUT == kModeF32 ? 4u : OUT == kModeBF16 ? 8u : OUT == kModeU8 ? 16u : 32u;   // per 16 bytes
            constexpr uint32_t TB = PAIR && OUT != kModeU4 ? SYMS / 2u : OUT == kModeU4 ? 16u : SYMS;   // tile bytes for them
            constexpr uint32_t NST = ROW / (LPR * TB);
            static_assert(NST * LPR * TB == ROW && NST * LPR * 16u == static_cast<uint32_t>(OUT_ROW), "the stores tile the row");
#pragma unroll
            for (uint32_t k = 0; k < NST; ++k) {
                const uint32_t tb0 = (k * LPR + piece) * TB;        // first tile byte of this lane's share
                uint32_t raw[TB >= 4 ? TB / 4 : 1];
#pragma unroll
                for (uint32_t j = 0; j < (TB >= 4 ? TB / 4 : 1); ++j) raw[j] = tile[WaveMem<ROW>::tile_at(rr, tb0 / 4 + j)];
                if (TB < 4) raw[0] = (raw[0] >> (8u * (tb0 & 3u))) & 0xffffu;    // two pair bytes out of a dword
                uint8_t *const at = dst + k * (LPR * 16u) + piece * 16u;
                if constexpr (OUT == kModeU8 || OUT == kModeU4) {
                    u32x4 v;
                    if constexpr (PAIR && OUT == kModeU8) {
                        // 8 pair bytes -> 16 symbol bytes
                        uint32_t u[4];
                        unpack_nibbles(raw[0], u[0], u[1]);
                        unpack_nibbles(raw[1], u[2], u[3]);
                        v = u32x4{u[0], u[1], u[2], u[3]};
                    } else {
                        // the tile bytes are the output bytes (4-bit pairs come packed out of the table)
                        v = u32x4{raw[0], raw[1], raw[2], raw[3]};
                    }
                    if constexpr (HOLD) {
                        // a block makes only 64 bytes per row: the even block's piece waits for the odd
                        // block's, and the two go out in neighbouring store instructions, which the L2
                        // merges into whole 128-byte lines (64 bytes at a time reach memory at 2.8 TB/s,
                        // the merged lines at 4.8)
                        if ((bs & 1u) == 0 && bs + 1 < wave_blocks) {
                            held[it] = v;
                            held_full[it] = full;
                        } else {
                            if ((bs & 1u) && held_full[it]) *(global_u4_wptr)(at - OUT_ROW) = held[it];
                            if (full) *(global_u4_wptr)at = v;
                        }
                    } else {
                        if (full) *(global_u4_wptr)at = v;
                    }
                } else {
                    // w = (q - z) * s: exact difference, one fp32 multiply
                    uint32_t sym4[SYMS / 4];                         // one symbol per byte
                    if constexpr (PAIR) {
                        if constexpr (SYMS == 8) {
                            unpack_nibbles(raw[0], sym4[0], sym4[1]);
                        } else {
                            uint32_t unused;
                            unpack_nibbles(raw[0], sym4[0], unused);
                        }
                    } else {
#pragma unroll
                        for (uint32_t j = 0; j < SYMS / 4; ++j) sym4[j] = raw[j];
                    }
                    float f[SYMS];
#pragma unroll
                    for (uint32_t j = 0; j < SYMS; ++j)
                        f[j] = (static_cast<float>((sym4[j / 4] >> (8 * (j % 4))) & 0xffu) - zf) * scale;
                    u32x4 v;
                    if constexpr (OUT == kModeF32) {
                        v = u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const f32x2 pr = {f[2 * j], f[2 * j + 1]};
                            const bf16x2 b = __builtin_convertvector(pr, bf16x2);   // round to nearest even
                            v[j] = __builtin_bit_cast(uint32_t, b);
                        }
                    }
                    if (full) {
                        if constexpr (OUT == kModeF32) *(global_u4_wptr)at = v;
                        else __builtin_nontemporal_store(v, (global_u4_wptr)at);
                    }
                }
            }
        }
        wave_sync_lds();
    }
    const uint32_t rest = nsym - my_blocks * SPB;
    if (rest) decode_scalar_from<MODE>(t, tb, tail_pos, static_cast<uint64_t>(k) * C + my_blocks * SPB, rest);
}

// decode_rows for the fp32 and bf16 outputs with a tile of half a block: sixteen wavefronts per
// workgroup instead of fourteen.  A block of 64 symbols per lane is decoded and flushed in two halves of 32.  A
// half makes 128 bytes of fp32 per row, which go out as they are; of bf16 it makes 64, so the first
// half's symbols wait in registers (in the lanes that will convert them) and the second half's flush
// writes whole 128-byte rows.
// ALLFULL: the unit's 64 segments all have full length (decided per wavefront): no store needs a
// condition, no lane a tail.
template <int MODE, bool ALLFULL, bool FIND, bool FLAT>
__device__ __forceinline__ void decode_rows2_impl(const DevTensor &t, const Tables &tb, WaveMem2 &wm, const Unit &u, uint64_t tail_pos) {
    static_assert(MODE == kModeF32 || MODE == kModeBF16, "single codes, two or four bytes per symbol");
    constexpr int SPB = Cfg<MODE>::spb;                   // 64
    constexpr uint32_t EBITS = OutTraits<MODE>::ebits;
    constexpr int HALF_GROUPS = 8;                        // groups of four symbols per half block
    static_assert(SPB == 64 && HALF_GROUPS * kGroup * 2 == SPB && HALF_GROUPS % kTripGroups == 0, "two halves of two trips");
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave_first = u.first;
    const uint32_t C = u.symbols;
    const uint32_t blocks_total = C / SPB;
    const uint32_t k = wave_first + lane;
    uint32_t nsym = C;
    if (!ALLFULL) {
        nsym = 0;
        if (k < u.end) {
            const uint64_t left = t.n - static_cast<uint64_t>(k) * C;
            nsym = left < C ? static_cast<uint32_t>(left) : C;
        }
    }
    const uint32_t my_blocks = nsym / SPB;
    Ring2 r;
    r.stale = Tables::stale;
    r.stream = t.stream;
    r.last_blk = t.stream_bytes - 16u;
    r.ring = (lds_v32)(wm.ring + lane);
    ring2_fill<false>(r, tail_pos);
    const uint64_t bytes_per_chunk = (static_cast<uint64_t>(C) * EBITS) >> 3;
    const uint32_t n_full = full_lanes<FIND>(t, u);
    const uint32_t tail_blocks = tail_symbols<FIND>(t, u, n_full) / SPB;
    const uint32_t wave_blocks = ALLFULL || wave_first < n_full ? blocks_total : tail_blocks;
    // a flush pass serves eight rows, eight lanes each; the passes are eight rows apart
    const uint32_t piece = lane & 7u;
    uint8_t *const row0 = static_cast<uint8_t *>(t.out) + (wave_first + (lane >> 3)) * bytes_per_chunk + piece * 16u;
    const uint32_t max_len = t.max_len;
    const float zf = static_cast<float>(t.zero_point);    // exact: the host rejects |z| > 2^24
    const float scale = t.scale;
    lds_v32 tile = (lds_v32)wm.tile;
    typedef const u32x2 __attribute__((address_space(3))) *lds_p64;
    u32x2 held[8];                                        // bf16: the first half's eight symbols of each pass
    for (uint32_t bs = 0; bs < wave_blocks; ++bs) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll 1
            for (int trip = 0; trip < HALF_GROUPS / kTripGroups; ++trip) {
                if (__builtin_expect(ring_short(r, kTripBits - 64), 0)) ring_reload(r);
                if constexpr (FLAT) {
                    uint32_t four[kTripGroups];              // (written behind the trip's last lookup)
                    ring_trip_flat(r, tb, t, four);
#pragma unroll
                    for (int g = 0; g < kTripGroups; ++g) tile[WaveMem2::tile_at(lane, trip * kTripGroups + g)] = four[g];
                } else {
#pragma unroll
                    for (int g = 0; g < kTripGroups; ++g)
                        tile[WaveMem2::tile_at(lane, trip * kTripGroups + g)] = ring_group<false>(r, tb, max_len);
                }
            }
            if (!ALLFULL && half == 1 && bs + 1 == my_blocks) tail_pos = (static_cast<uint64_t>(r.start64) << 3) + r.q + r.stale;
            ring2_topup(r);
            wave_sync_lds();
#pragma unroll
            for (uint32_t it = 0; it < 8; ++it) {
                if (FLAT && wave_first + it * 8u > n_full) break;      // (none of these rows: a small launch has few)
                const uint32_t rr = it * 8u + (lane >> 3);
                const uint32_t kk = wave_first + rr;
                const bool full = ALLFULL || kk < n_full || (kk == n_full && bs < tail_blocks);
                uint8_t *const dst = row0 + static_cast<uint64_t>(it) * (8u * bytes_per_chunk);
                if constexpr (MODE == kModeF32) {
                    const uint32_t raw = tile[WaveMem2::tile_at(rr, piece)];
                    u32x4 v;
#pragma unroll
                    for (uint32_t j = 0; j < 4; ++j)
                        v[j] = __float_as_uint((static_cast<float>((raw >> (8 * j)) & 0xffu) - zf) * scale);
                    if (full) *(global_u4_wptr)(dst + (static_cast<uint64_t>(bs) * 2u + half) * 128u) = v;
                } else {
                    // lanes 0..3 of a row convert the first half's symbols, lanes 4..7 the second half's
                    const u32x2 raw = *(lds_p64)(wm.tile + WaveMem2::tile_at(rr, 2u * (piece & 3u)));
                    if (half == 0) {
                        held[it] = raw;
                    } else {
                        const u32x2 sym8 = piece < 4u ? held[it] : raw;
                        u32x4 v;
#pragma unroll
                        for (uint32_t j = 0; j < 4; ++j) {
                            const uint32_t d = sym8[j / 2];
                            const f32x2 pr = {(static_cast<float>((d >> (16 * (j & 1))) & 0xffu) - zf) * scale,
                                              (static_cast<float>((d >> (16 * (j & 1) + 8)) & 0xffu) - zf) * scale};
                            v[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));   // round to nearest even
                        }
                        if (full) __builtin_nontemporal_store(v, (global_u4_wptr)(dst + static_cast<uint64_t>(bs) * 128u));
                    }
                }
            }
            wave_sync_lds();
        }
    }
    if (!ALLFULL) {
        const uint32_t rest = nsym - my_blocks * SPB;
        if (rest) decode_scalar_from<MODE>(t, tb, tail_pos, static_cast<uint64_t>(k) * C + my_blocks * SPB, rest);
    }
}

template <int MODE, bool FIND = false, bool FLAT = false>
__device__ __forceinline__ void decode_rows2(const DevTensor &t, const Tables &tb, WaveMem2 *wms, uint32_t wave_first) {
    if (wave_first >= t.n_chunks) return;
    WaveMem2 &wm = wms[threadIdx.x >> 6];
    Unit u = {wave_first, t.n_chunks, t.chunk_symbols};
    const uint64_t start = lane_start<MODE, FIND>(t, tb, (lds_v32)wm.ring, u);
    if (u.first + kUnit <= full_lanes<FIND>(t, u)) decode_rows2_impl<MODE, true, FIND, FLAT>(t, tb, wm, u, start);
    else decode_rows2_impl<MODE, false, FIND, FLAT>(t, tb, wm, u, start);
}

// Decode one segment straight into dot products with x.  A segment covers one
// or more row fragments; complete rows are stored, a leading / trailing
// incomplete fragment goes to the segment's head / tail partial.
template <int MODE, class TB>
__device__ __forceinline__ void gemv_segment(const DevTensor &t, const TB &tb, uint32_t k) {
    const uint32_t C = t.chunk_symbols;
    const uint64_t first_sym = static_cast<uint64_t>(k) * C;
    const uint64_t left = t.n - first_sym;
    const uint32_t nsym = left < C ? static_cast<uint32_t>(left) : C;
    ScalarReader r;
    r.stream = t.stream;
    r.last_off = t.stream_bytes - 8u;
    r.pos = seg_start(t, k);
    r.buf = 0;
    const uint32_t max_len = t.max_len;
    const int32_t z = t.zero_point;
    const uint32_t cols = t.cols;

    uint32_t row = static_cast<uint32_t>(first_sym / cols);
    uint32_t col = static_cast<uint32_t>(first_sym - static_cast<uint64_t>(row) * cols);
    const uint32_t start_col = col;
    bool first_fragment = true;
    float acc = 0.0f;
    float head = 0.0f, tail = 0.0f;
    for (uint32_t i = 0; i < nsym; ++i) {
        if (i % kScalarProbes == 0) r.buf = load_bits(r.stream, r.pos, r.last_off);
        const uint32_t sym = entry_sym(next_entry<kPairMode<MODE>>(r, tb, max_len));
        const float xv = __uint_as_float(static_cast<uint32_t>(t.x[col]) << 16);
        acc = fmaf(static_cast<float>(static_cast<int32_t>(sym) - z), xv, acc);
        if (++col == cols) {
            if (first_fragment && start_col != 0) {
                head = acc;                              // row began in an earlier segment
            } else {
                const float y = acc * t.scale;
                if (gemv_f32(MODE)) reinterpret_cast<float *>(t.out)[row] = y;
                else reinterpret_cast<uint16_t *>(t.out)[row] = static_cast<uint16_t>(bf16_bits(y));
            }
            first_fragment = false;
            acc = 0.0f;
            col = 0;
            ++row;
        }
    }
    if (col != 0) {                                          // row continues in the next segment
        if (first_fragment) head = acc;
        else tail = acc;
    }
    if (t.need_fix) {
        t.partials[2 * static_cast<uint64_t>(k)] = head;
        t.partials[2 * static_cast<uint64_t>(k) + 1] = tail;
    }
}

// Lanes that take pieces of a row, t.row_lanes (a power of two, 2..64) side by side in one wavefront: every
// lane's piece lies inside one row and `mine` is its sum; the row's lanes add theirs up in a fixed tree and
// the first of them stores the row.  Neither partial sums in memory nor a second kernel are needed then.
template <int MODE>
__device__ __forceinline__ void wave_row_sums(const DevTensor &t, uint32_t k, bool full, float mine) {
    const uint32_t rl = t.row_lanes;
    float v = full ? mine : 0.0f;                          // (lanes behind the tensor's end)
#pragma unroll
    for (uint32_t m = 1; m < 64u; m <<= 1)
        if (m < rl) v += __shfl_xor(v, static_cast<int>(m), 64);
    if (full && (k & (rl - 1u)) == 0) {
        const float y = v * t.scale;
        const uint32_t row = k / rl;
        if (gemv_f32(MODE)) reinterpret_cast<float *>(t.out)[row] = y;
        else reinterpret_cast<uint16_t *>(t.out)[row] = static_cast<uint16_t>(bf16_bits(y));
    }
}

// GEMV: the lane that decodes a segment also multiplies it into x, a group of symbols at a time as
// they come out of the table; there is no tile and no flush, which leaves LDS for 14 wavefronts.
// All lanes are at the same place of their segments, so where segments and rows coincide the lanes
// of a wave ask for the same piece of x (one request); elsewhere they ask for a handful of
// different ones.  The 64 activations of a half block are requested one half block ahead, before
// the stream lines that ring_topup asks for: loads return in order, and a wait for x must not
// become a wait for the stream.
// A segment may begin and end anywhere in a row and hold any number of row ends (cols >= 64, so a
// half block holds at most one): the sum up to the first row end is the head fragment (or a whole
// row, if the segment starts one), every further row end completes a whole row, which the lane
// stores itself, and what is left at the end is the tail fragment; the fragments go to the
// segment's two partial sums, which the second stage adds up per row.
template <int MODE>
__device__ __forceinline__ void gemv_direct(const DevTensor &t, const Tables &tb, uint32_t *ring_mem, uint32_t wave_first) {
    constexpr bool PAIR = kPairMode<MODE>;                 // two 4-bit symbols per table lookup
    constexpr int SPG = PAIR ? 8 : 4;                      // symbols per group
    constexpr int GPH = 64 / SPG;                          // groups per half block of 64 symbols
    const uint32_t lane = threadIdx.x & 63u;
    if (wave_first >= t.n_chunks) return;
    const uint32_t C = t.chunk_symbols;
    const uint32_t k = wave_first + lane;
    uint32_t nsym = 0;
    if (k < t.n_chunks) {
        const uint64_t left = t.n - static_cast<uint64_t>(k) * C;
        nsym = left < C ? static_cast<uint32_t>(left) : C;
    }
    const bool fast = nsym == C;                           // a shorter last segment takes the element-by-element path
    RingReader<4> r;
    r.stream = t.stream;
    r.last_blk = t.stream_bytes - 16u;
    r.ring = (lds_v32)(ring_mem + lane);
    // a lane without a full segment decodes the start of the stream along with the others; nothing of it is stored
    ring_load(r, fast ? seg_start(t, k) : 0);
    const uint32_t cols = t.cols;
    const uint16_t *xvec = t.x;
    const uint32_t max_len = t.max_len;
    const float zf = static_cast<float>(t.zero_point);    // exact: the host rejects |z| > 2^24
    const float scale = t.scale;
    const uint64_t flat0 = static_cast<uint64_t>(k) * C;
    uint32_t col = fast ? static_cast<uint32_t>(flat0 % cols) : 0u;    // column of the half block's first symbol
    uint32_t row = fast ? static_cast<uint32_t>(flat0 / cols) : 0u;    // the row the lane is in
    const bool starts_row = col == 0;
    float acc = 0.0f, first = 0.0f, end_sum = 0.0f;
    bool crossed = false;                                  // a row end has been passed
    bool ended = false;                                    // a row ended in this half block: end_sum holds its sum
    // eight activations per piece; a piece never straddles a row end (cols % 8 == 0, segments start at multiples of 64)
    u32x4 xb[8];
    auto ask_x = [&](uint32_t c0) {
#pragma unroll
        for (uint32_t p = 0; p < 8; ++p) {
            uint32_t c = c0 + 8u * p;
            c -= c >= cols ? cols : 0u;
            xb[p] = *(global_u4_ptr)(xvec + c);
        }
    };
    auto mul4 = [&](uint32_t s4, uint32_t xa, uint32_t xc) {
        acc = fmaf(static_cast<float>(s4 & 0xffu) - zf, __uint_as_float(xa << 16), acc);
        acc = fmaf(static_cast<float>((s4 >> 8) & 0xffu) - zf, __uint_as_float(xa & 0xffff0000u), acc);
        acc = fmaf(static_cast<float>((s4 >> 16) & 0xffu) - zf, __uint_as_float(xc << 16), acc);
        acc = fmaf(static_cast<float>(s4 >> 24) - zf, __uint_as_float(xc & 0xffff0000u), acc);
    };
    ask_x(col);
    const uint32_t halves = C / 64u;
    for (uint32_t h = 0; h < halves; ++h) {
#pragma unroll
        for (int g = 0; g < GPH; ++g) {
            if (g % kTripGroups == 0)
                if (__builtin_expect(ring_short(r, kTripBits - 64), 0)) ring_reload(r);
            const uint32_t s4 = ring_group<PAIR>(r, tb, max_len);
            if constexpr (PAIR) {
                uint32_t lo, hi;
                unpack_nibbles(s4, lo, hi);
                mul4(lo, xb[g].x, xb[g].y);
                mul4(hi, xb[g].z, xb[g].w);
            } else {
                const u32x4 xv = xb[g / 2];
                mul4(s4, (g & 1) ? xv.z : xv.x, (g & 1) ? xv.w : xv.y);
            }
            if (PAIR || (g & 1)) {
                // a row ends behind this piece (at most once per half block: cols >= 64): its sum is set
                // aside without a branch, so that the groups of the half block stay one stretch of code
                const uint32_t piece = PAIR ? g : g / 2;
                const bool row_end = col + 8u * piece + 8u == cols;
                end_sum = row_end ? acc : end_sum;
                acc = row_end ? 0.0f : acc;
                ended |= row_end;
            }
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(ended) != 0, 0)) {
            if (ended) {
                if (!crossed && !starts_row) {
                    first = end_sum;                       // the head fragment
                } else if (fast) {                         // a whole row
                    const float y = end_sum * scale;
                    if (gemv_f32(MODE)) reinterpret_cast<float *>(t.out)[row] = y;
                    else reinterpret_cast<uint16_t *>(t.out)[row] = static_cast<uint16_t>(bf16_bits(y));
                }
                crossed = true;
                row += 1u;
                ended = false;
            }
        }
        col += 64u;
        col -= col >= cols ? cols : 0u;
        if (h + 1 < halves) ask_x(col);
        if (!PAIR || (h & 1u)) ring_topup(r);              // once per block of 16 groups
    }
    if (t.row_lanes) {
        wave_row_sums<MODE>(t, k, fast, crossed ? first : acc);
    } else if (fast) {
        if (!crossed) {
            t.partials[2 * static_cast<uint64_t>(k)] = acc;              // the segment lies inside one row
        } else {
            if (!starts_row) t.partials[2 * static_cast<uint64_t>(k)] = first;
            if (col != 0) t.partials[2 * static_cast<uint64_t>(k) + 1] = acc;   // the segment ends inside a row
        }
    } else if (nsym) {
        gemv_segment<MODE>(t, tb, k);
    }
}

// gemv_direct on wide tables and the short ring (8-bit symbols whose zero-point lies in [-1, 256], so that
// symbol - zero_point is a bf16 as it stands): the table entry carries that value, two v_perm gather a group's
// four values into two bf16 pairs and two v_dot2c_f32_bf16 multiply them into x; no conversion and no
// subtraction per symbol.  The 64 KB table and a ring of 64 bytes per lane leave LDS for sixteen wavefronts.
// The ring is topped up after every eight groups.  Row ends, fragments and the request for x one half block
// ahead are gemv_direct's; lanes that cut a row into a power of two of pieces add the row up themselves
// (wave_row_sums) instead of writing partial sums.
template <int MODE>
__device__ __forceinline__ void gemv_direct2(const DevTensor &t, const Tables32 &tb, uint32_t *ring_mem, uint32_t wave_first) {
    constexpr int GPH = 16;                                // groups of four symbols per half block of 64 symbols
    const uint32_t lane = threadIdx.x & 63u;
    if (wave_first >= t.n_chunks) return;
    const uint32_t C = t.chunk_symbols;
    const uint32_t k = wave_first + lane;
    uint32_t nsym = 0;
    if (k < t.n_chunks) {
        const uint64_t left = t.n - static_cast<uint64_t>(k) * C;
        nsym = left < C ? static_cast<uint32_t>(left) : C;
    }
    const bool fast = nsym == C;                           // a shorter last segment takes the element-by-element path
    Ring2 r;
    r.stale = Tables32::stale;
    r.stream = t.stream;
    r.last_blk = t.stream_bytes - 16u;
    r.ring = (lds_v32)(ring_mem + lane);
    // a lane without a full segment decodes the start of the stream along with the others; nothing of it is stored
    ring2_fill<false>(r, fast ? seg_start(t, k) : 0);
    const uint32_t cols = t.cols;
    const uint16_t *xvec = t.x;
    const uint32_t max_len = t.max_len;
    const float zf = static_cast<float>(t.zero_point);    // exact: the host rejects |z| > 2^24
    const float scale = t.scale;
    const uint64_t flat0 = static_cast<uint64_t>(k) * C;
    uint32_t col = fast ? static_cast<uint32_t>(flat0 % cols) : 0u;    // column of the half block's first symbol
    uint32_t row = fast ? static_cast<uint32_t>(flat0 / cols) : 0u;    // the row the lane is in
    const bool starts_row = col == 0;
    float acc = 0.0f, first = 0.0f, end_sum = 0.0f;
    bool crossed = false;                                  // a row end has been passed
    bool ended = false;                                    // a row ended in this half block: end_sum holds its sum
    // eight activations per piece; a piece never straddles a row end (cols % 8 == 0, segments start at multiples of 64)
    u32x4 xb[8];
    auto ask_x = [&](uint32_t c0) {
#pragma unroll
        for (uint32_t p = 0; p < 8; ++p) {
            uint32_t c = c0 + 8u * p;
            c -= c >= cols ? cols : 0u;
            xb[p] = *(global_u4_ptr)(xvec + c);
        }
    };
    // two products per instruction: the table entries hold symbol - zero_point as bf16, x is bf16 as it stands
    // (the halves of v go through scalars: a bit cast applied to a vector's element reads element 0 whichever is named)
    auto mul4 = [&](u32x2 v, uint32_t xa, uint32_t xc) {
        const uint32_t lo = v.x, hi = v.y;
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, lo), __builtin_bit_cast(bf16x2, xa), acc, false);
        acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, hi), __builtin_bit_cast(bf16x2, xc), acc, false);
    };
    ask_x(col);
    const uint32_t halves = C / 64u;
    // eight groups as one stretch of straight-line code; PART says which eight of the half block's sixteen
    auto eight = [&](auto part_tag) __attribute__((always_inline)) {
        constexpr int PART = decltype(part_tag)::value;
#pragma unroll
        for (int gg = 0; gg < GPH / 2; ++gg) {
            const int g = PART * (GPH / 2) + gg;
            if (g % kTripGroups == 0)
                if (__builtin_expect(ring_short(r, kTripBits - 64), 0)) ring_reload(r);
            const u32x2 v4 = ring_group_wide(r, tb, max_len, zf);
            const u32x4 xv = xb[g / 2];
            mul4(v4, (g & 1) ? xv.z : xv.x, (g & 1) ? xv.w : xv.y);
            if (g & 1) {
                // a row ends behind this piece (at most once per half block: cols >= 64): its sum is set
                // aside without a branch, so that the groups stay one stretch of code
                const uint32_t piece = g / 2;
                const bool row_end = col + 8u * piece + 8u == cols;
                end_sum = row_end ? acc : end_sum;
                acc = row_end ? 0.0f : acc;
                ended |= row_end;
            }
        }
    };
    for (uint32_t h = 0; h < halves; ++h) {
        eight(std::integral_constant<int, 0>{});
        ring2_topup(r);                                    // the short ring is topped up after every eight groups
        eight(std::integral_constant<int, 1>{});
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(ended) != 0, 0)) {
            if (ended) {
                if (!crossed && !starts_row) {
                    first = end_sum;                       // the head fragment
                } else if (fast) {                         // a whole row
                    const float y = end_sum * scale;
                    if (gemv_f32(MODE)) reinterpret_cast<float *>(t.out)[row] = y;
                    else reinterpret_cast<uint16_t *>(t.out)[row] = static_cast<uint16_t>(bf16_bits(y));
                }
                crossed = true;
                row += 1u;
                ended = false;
            }
        }
        col += 64u;
        col -= col >= cols ? cols : 0u;
        if (h + 1 < halves) ask_x(col);
        ring2_topup(r);
    }
    if (t.row_lanes) {
        wave_row_sums<MODE>(t, k, fast, crossed ? first : acc);
    } else if (fast) {
        if (!crossed) {
            t.partials[2 * static_cast<uint64_t>(k)] = acc;              // the segment lies inside one row
        } else {
            if (!starts_row) t.partials[2 * static_cast<uint64_t>(k)] = first;
            if (col != 0) t.partials[2 * static_cast<uint64_t>(k) + 1] = acc;   // the segment ends inside a row
        }
    } else if (nsym) {
        gemv_segment<MODE>(t, tb, k);
    }
}

// The GEMV kernels need the tables and the scratch table only.
struct alignas(256) RingMem { uint32_t ring[kRingDwords * 64]; };
// which modes decode on the short ring (decode_rows2)
constexpr bool short_ring(int mode) { return mode == kModeF32 || mode == kModeBF16; }
struct alignas(256) Ring2Mem { uint32_t ring[kRing2Dwords * 64]; };
template <int MODE, bool GEMV = is_gemv(MODE), bool SHORT = short_ring(MODE), bool WIDE = wide_gemv(MODE)>
struct SmemFor { Tables tb; WaveMem<Cfg<MODE>::row> wm[Cfg<MODE>::waves]; };
template <int MODE> struct SmemFor<MODE, true, false, false> { Tables tb; RingMem wm[Cfg<MODE>::waves]; };
template <int MODE> struct SmemFor<MODE, true, false, true> { Tables32 tb; Ring2Mem wm[Cfg<MODE>::waves]; };
template <int MODE> struct SmemFor<MODE, false, true, false> { Tables tb; WaveMem2 wm[Cfg<MODE>::waves]; };

// Does the tensor go through decode_rows?  Segments must tile into blocks; for the
// GEMV, pieces of eight must not straddle a matrix row and a segment must touch at
// most two rows.
template <int MODE>
__device__ __forceinline__ bool rows_fit(const DevTensor &t) {
    if (t.chunk_symbols % Cfg<MODE>::spb != 0) return false;
    if constexpr (is_gemv(MODE)) return t.cols % 8 == 0 && t.cols >= 64;
    return true;
}

// Segments [first, end) of a tensor that does not fit the row path: one lane per
// segment, element by element, the whole workgroup striding over them.
template <int MODE, class TB>
__device__ __forceinline__ void scalar_chunks(const DevTensor &t, const TB &tb, uint32_t first, uint32_t end) {
    constexpr uint32_t WG = 64 * Cfg<MODE>::waves;
    for (uint32_t k = first + threadIdx.x; k < end; k += WG) {
        if constexpr (is_gemv(MODE)) {
            gemv_segment<MODE>(t, tb, k);
        } else {
            const uint64_t left = t.n - static_cast<uint64_t>(k) * t.chunk_symbols;
            decode_scalar<MODE>(t, tb, k, left < t.chunk_symbols ? static_cast<uint32_t>(left) : t.chunk_symbols);
        }
    }
}

// One tensor per launch: workgroup b builds the tables and takes `wg_units` units
// (kUnit segments each, one unit per wavefront; at most as many as it has
// wavefronts) from unit b * wg_units on.
template <int MODE, bool FIND, bool FLAT>
__device__ __forceinline__ void single_body(const DevTensor &t, uint32_t wg_units) {
    constexpr uint32_t WG = 64 * Cfg<MODE>::waves;
    __shared__ SmemFor<MODE> sm;
    // the per-wave symbol counts of the build live in the first wave's buffers, which are not in use yet
    build_tables<WG, kPairMode<MODE>>(t, sm.tb, reinterpret_cast<uint32_t *>(sm.wm));
    const uint32_t first = blockIdx.x * wg_units * kUnit;
    if (rows_fit<MODE>(t)) {
        const uint32_t wave = threadIdx.x >> 6;
        if (wave < wg_units) {
            if constexpr (wide_gemv(MODE)) gemv_direct2<MODE>(t, sm.tb, sm.wm[wave].ring, first + wave * kUnit);
            else if constexpr (is_gemv(MODE)) gemv_direct<MODE>(t, sm.tb, sm.wm[wave].ring, first + wave * kUnit);
            else if constexpr (short_ring(MODE)) decode_rows2<MODE, FIND, FLAT>(t, sm.tb, sm.wm, first + wave * kUnit);
            else decode_rows<MODE, FIND>(t, sm.tb, sm.wm, first + wave * kUnit);
        }
    } else {
        const uint32_t end = first + wg_units * kUnit;
        scalar_chunks<MODE>(t, sm.tb, first, end < t.n_chunks ? end : t.n_chunks);
    }
}

// Many tensors per launch.  A unit is kUnit consecutive segments of one tensor:
// what a wavefront decodes at a time.  The work list has one item per
// `item_units` units of a tensor (fewer at the tensor's end), in tensor order;
// workgroup b of G takes the items [b * n / G, (b + 1) * n / G): a few stretches
// of one tensor each.  Per stretch it loads the tensor's tables, then its wavefronts take a unit each and draw
// further ones from a counter in LDS until the stretch is used up.  The wavefronts of a workgroup do not run equally
// fast (fourteen of them share four SIMDs unevenly; lanes meet long codes at different
// times), so a fixed split would leave the faster ones waiting.
template <int MODE>
__device__ __forceinline__ void batch_body(const DevTensor *__restrict__ tensors, const WorkItem *__restrict__ items,
                                           uint32_t n_items, uint32_t item_units) {
    constexpr uint32_t WG = 64 * Cfg<MODE>::waves;
    __shared__ SmemFor<MODE> sm;
    __shared__ uint32_t next_unit;
    const uint32_t lo = static_cast<uint32_t>(static_cast<uint64_t>(blockIdx.x) * n_items / gridDim.x);
    const uint32_t hi = static_cast<uint32_t>(static_cast<uint64_t>(blockIdx.x + 1) * n_items / gridDim.x);
    uint32_t i = lo;
    while (i < hi) {
        const WorkItem it = items[i];
        const DevTensor &t = tensors[it.tensor];
        // the stretch ends with the tensor or with the workgroup's share
        const uint32_t left_in_tensor = (t.n_chunks - it.first + kUnit - 1) / kUnit;
        const uint64_t share = static_cast<uint64_t>(hi - i) * item_units;
        const uint32_t n_units = left_in_tensor < share ? left_in_tensor : static_cast<uint32_t>(share);
        // The units beyond the stretch's last whole round (a unit per wavefront), where the tensor is described
        // a second time with finer lanes (t.fine): they are drawn as 2^fine_shift times as many short ones, so
        // that the wavefronts run out of work at nearly the same time instead of most of them idling for the
        // length of a whole segment.
        const DevTensor *tf = &t;
        uint32_t n_coarse = n_units, n_all = n_units, fine_first = 0;
        if (!is_gemv(MODE) && t.fine) {                      // (the GEMV's descriptions have none)
            tf = &tensors[t.fine];
            const uint32_t refined = n_units % static_cast<uint32_t>(Cfg<MODE>::waves);   // what does not fill a round
            n_coarse = n_units - refined;
            fine_first = (it.first + n_coarse * kUnit) << t.fine_shift;
            uint64_t fine_end = static_cast<uint64_t>(it.first + n_units * kUnit) << t.fine_shift;
            if (fine_end > tf->n_chunks) fine_end = tf->n_chunks;
            n_all = n_coarse + static_cast<uint32_t>((fine_end - fine_first + kUnit - 1) / kUnit);
        }
        __syncthreads();                                     // nobody reads the previous tables or the counter any more
        // Built once when the launch was prepared.  (Every launch that
        // comes here has been prepared with tables.  A build in an else branch, never taken, decided the register
        // allocation: 20 spilled vector registers in the 8-bit product against 6 without, 3 and 4 against none
        // for packed nibbles and fp32; the step over 32 layers of 8-bit products 6510 -> 6232 us.)
        if constexpr (wide_gemv(MODE)) {
            // (one piece after the other: asked for at once they cost the product loop five more spilled registers)
            for (uint32_t j = threadIdx.x; j < sizeof(sm.tb) / 16u; j += WG) reinterpret_cast<u32x4 *>(&sm.tb)[j] = ((global_u4_ptr)t.tables)[j];
        } else {
            copy_tables<sizeof(sm.tb), WG>(&sm.tb, t.tables);
        }
        __syncthreads();
        if (rows_fit<MODE>(t)) {
            // A wavefront's first unit has its own number: a stretch of fewer units than wavefronts is spread evenly over
            // the four SIMDs.  Drawn from the counter, the first units go to whichever wavefronts leave the barrier
            // first, often two of one SIMD, and which these are changes with any change to the code in front.
            // Measured: 4-bit product with four units per workgroup 31.3 -> 26.1 us, with one 25.9 -> 25.6;
            // 8-bit product with six 66.0 -> 60.7; the step over 32 layers of 4-bit products 4622 -> 4254 us.
            if (threadIdx.x == 0) next_unit = Cfg<MODE>::waves;
            __syncthreads();
            for (uint32_t u = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); u < n_all;) {
                const bool fine = !is_gemv(MODE) && u >= n_coarse;
                const DevTensor &d = fine ? *tf : t;
                const uint32_t first = fine ? fine_first + (u - n_coarse) * kUnit : it.first + u * kUnit;
                if constexpr (wide_gemv(MODE)) gemv_direct2<MODE>(d, sm.tb, sm.wm[threadIdx.x >> 6].ring, first);
                else if constexpr (is_gemv(MODE)) gemv_direct<MODE>(d, sm.tb, sm.wm[threadIdx.x >> 6].ring, first);
                else if constexpr (short_ring(MODE)) decode_rows2<MODE>(d, sm.tb, sm.wm, first);
                else decode_rows<MODE>(d, sm.tb, sm.wm, first);
                if ((threadIdx.x & 63u) == 0) u = atomicAdd(&next_unit, 1u);
                u = __builtin_amdgcn_readfirstlane(u);
            }
        } else {
            const uint32_t end = it.first + n_units * kUnit;
            scalar_chunks<MODE>(t, sm.tb, it.first, end < t.n_chunks ? end : t.n_chunks);
        }
        i += (n_units + item_units - 1) / item_units;
    }
}

template <int MODE, bool FIND, bool FLAT>
__global__ __launch_bounds__(64 * Cfg<MODE>::waves) void k_single(const DevTensor t, uint32_t wg_units) {
    single_body<MODE, FIND, FLAT>(t, wg_units);
}
template <int MODE>
__global__ __launch_bounds__(64 * Cfg<MODE>::waves) void k_batch(const DevTensor *__restrict__ tensors,
                                                                 const WorkItem *__restrict__ items, uint32_t n_items,
                                                                 uint32_t item_units) {
    batch_body<MODE>(tensors, items, n_items, item_units);
}

// The lookup tables of the tensors of a prepared launch, built once (workgroup b: tensor b) and kept in
// memory for the launch's workgroups to load.  Workgroups behind the tensors' write the work list, where the host has not:
// `step` lanes an item, tensor by tensor.
template <int MODE>
__global__ __launch_bounds__(64 * Cfg<MODE>::waves) void k_tables(const DevTensor *__restrict__ tensors, uint32_t count,
                                                                  WorkItem *__restrict__ items, uint32_t n_items, uint32_t step) {
    constexpr uint32_t WG = 64 * Cfg<MODE>::waves;
    __shared__ SmemFor<MODE> sm;
    if (blockIdx.x >= count) {
        const uint32_t at = (blockIdx.x - count) * WG + threadIdx.x;
        uint32_t i = 0, rest = at;
        for (uint32_t n; i < count; rest -= n, ++i) {
            n = static_cast<uint32_t>((static_cast<uint64_t>(tensors[i].n_chunks) + step - 1u) / step);
            if (rest < n) break;
        }
        if (at < n_items && i < count) items[at] = WorkItem{i, rest * step};
        return;
    }
    const DevTensor &t = tensors[blockIdx.x];
    build_tables<WG, kPairMode<MODE>>(t, sm.tb, reinterpret_cast<uint32_t *>(sm.wm));
    static_assert(sizeof(sm.tb) % 16 == 0, "copied in 16-byte steps");
    const u32x4 *src = reinterpret_cast<const u32x4 *>(&sm.tb);
    u32x4 *dst = static_cast<u32x4 *>(t.tables);
    for (uint32_t j = threadIdx.x; j < sizeof(sm.tb) / 16u; j += WG) dst[j] = src[j];
}

// ---------------------------------------------------------------- segments shared by a wavefront's lanes
// Small launches (k_shared, k_shared_batch).  What bounds them is not the bytes but one lane's serial chain of lookups, so
// 2^share_shift lanes share a segment, about 64 symbols each, and a lookup answers up to four codes at once.
//   1. The unit's part of the stream (the segments of a wavefront lie side by side) comes into LDS in whole lines.
//   2. Each lane takes an equal stretch of its segment's bits and counts the codes that start in it, from a guessed first
//      bit: Huffman codes fall into step with the true boundaries within a few codes.  Then a lane whose neighbour ended
//      elsewhere than it began counts its stretch again from there, until all agree.  Lane 0 of a segment begins at a true
//      boundary and every round settles at least one more lane, so the starts are true whatever the data (one round as a
//      rule; as many as lanes where a run of one symbol keeps the guesses out of step, of which few count: share_settle).
//   3. The counts say where each lane's symbols belong; it decodes its stretch once more and leaves them there, in LDS.
//   4. The whole wavefront turns the unit's symbols, now in order, into output: consecutive 16 bytes by consecutive lanes,
//      or rows of the product.
// A lane's chain is three times 64 symbols at about 2.9 a lookup instead of a segment's length at one a lookup.
constexpr int kMulti = 12;               // stream bits that index the table of several codes
constexpr uint32_t kShareSymbols = 64;   // symbols of a lane, about
constexpr uint32_t kShareWaves = 16;
constexpr uint32_t kShareMost = 8192;    // most symbols of a segment: its symbols and its stream have to fit into LDS
constexpr uint32_t kTried = 12;          // starts of which a lane keeps what it counted from them, where lanes do not agree at once
constexpr uint32_t kShareLeast = 48u * kShareSymbols;   // fewest symbols of a unit's segments (share_fits)
// A unit's symbols in LDS: a byte each, and four free bytes behind each 64.
__host__ __device__ constexpr uint32_t share_symbol_bytes(uint32_t symbols) { return (symbols / 16u * 17u + 15u) / 16u * 16u; }
static_assert(64u * 4u * kTried <= share_symbol_bytes(kShareLeast), "a unit's symbols leave room for the starts that its lanes tried");

// Entry of the table of several codes: the next codes that kMulti bits hold in full, at most four.
// x: their symbols, first one lowest.  y: bits 0..5 their lengths' sum, bits 8..10 their number, from bit 12 on, four bits
// each, the lengths' sums up to the first, second and third code, 15 from the last code on.  All zero: a longer code.
constexpr uint32_t kLimits = 8;          // longer codes of up to kMulti + kLimits bits are told apart by one look at their limits
struct alignas(16) ShareMem {
    u32x2 multi[1 << kMulti];
    u32x4 limits[kLimits / 4];           // see share_long
    TablesTail tail;                     // the canonical tables; with what follows, a Tables while the tables are built
    uint8_t pool[160u * 1024u - (sizeof(u32x2) << kMulti) - 4u * kLimits - sizeof(TablesTail)];
    static constexpr uint32_t table_bytes = 160u * 1024u - sizeof(pool);   // all in front of the pool
    __device__ __forceinline__ Tables &building() { return *reinterpret_cast<Tables *>(&tail); }
};
static_assert(sizeof(ShareMem) == 160u * 1024u && sizeof(Tables) <= sizeof(TablesTail) + sizeof(ShareMem::pool) &&
              sizeof(TablesTail) % 16 == 0 && ShareMem::table_bytes <= sizeof(Tables32), "all of a compute unit's LDS; the tables fit the workspace");

typedef uint32_t __attribute__((address_space(3))) *lds_w32;
typedef u32x4 __attribute__((address_space(3))) *lds_128;

// Symbol i of a unit, four a dword: sixteen dwords and one free, or lanes 64 symbols apart would write to four banks only.
__device__ __forceinline__ uint32_t share_at(uint32_t dword) { return dword + (dword >> 4); }

// Puts the table of several codes together from the first-level table (1024 lanes, four entries each), and the limits of the
// longer codes: limit j is the first value, of 32 stream bits in code order, that no code of up to kMulti + 1 + j bits has.
__device__ __forceinline__ void build_multi(ShareMem &sm) {
    const Tables &tb = sm.building();
    // (a lane's four entries side by side: a chain of lookups each)
    static_assert((1u << kMulti) == 4u * 64u * kShareWaves, "four entries a lane");
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t i = k * 64u * kShareWaves + threadIdx.x;
        uint32_t w = i, bits = 0, n = 0, syms = 0, ends = 0xfff000u;
        bool more = true;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            const uint32_t e = tb.lut[w];                        // (zeros behind the index bits: only codes within them count)
            const uint32_t len = entry_len(e);
            more = more && len != 0 && bits + len <= static_cast<uint32_t>(kMulti);
            if (more) {
                if (j != 0) ends = (ends & ~(15u << (8 + 4 * j))) | (bits << (8 + 4 * j));
                syms |= entry_sym(e) << (8 * j);
                bits += len;
                w >>= len;
                n = j + 1;
            }
        }
        sm.multi[i] = n ? u32x2{syms, bits | (n << 8) | ends} : u32x2{0u, 0u};
    }
    if (threadIdx.x < kLimits) {
        const uint32_t l = kMulti + 1 + threadIdx.x;
        const uint64_t v = static_cast<uint64_t>(tb.first[l] + tb.cnt[l]) << (32u - l);
        reinterpret_cast<uint32_t *>(sm.limits)[threadIdx.x] = v < 0xffffffffu ? static_cast<uint32_t>(v) : 0xffffffffu;
    }
}

// Where a lane reads its segment's stream.
struct ShareReader {
    uint64_t base;              // absolute bit of the segment's start
    uint32_t lds_bit;           // and its bit in the wavefront's copy
    bool in_lds;                // the copy holds the whole unit (else: straight from memory)
    lds_p32 words;
};

// At least 57 stream bits from bit `rel` of the segment on.
__device__ __forceinline__ uint64_t share_window(const DevTensor &t, const ShareReader &r, uint32_t rel) {
    if (__builtin_expect(!r.in_lds, 0)) return load_bits57(t, r.base + rel);
    const uint32_t p = r.lds_bit + rel;
    const lds_p32 src = r.words + (p >> 5);
    const uint32_t w0 = src[0], w1 = src[1], w2 = src[2];
    return static_cast<uint64_t>(__builtin_amdgcn_alignbit(w1, w0, p)) | (static_cast<uint64_t>(__builtin_amdgcn_alignbit(w2, w1, p)) << 32);
}

// The code at bit `rel`, longer than kMulti bits.  Canonical codes grow with their length, so the number of limits that its
// bits have reached is its length; one in 64 to 500 codes comes here (one in two groups of a wavefront has such a lane).
__device__ __forceinline__ uint32_t share_long(const DevTensor &t, const ShareMem &sm, const ShareReader &r, uint32_t rel) {
    const uint32_t window = static_cast<uint32_t>(share_window(t, r, rel)), v = __brev(window);
    uint32_t l = kMulti + 1;
#pragma unroll
    for (uint32_t j = 0; j < kLimits; ++j) l += v >= sm.limits[j / 4][j % 4] ? 1u : 0u;
    if (__builtin_expect(l > kMulti + kLimits && t.max_len > kMulti + kLimits, 0))
        return decode_canonical(sm.tail, window, kMulti + kLimits + 1, t.max_len);
    l = l < t.max_len ? l : t.max_len;                           // (the last limit of a full code is one too low)
    const uint32_t d = (v >> (32u - l)) - sm.tail.first[l];
    return d < sm.tail.cnt[l] ? pack_entry(sm.tail.sorted[sm.tail.offs[l] + d], l) : pack_entry(0, 1);   // not a code: keep moving
}

// A lane's symbols on their way into the unit's, which are zero at first: whole dwords, to which lanes that share one add
// their bytes.
struct ShareWriter {
    lds_w32 out;
    uint32_t dword;             // next one to write
    uint32_t fill;              // bytes of it that have passed, 0..3
    uint64_t held;
    __device__ __forceinline__ void begin(lds_w32 o, uint32_t i) { out = o; dword = i >> 2; fill = i & 3u; held = 0; }
    __device__ __forceinline__ void flush() {
        __hip_atomic_fetch_or(out + share_at(dword), static_cast<uint32_t>(held), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    // n <= 4 symbols (the bytes behind them are zero)
    __device__ __forceinline__ void put(uint32_t syms, uint32_t n) {
        held |= static_cast<uint64_t>(syms) << (8u * fill);
        fill += n;
        if (fill >= 4u) {
            flush();
            held >>= 32;
            ++dword;
            fill -= 4u;
        }
    }
};

// The codes that start in [rel, limit): four lookups a window while the lane has kMulti bits to go, then, for the end of the
// stretch, one a window of which only the codes that start in front of the limit count.  Moves rel behind the last of them
// and adds their number to `count`.  WRITE: their symbols go to `out`.
template <bool WRITE>
__device__ __forceinline__ void share_pass(const DevTensor &t, const ShareMem &sm, const ShareReader &r, uint32_t &rel, uint32_t limit,
                                           uint32_t &count, ShareWriter &out) {
    int32_t room = static_cast<int32_t>(limit - rel);            // (negative: the lane begins behind its limit)
    while (__builtin_amdgcn_ballot_w64(room >= kMulti) != 0) {
        uint64_t w = share_window(t, r, limit - static_cast<uint32_t>(room));
        bool miss = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x2 e = sm.multi[static_cast<uint32_t>(w) & ((1u << kMulti) - 1u)];
            const bool on = room >= kMulti;
            const uint32_t y = on ? e.y : 0u;
            if (WRITE) out.put(on ? e.x : 0u, (y >> 8) & 7u);
            w >>= y & 63u;
            room -= static_cast<int32_t>(y & 63u);
            count += (y >> 8) & 7u;
            miss = on && y == 0;                                 // (a lane that meets a longer code does not move any more)
        }
        if (__builtin_amdgcn_ballot_w64(miss) != 0) {
            if (miss) {
                const uint32_t e = share_long(t, sm, r, limit - static_cast<uint32_t>(room));
                if (WRITE) out.put(entry_sym(e), 1u);
                room -= static_cast<int32_t>(entry_len(e));
                ++count;
            }
        }
    }
    while (__builtin_amdgcn_ballot_w64(room > 0) != 0) {
        if (room > 0) {
            const uint32_t at = limit - static_cast<uint32_t>(room);
            const u32x2 e = sm.multi[static_cast<uint32_t>(share_window(t, r, at)) & ((1u << kMulti) - 1u)];
            uint32_t syms = e.x, len = e.y & 63u, n = (e.y >> 8) & 7u;
            if (__builtin_expect(n == 0, 0)) {
                const uint32_t l = share_long(t, sm, r, at);
                syms = entry_sym(l);
                len = entry_len(l);
                n = 1;
            } else {
                const uint32_t left = static_cast<uint32_t>(room), c1 = (e.y >> 12) & 15u, c2 = (e.y >> 16) & 15u, c3 = (e.y >> 20) & 15u;
                const uint32_t k = left <= c1 ? 1u : left <= c2 ? 2u : left <= c3 ? 3u : 4u;
                const uint32_t upto = left <= c1 ? c1 : left <= c2 ? c2 : left <= c3 ? c3 : len;
                n = k < n ? k : n;
                len = upto < len ? upto : len;
                syms &= ~0u >> (32u - 8u * n);
            }
            if (WRITE) out.put(syms, n);
            room -= static_cast<int32_t>(len);
            count += n;
        }
    }
    rel = limit - static_cast<uint32_t>(room);
}

// m symbols in LDS, the tensor's from u0 (a multiple of 128) on, to the output: 16 bytes a lane and step.
template <int MODE>
__device__ __forceinline__ void share_store(const DevTensor &t, lds_w32 sym, uint64_t u0, uint32_t m) {
    constexpr uint32_t SYMS = MODE == kModeF32 ? 4u : MODE == kModeBF16 ? 8u : MODE == kModeU8 ? 16u : 32u;   // per 16 bytes
    const uint32_t lane = threadIdx.x & 63u;
    uint8_t *const out = static_cast<uint8_t *>(t.out) + ((u0 * OutTraits<MODE>::ebits) >> 3);
    const float zf = static_cast<float>(t.zero_point), scale = t.scale;
    const uint32_t whole = m / SYMS;
    for (uint32_t j = lane; j < whole; j += 64u) {
        uint32_t src[SYMS / 4];                                  // (they lie within one run of sixteen dwords)
#pragma unroll
        for (uint32_t i = 0; i < SYMS / 4; ++i) src[i] = sym[share_at(j * (SYMS / 4)) + i];
        u32x4 v;
        if constexpr (MODE == kModeU8) {
            v = u32x4{src[0], src[1], src[2], src[3]};
        } else if constexpr (MODE == kModeU4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t a = src[2 * i], b = src[2 * i + 1];
                const uint32_t pa = (a & 0x000f000fu) | ((a >> 4) & 0x00f000f0u), pb = (b & 0x000f000fu) | ((b >> 4) & 0x00f000f0u);
                v[i] = __builtin_amdgcn_perm(pb, pa, 0x06040200u);
            }
        } else {
            float f[SYMS];
#pragma unroll
            for (uint32_t i = 0; i < SYMS; ++i) f[i] = (static_cast<float>((src[i / 4] >> (8 * (i % 4))) & 0xffu) - zf) * scale;
            if constexpr (MODE == kModeF32) {
                v = u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const f32x2 pr = {f[2 * i], f[2 * i + 1]};
                    v[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));   // round to nearest even
                }
            }
        }
        *(global_u4_wptr)(out + j * 16u) = v;
    }
    // the tensor's end
    for (uint32_t i = whole * SYMS + lane; i < m; i += 64u) {
        const uint32_t q = (sym[share_at(i >> 2)] >> (8u * (i & 3u))) & 0xffu;
        if constexpr (MODE == kModeU8) out[i] = static_cast<uint8_t>(q);
        if constexpr (MODE == kModeU4)
            if ((i & 1u) == 0) out[i >> 1] = static_cast<uint8_t>((q & 0xfu) | (i + 1u < m ? (sym[share_at(i >> 2)] >> (8u * (i & 3u) + 4u)) & 0xf0u : 0u));
        if constexpr (MODE == kModeF32) reinterpret_cast<float *>(out)[i] = dequant(q, t.zero_point, scale);
        if constexpr (MODE == kModeBF16) reinterpret_cast<uint16_t *>(out)[i] = static_cast<uint16_t>(bf16_bits(dequant(q, t.zero_point, scale)));
    }
}

// The rows of the product that m symbols in LDS, the tensor's from u0 on, hold in full or in part.  As many
// lanes take a row as have eight columns each of it (a power of two, at most all), several rows at a time where rows are short.
// cols and m are multiples of 8, u0 of 128: eight columns lie side by side, and their activations on 16 bytes.
// A row that does not lie in the unit as a whole leaves a partial sum, as k_fix_* reads it (fix_symbols: the unit's).
template <int MODE>
__device__ __forceinline__ void share_rows(const DevTensor &t, lds_w32 sym, uint32_t unit, uint64_t u0, uint32_t m) {
    const uint32_t lane = threadIdx.x & 63u, cols = t.cols;
    uint32_t per = 1;
    while (per < 64u && per * 8u < cols) per <<= 1;
    const uint32_t r0 = static_cast<uint32_t>(u0 / cols), r1 = static_cast<uint32_t>((u0 + m - 1u) / cols);
    const uint32_t head = static_cast<uint32_t>(u0 - static_cast<uint64_t>(r0) * cols);      // columns of row r0 in front of the unit
    const float zf = static_cast<float>(t.zero_point);
    for (uint32_t r = r0 + lane / per; r <= r1; r += 64u / per) {
        // the row's columns [c0, c1) are the unit's symbols from s0 on
        const uint64_t before = static_cast<uint64_t>(r - r0) * cols;
        const uint32_t c0 = r == r0 ? head : 0u;
        const uint32_t s0 = r == r0 ? 0u : static_cast<uint32_t>(before - head);
        const uint32_t c1 = cols - c0 < m - s0 ? cols : c0 + (m - s0);
        float acc = 0.0f;
#pragma unroll 4
        for (uint32_t i = 8u * (lane & (per - 1u)); i < c1 - c0; i += 8u * per) {
            const u32x4 xv = *(global_u4_ptr)(t.x + c0 + i);
            const uint32_t at = share_at((s0 + i) >> 2);
            const uint32_t q[2] = {sym[at], sym[at + 1u]};           // (an even dword and the next: within one run)
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j) {
                const float d = static_cast<float>((q[j / 4] >> (8 * (j % 4))) & 0xffu) - zf;
                const float x = __uint_as_float((j & 1u) ? xv[j / 2] & 0xffff0000u : xv[j / 2] << 16);
                acc = __builtin_fmaf(d, x, acc);
            }
        }
        for (uint32_t d = 1; d < per; d <<= 1) acc += __shfl_xor(acc, d, 64);
        if ((lane & (per - 1u)) == 0) {
            if (c0 == 0 && c1 == cols) {
                const float y = acc * t.scale;
                if (gemv_f32(MODE)) reinterpret_cast<float *>(t.out)[r] = y;
                else reinterpret_cast<uint16_t *>(t.out)[r] = static_cast<uint16_t>(bf16_bits(y));
            } else {
                t.partials[2 * static_cast<uint64_t>(unit) + (r == r0 ? 0 : 1)] = acc;
            }
        }
    }
}

// What a wavefront keeps about the unit it works on.
struct ShareUnit {
    ShareReader r;
    uint32_t nsym, span;        // the symbols of the lane's segment, and its bits in the stream
};

__device__ __forceinline__ void share_look_up(const DevTensor &t, uint32_t unit, ShareUnit &u) {
    const uint32_t at = (threadIdx.x & 63u) >> t.share_shift, k = unit * t.share_per + at;
    u.nsym = u.span = 0;
    u.r.base = 0;
    if (at < t.share_per && k < t.n_chunks) {
        const uint64_t left = t.n - static_cast<uint64_t>(k) * t.chunk_symbols;
        u.nsym = left < t.chunk_symbols ? static_cast<uint32_t>(left) : t.chunk_symbols;
        u.r.base = seg_start(t, k);
        uint64_t bits;
        if (t.sub_shift) {
            bits = t.sub[k];
        } else {
            const uint64_t end = t.offsets[k + 1];
            bits = end > u.r.base ? end - u.r.base : 0;
        }
        const uint64_t most = static_cast<uint64_t>(u.nsym) * ENTRO_MAX_CODE_LEN;
        u.span = static_cast<uint32_t>(bits < most ? bits : most);
    }
}

// The rounds of a wavefront whose lanes have not agreed after two of them, until they do.  A run of one symbol sends the same
// few starts, as many as its code has bits, from lane to lane: a lane keeps what it found from each (in the symbols' place,
// which holds zeros before and after: word d * 64 + lane for the start d bits behind its guess) and counts from it once.
// (A neighbour passes its limit by less than a code's 32 bits.)
// Measured, counting in every round -> now (a lane per segment).  Single calls, 4096 segments of 8192 symbols, a run in each:
// to bf16 from 8 bits 528 -> 299 us (542), to nibbles from 4 bits 361 -> 231 (261).  Prepared 4-bit products: 40960 segments of 4096, a
// run in each, 1172 -> 482 (149); 28672 of 1024, one in 64 of them a run, 119 -> 73 (45).  Without runs the calls take what they
// took (within 0.6 %; 1 % more with the first rounds in one loop with these).
__device__ __forceinline__ void share_settle(const DevTensor &t, const ShareMem &sm, const ShareReader &r, lds_w32 sym, uint32_t guess,
                                             uint32_t limit, uint32_t part, uint32_t &from, uint32_t &upto, uint32_t &count) {
    const uint32_t lane = threadIdx.x & 63u;
    ShareWriter none;
    for (;;) {
        const uint32_t before = __shfl_up(upto, 1, 64);
        const uint32_t want = part == 0 ? 0u : before;
        const bool todo = want != from;
        if (__builtin_amdgcn_ballot_w64(todo) == 0) break;
        if (from - guess < kTried) sym[(from - guess) * 64u + lane] = (1u << 31) | (count << 5) | (upto - limit);
        const uint32_t known = todo && want - guess < kTried ? sym[(want - guess) * 64u + lane] : 0u;
        const bool look = todo && known == 0;
        uint32_t rel = look ? want : limit, n = 0;
        if (__builtin_amdgcn_ballot_w64(look) != 0) share_pass<false>(t, sm, r, rel, limit, n, none);
        upto = look ? rel : todo ? limit + (known & 31u) : upto;
        count = look ? n : todo ? (known << 1) >> 6 : count;
        from = want;
    }
#pragma unroll
    for (uint32_t d = 0; d < kTried; ++d) sym[d * 64u + lane] = 0u;
    wave_sync_lds();
}

// One unit, looked up already, by one wavefront with `wave_bytes` of LDS at `sym`.
template <int MODE>
__device__ __forceinline__ void share_unit(const DevTensor &t, const ShareMem &sm, lds_w32 sym, uint32_t wave_bytes, uint32_t unit, ShareUnit &u) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t sh = t.share_shift, parts = 1u << sh, part = lane & (parts - 1u), S = t.chunk_symbols;
    const uint32_t unit_symbols = S * t.share_per, symbol_bytes = share_symbol_bytes(unit_symbols), copy_bytes = wave_bytes - symbol_bytes;
    const lds_w32 copy = sym + symbol_bytes / 4u;
    ShareReader &r = u.r;
    const uint32_t nsym = u.nsym, span = u.span;
    r.words = (lds_p32)copy;
    // the unit's part of the stream, and zeros for its symbols (its first segment is always there: no unit is empty)
    const uint64_t lo = (static_cast<uint64_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(r.base >> 32))) << 32 |
                         __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(r.base))) & ~uint64_t{127};
    const uint32_t room = 8u * (copy_bytes - 32u);               // (a window reaches some bytes behind a segment's end)
    const bool held = nsym == 0 || (r.base - lo <= room && r.base - lo + span <= room);   // (also in front of lo: not held)
    r.in_lds = __builtin_amdgcn_ballot_w64(!held) == 0;
    r.lds_bit = nsym != 0 ? static_cast<uint32_t>(r.base - lo) : 0u;
    if (r.in_lds)
        for (uint32_t b = lane; b < copy_bytes / 16u; b += 64u)
            *(lds_128)(copy + b * 4u) = load_block(t.stream, static_cast<uint32_t>(lo >> 3) + b * 16u, t.stream_bytes - 16u);
    for (uint32_t b = lane; b < symbol_bytes / 16u; b += 64u) *(lds_128)(sym + b * 4u) = u32x4{0u, 0u, 0u, 0u};
    wave_sync_lds();
    const uint32_t guess = static_cast<uint32_t>((static_cast<uint64_t>(span) * part) >> sh);
    const uint32_t limit = static_cast<uint32_t>((static_cast<uint64_t>(span) * (part + 1u)) >> sh);
    ShareWriter out;
    uint32_t from = guess, upto = guess, count = 0;
    share_pass<false>(t, sm, r, upto, limit, count, out);
    bool agreed = false;
    for (uint32_t round = 0; round < 2u; ++round) {
        const uint32_t before = __shfl_up(upto, 1, 64);
        const uint32_t want = part == 0 ? 0u : before;           // (never in front of the guess: the neighbour passed its limit)
        const bool todo = want != from;
        agreed = __builtin_amdgcn_ballot_w64(todo) == 0;
        if (agreed) break;
        uint32_t rel = todo ? want : limit, n = 0;
        share_pass<false>(t, sm, r, rel, limit, n, out);
        upto = todo ? rel : upto;
        count = todo ? n : count;
        from = want;
    }
    if (__builtin_expect(!agreed, 0)) share_settle(t, sm, r, sym, guess, limit, part, from, upto, count);
    uint32_t sum = count;
    for (uint32_t d = 1; d < parts; d <<= 1) {
        const uint32_t y = __shfl_up(sum, d, 64);
        sum += part >= d ? y : 0u;
    }
    // an offset table that does not fit the stream: the segment's first lane decodes it from its start
    const bool bad = __shfl(sum, static_cast<int>(lane | (parts - 1u)), 64) != nsym;
    out.begin(sym, (lane >> sh) * S + (bad ? 0u : sum - count));
    uint32_t rel = bad ? limit : from, n = 0;
    share_pass<true>(t, sm, r, rel, limit, n, out);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad) != 0, 0)) {
        if (bad && part == 0) {
            uint64_t pos = r.base;
            for (uint32_t i = 0; i < nsym; ++i) {
                const uint32_t e = decode_canonical(sm.tail, static_cast<uint32_t>(load_bits57(t, pos)), 1u, t.max_len);
                out.put(entry_sym(e), 1u);
                pos += entry_len(e);
            }
        }
    }
    if (out.fill != 0) out.flush();                              // (never behind the unit's symbols: fill is 0 at their end)
    wave_sync_lds();
    const uint64_t u0 = static_cast<uint64_t>(unit) * unit_symbols, left = t.n - u0;
    const uint32_t m = left < unit_symbols ? static_cast<uint32_t>(left) : unit_symbols;
    if constexpr (is_gemv(MODE)) share_rows<MODE>(t, sym, unit, u0, m);
    else share_store<MODE>(t, sym, u0, m);
    wave_sync_lds();
}

// One tensor per launch: every workgroup builds the tables, then `waves` of its wavefronts take units.
template <int MODE>
__global__ __launch_bounds__(64 * kShareWaves) void k_shared(const DevTensor t, uint32_t waves, uint32_t wave_bytes) {
    __shared__ ShareMem sm;
    const uint32_t wave = threadIdx.x >> 6;
    const lds_w32 sym = (lds_w32)(sm.pool + wave * wave_bytes);
    ShareUnit u;
    uint32_t unit = blockIdx.x * waves + wave;
    const bool works = wave < waves && unit < t.share_units;
    if (works) share_look_up(t, unit, u);                        // (on its way while the tables are built)
    build_tables<64 * kShareWaves, false, false>(t, sm.building(), reinterpret_cast<uint32_t *>(sm.multi));   // (scratch: not in use yet)
    build_multi(sm);
    __syncthreads();
    if (!works) return;
    for (;;) {
        share_unit<MODE>(t, sm, sym, wave_bytes, unit, u);
        unit += gridDim.x * waves;
        if (unit >= t.share_units) break;
        share_look_up(t, unit, u);
    }
}

// Units of a work item: about 64 segments, as in the other kernels' lists.
__host__ __device__ constexpr uint32_t share_item_units(uint32_t per) { return (kUnit + per - 1u) / per; }

// Many tensors per launch: workgroup b of G takes the items [b * n / G, (b + 1) * n / G), stretches of one tensor each, whose
// tables, built when the launch was prepared (k_share_tables), it loads; `waves` of its wavefronts take units in turn.
template <int MODE>
__global__ __launch_bounds__(64 * kShareWaves) void k_shared_batch(const DevTensor *__restrict__ tensors, const WorkItem *__restrict__ items,
                                                                   uint32_t n_items, uint32_t waves, uint32_t wave_bytes) {
    __shared__ ShareMem sm;
    const uint32_t lo = static_cast<uint32_t>(static_cast<uint64_t>(blockIdx.x) * n_items / gridDim.x);
    const uint32_t hi = static_cast<uint32_t>(static_cast<uint64_t>(blockIdx.x + 1) * n_items / gridDim.x);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const lds_w32 sym = (lds_w32)(sm.pool + wave * wave_bytes);
    uint32_t i = lo;
    while (i < hi) {
        const WorkItem it = items[i];
        const DevTensor &t = tensors[it.tensor];
        const uint32_t item_units = share_item_units(t.share_per), left = t.share_units - it.first;
        const uint64_t share = static_cast<uint64_t>(hi - i) * item_units;
        const uint32_t n_units = left < share ? left : static_cast<uint32_t>(share);
        uint32_t at = wave < waves ? wave : n_units;
        ShareUnit u;
        if (at < n_units) share_look_up(t, it.first + at, u);    // (on its way while the tables come in)
        __syncthreads();                                         // nobody reads the previous tables any more
        copy_tables<ShareMem::table_bytes, 64u * kShareWaves>(&sm, t.tables);
        __syncthreads();
        while (at < n_units) {
            share_unit<MODE>(t, sm, sym, wave_bytes, it.first + at, u);
            at += waves;
            if (at < n_units) share_look_up(t, it.first + at, u);
        }
        i += (n_units + item_units - 1u) / item_units;
    }
}

// The tables of k_shared_batch, for the tensors of a prepared launch (workgroup b: tensor b).
__global__ __launch_bounds__(64 * kShareWaves) void k_share_tables(const DevTensor *__restrict__ tensors) {
    __shared__ ShareMem sm;
    const DevTensor &t = tensors[blockIdx.x];
    build_tables<64 * kShareWaves, false, false>(t, sm.building(), reinterpret_cast<uint32_t *>(sm.multi));
    build_multi(sm);
    __syncthreads();
    const u32x4 *src = reinterpret_cast<const u32x4 *>(&sm);
    u32x4 *dst = static_cast<u32x4 *>(t.tables);
    for (uint32_t j = threadIdx.x; j < ShareMem::table_bytes / 16u; j += 64u * kShareWaves) dst[j] = src[j];
}

// Second stage of the GEMV: the partial sums of a row that straddles lanes are added up by sixteen lanes,
// lane j taking every sixteenth of them in segment order, then the sixteen in a fixed tree (the same sum
// in the same order on every run).
constexpr int kFixWG = 256;                                   // threads of a workgroup
constexpr int kFixRows = kFixWG / 16;                         // and the rows it sums

template <int MODE>
__device__ __forceinline__ void fix_row(const DevTensor &t, uint32_t row, uint32_t j) {
    const bool live = row < t.rows;
    uint32_t k_lo = 1, k_hi = 0;
    if (live) {
        const uint64_t lo = static_cast<uint64_t>(row) * t.cols;
        k_lo = static_cast<uint32_t>(lo / t.fix_symbols);
        k_hi = static_cast<uint32_t>((lo + t.cols - 1) / t.fix_symbols);
    }
    float acc = 0.0f;
    for (uint64_t k = static_cast<uint64_t>(k_lo) + j; k <= k_hi; k += 16u) {
        const uint32_t first_row = static_cast<uint32_t>((k * t.fix_symbols) / t.cols);
        acc += t.partials[2 * k + (first_row == row ? 0 : 1)];
    }
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) acc += __shfl_xor(acc, m, 64);
    if (!live || k_lo == k_hi || j != 0) return;             // (a whole row inside one lane's segment is stored already)
    const float y = acc * t.scale;
    if (gemv_f32(MODE)) reinterpret_cast<float *>(t.out)[row] = y;
    else reinterpret_cast<uint16_t *>(t.out)[row] = static_cast<uint16_t>(bf16_bits(y));
}

template <int MODE>
__global__ __launch_bounds__(kFixWG) void k_fix_single(const DevTensor t) {
    fix_row<MODE>(t, blockIdx.x * kFixRows + threadIdx.x / 16u, threadIdx.x & 15u);
}

// A part of a launch's table that comes as a kernel argument.
struct PutWords {
    static constexpr uint32_t most = 960;                     // (arguments of a kernel: 4 KB)
    uint32_t w[most];
};
__global__ __launch_bounds__(PutWords::most) void k_put(uint32_t *__restrict__ dst, uint32_t n, const PutWords words) {
    if (threadIdx.x < n) dst[threadIdx.x] = words.w[threadIdx.x];
}

template <int MODE>
__global__ __launch_bounds__(kFixWG) void k_fix_batch(const DevTensor *__restrict__ tensors,
                                                   const WorkItem *__restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    fix_row<MODE>(tensors[it.tensor], it.first + threadIdx.x / 16u, threadIdx.x & 15u);
}

// ---------------------------------------------------------------- products of prepared launches: lanes of about 64 symbols
// k_fine.  A token step is a chain of small launches, each as long as one lane's serial chain of lookups behind the launch and
// its cold reads.  With a lane per piece of 256 or 512 symbols that chain took 15 to 50 us, and sharing pieces as k_shared does
// costs three passes.  So the preparation of a launch, which a program pays once for all its steps, walks the streams once
// (k_fine_index) and notes where the codes of every `fine_len` symbols begin: 32 bits per 64 symbols, kept beside the tables.
//   A wavefront's unit is 64 lanes of fine_len symbols side by side, whole pieces of the tensor.  A lane decodes its symbols as
//   two chains, interleaved (what limits a compute unit are the round trips to LDS, and LDS holds sixteen wavefronts at most).
//   Its stream, at most 64 bytes, is asked for in one go a unit ahead and lies in a column of LDS: no ring, no refills.
//   Rows are cut into lanes so that a wavefront holds whole rows, or goes through a row unit by unit, where the shape allows it.
// The noted places are a guess, as in k_shared: the unit's first bit is read from the tensor's own tables on every run, every
// chain has to end where the next one begins, and so by induction all of them are true, whatever the streams hold by now.  A
// unit of lanes whose codes are longer than their columns is decoded from the same places with columns that are filled as it goes
// (fine_again), and proven likewise; a unit whose places are not true is walked piece by piece from the tensor's tables (fine_walk),
// which also notes its places anew, and decoded from there.
//   Measured, a lane per piece -> now, us a launch.  8 bits, 3.5 bits a symbol: 25 M symbols in rows of 4096 36 -> 22, 16.8 M 31 -> 16,
// 117 M 74 -> 46, 58.7 M in rows of 14336 44 and 5 for the second stage -> 34; the step over 32 layers 6098 -> 3881.  4 bits, 1.55
// bits a symbol: 9.4 M symbols in rows of 3072, shared by k_shared_batch before, 28 -> 10; the step over 32 layers 4035 -> 1863.
// Rows that begin and end inside units, second stage included (kFineParts), 8 bits: 60.5 M symbols in rows of 5504 73 -> 35, 41.5 M of
// 13824 55 -> 28, 0.86 M of 2880 31 -> 15; 4 bits: 60.5 M of 5504 43 -> 22, 0.86 M of 2880 19 -> 10; no shape was found that loses.
//   What bounds a large launch now: the LDS pipe is busy in 0.68 of the cycles (over half of that bank conflicts of the lookups) and
// the vector ALUs in 0.62; a small one: about 6 us of cold reads one behind the other (item, description, places, stream) and what
// a launch takes by itself.
constexpr uint32_t kFineWaves = 16;
constexpr uint32_t kFineData = 16;                       // dwords of stream that a lane holds
constexpr uint32_t kFineX = 14848;                       // columns of the activations that LDS has room for
constexpr uint32_t kFineEnd = 32u * (kFineData + 1u);    // position of the first bit behind them
constexpr uint32_t kFineRow = 1, kFineUnits = 2, kFineParts = 3;   // a unit holds whole rows cut into 2^i lanes; a row is whole units; any

struct alignas(16) FineMem {
    Tables32 tb;
    // Dword d of a lane's column lies at (16 * wave + d) * 64 + lane; 1 to 16 hold its stream.  A window's stale bits come from
    // dword 0 and what it reads behind the lane's codes from 17 to 19: whatever the neighbours have there.
    uint32_t col[(kFineWaves * kFineData + 4u) * 64u];
    u32x4 x[kFineX / 8u];
    uint32_t next;
};
static_assert(sizeof(FineMem) <= 160u * 1024u, "one workgroup per compute unit");
typedef u32x4 __attribute__((aligned(4))) u32x4_a4;
typedef const void __attribute__((address_space(1))) *global_void_ptr;
typedef void __attribute__((address_space(3))) *lds_void_ptr;
typedef const u32x4_a4 __attribute__((address_space(1))) *global_u4a4_ptr;
typedef const uint32_t __attribute__((address_space(1))) *global_u32_ptr;

// The code at the start of `w` among those of `from` bits and more.  (Not decode_canonical: a call, even one that is never made,
// takes half the registers of the kernel around it.)
__device__ __forceinline__ uint32_t fine_search(const TablesTail &tb, uint32_t w, uint32_t from, uint32_t max_len) {
    const uint32_t v = __brev(w);
#pragma unroll 1
    for (uint32_t l = from; l <= max_len; ++l) {
        const uint32_t d = (v >> (32 - l)) - tb.first[l];
        if (d < tb.cnt[l]) return pack_entry(tb.sorted[tb.offs[l] + d], l);
    }
    return pack_entry(0, 1);                             // not a code (corrupt stream): keep moving
}
// One code, whatever its length.
template <bool PAIR>
__device__ __forceinline__ uint32_t fine_single(const Tables32 &tb, uint32_t w, uint32_t max_len) {
    uint32_t e = PAIR ? tb.lut2[w & ((1u << kSingleBits) - 1u)] : tb.lut[w & kL1Mask];
    if (entry_len(e) == 0) {
        e = PAIR ? 0u : lookup_l2(tb, e, w);
        if (e == 0) e = fine_search(tb, w, PAIR ? kSingleBits + 1 : kL1 + 1, max_len);
    }
    return e;
}

// A place as it is noted.  (Of a unit of 2^16 bits and more, whose lanes cannot all hold their codes, the lower half: fine_again's
// caller counts how often it begins anew.  A chain has at most 32 codes of 32 bits.)
__device__ __forceinline__ uint16_t fine_note(uint32_t bits) { return static_cast<uint16_t>(bits); }

// The places of all chains of the tensors of a prepared launch (blockIdx.x: the tensor, described with a lane per piece), noted
// on a walk through the pieces with the block path's reader.
// What it costs a preparation, against a walk by single loads from memory (which reads every line many times over): a launch over
// 58.7 M symbols of 8 bits 692 -> 83 us, over 50 M symbols of 4 bits 247 -> 50 us.
template <bool PAIR>
__global__ __launch_bounds__(64 * kFineWaves) void k_fine_index(const DevTensor *__restrict__ tensors) {
    __shared__ struct {
        Tables tb;
        uint32_t ring[kFineWaves][kRing2Dwords * 64];
    } sm;
    constexpr uint32_t SPG = PAIR ? 8u : 4u;             // symbols of a group
    const DevTensor &t = tensors[blockIdx.x];
    if (blockIdx.y * 1024u >= t.n_chunks) return;
    build_tables<64 * kFineWaves, PAIR>(t, sm.tb, &sm.ring[0][0]);
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    const uint32_t P = t.chunk_symbols, L = t.fine_len, A = t.fine_first, per = t.fine_pieces, max_len = t.max_len;
    uint16_t *index = reinterpret_cast<uint16_t *>(t.fine_index);
    for (uint32_t first = blockIdx.y * 1024u + wave * 64u; first < t.n_chunks; first += gridDim.y * 1024u) {
        const bool live = first + lane < t.n_chunks;
        const uint32_t k = live ? first + lane : first;  // (a lane without a piece walks the wavefront's first and notes nothing)
        const uint32_t unit = k / per, in_unit = (k - unit * per) * P;
        const uint64_t left = t.n - static_cast<uint64_t>(k) * P;
        const uint32_t nsym = !live ? 0u : left < P ? static_cast<uint32_t>(left) : P;
        const uint32_t base = static_cast<uint32_t>(seg_start(t, unit * per));
        uint32_t at = in_unit / L, i = in_unit - at * L; // the lane of the unit and the symbol of it that the walk has come to
        at += unit * 64u;
        Ring2 r;
        r.stale = Tables::stale;
        r.stream = t.stream;
        r.last_blk = t.stream_bytes - 16u;
        r.ring = (lds_v32)(sm.ring[wave] + lane);
        ring2_fill<false>(r, seg_start(t, k));
        for (uint32_t s = 0; s < P; s += 8u * SPG) {
#pragma unroll
            for (uint32_t g = 0; g < 8; ++g) {
                if (g % kTripGroups == 0)
                    if (__builtin_expect(ring_short(r, kTripBits - 64), 0)) ring_reload(r);
                if (PAIR || g % 2u == 0) {               // a chain begins at a multiple of eight symbols
                    if ((i == 0 || i == A) && s + g * SPG < nsym)
                        index[2u * at + (i ? 1u : 0u)] = fine_note((r.start64 << 3) + r.q + r.stale - base);
                    i += 8u;
                    at += i == L ? 1u : 0u;
                    i = i == L ? 0u : i;
                }
                ring_group<PAIR>(r, sm.tb, max_len);
            }
            ring2_topup(r);
        }
    }
}

// Wide pair tables: the first level's entry holds both symbols' values as bf16, the second one in the high half, and the codes'
// length (at most 14) in the low four bits, which an integer of at most 16 in magnitude leaves zero.
__global__ __launch_bounds__(1024) void k_fine_pairs(const DevTensor *__restrict__ tensors) {
    __shared__ Tables tb;
    __shared__ uint32_t wcnt[4 * (ENTRO_MAX_CODE_LEN + 1)];
    const DevTensor &t = tensors[blockIdx.x];
    build_tables<1024, true>(t, tb, wcnt);
    Tables32 *dst = static_cast<Tables32 *>(t.tables);
    static_assert(sizeof(TablesTail) % 16 == 0 && sizeof(TablesTail) / 16u <= 1024u, "copied in 16-byte steps");
    if (threadIdx.x < sizeof(TablesTail) / 16u)
        reinterpret_cast<u32x4 *>(dst)[threadIdx.x] = reinterpret_cast<const u32x4 *>(&tb)[threadIdx.x];
    for (uint32_t i = threadIdx.x; i < (1u << kL1); i += 1024u) {
        const uint32_t e = tb.lut[i], both = entry_sym(e);
        const uint32_t lo = __float_as_uint(static_cast<float>(static_cast<int32_t>(both & 15u) - t.zero_point)) >> 16;
        const uint32_t hi = __float_as_uint(static_cast<float>(static_cast<int32_t>(both >> 4) - t.zero_point)) & 0xffff0000u;
        dst->lut[i] = entry_len(e) ? hi | lo | entry_len(e) : 0u;
    }
}

// What a wavefront holds of a unit before it decodes it.
struct FineUnit {
    uint32_t places;        // where the lane's two chains begin, in bits from the unit's first: 16 bits each
    uint32_t next;          // where the next lane's first chain begins (of the last lane: its own)
    uint32_t q;             // where the lane's first chain begins in its column
    uint32_t sub;           // an entry of the entry-point table (lanes 0..14)
    uint64_t offset;        // of the segment
    u32x4 data[kFineData / 4];
};

// Ask for what says where the unit's codes are ...
__device__ __forceinline__ void fine_ask(const DevTensor &t, uint32_t unit, FineUnit &u) {
    const uint32_t lane = threadIdx.x & 63u, fl = unit * 64u + lane;
    u.places = ((global_u32_ptr)t.fine_index)[fl < t.fine_n ? fl : t.fine_n - 1u];
    const uint32_t k = unit * t.fine_pieces, sh = t.sub_shift, c = k >> sh, before = k - (c << sh);
    u.offset = ((global_u64_ptr)t.offsets)[c];
    u.sub = 0;
    if (sh) {
        const uint32_t v = ((global_u16_ptr)t.sub)[(static_cast<uint64_t>(c) << sh) + (lane < before ? lane : 0u)];
        u.sub = lane < before ? v : 0u;
    }
}

// ... and for the codes themselves.
__device__ __forceinline__ void fine_load(const DevTensor &t, FineUnit &u) {
    uint32_t add = u.sub;                                // (the first row of sixteen lanes holds all entries)
    add += __builtin_amdgcn_update_dpp(0u, add, 0x111, 0xf, 0xf, true);
    add += __builtin_amdgcn_update_dpp(0u, add, 0x112, 0xf, 0xf, true);
    add += __builtin_amdgcn_update_dpp(0u, add, 0x114, 0xf, 0xf, true);
    add += __builtin_amdgcn_update_dpp(0u, add, 0x118, 0xf, 0xf, true);
    const uint64_t base = u.offset + __builtin_amdgcn_readlane(add, 15);
    const uint32_t a = u.places & 0xffffu;
    u.next = __shfl_down(a, 1, 64);
    const uint64_t pos = base + a;
    u.q = (static_cast<uint32_t>(pos) & 31u) + 32u - Tables32::stale;
    const uint32_t at = static_cast<uint32_t>(pos >> 5) << 2, last = t.stream_bytes - 16u;
#pragma unroll
    for (uint32_t i = 0; i < kFineData / 4u; ++i) {
        // (a piece that begins behind the last sixteen bytes, which are padding, holds no code)
        const uint32_t off = at + 16u * i;
        u.data[i] = *(global_u4a4_ptr)(t.stream + (off < last ? off : last));
    }
}

__device__ __forceinline__ uint64_t fine_window(lds_v32 col, uint32_t q) {
    uint32_t d = q >> 5;
    d = d < kFineData + 1u ? d : kFineData + 1u;
    const lds_p32 src = (lds_p32)(col + d * 64u);
    const uint32_t w0 = src[0], w1 = src[64], w2 = src[128];
    const uint32_t lo = __builtin_amdgcn_alignbit(w1, w0, q);
    const uint32_t hi = __builtin_amdgcn_alignbit(w2, w1, q);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// A group is four lookups of one chain: four symbols, or eight of 4 bits.
template <bool PAIR>
struct FineGroup {
    static constexpr int kVals = PAIR ? 4 : 2;
    static constexpr uint32_t kLenMask = PAIR ? 15u : 63u;
    uint32_t v[kVals];                                   // the symbols' values as bf16, two per dword, first one lowest
};

__device__ __forceinline__ uint32_t bf16_of(uint32_t sym, float zf) { return __float_as_uint(static_cast<float>(sym) - zf) >> 16; }

// The group of a lane that met a code (or pair of codes) that the first level does not hold: `w` is the window as it stopped in
// front of it, `e` its miss entry.  The window still holds the 20 bits that the second level needs.
template <bool PAIR>
__device__ __forceinline__ uint32_t fine_careful(lds_v32 col, const Tables32 &tb, uint32_t max_len, float zf, uint32_t q, uint64_t w,
                                                 uint32_t e0, uint32_t e1, uint32_t e2, uint32_t e, FineGroup<PAIR> &g) {
    constexpr uint32_t M = FineGroup<PAIR>::kLenMask;
    const uint32_t l0 = e0 & M, l1 = e1 & M, l2 = e2 & M;
    uint32_t i = l0 == 0 ? 0u : l1 == 0 ? 1u : l2 == 0 ? 2u : 3u;
    q += l0 + l1 + l2;                                   // (from the long code on the entries have no length)
    for (;;) {
        const bool miss = (e & M) == 0;
        uint32_t val;
        if constexpr (PAIR) {
            val = e & ~M;
            uint32_t len = e & M, used = len;
            if (miss) {
                // (a window holds a code of 15 bits behind three lookups, and three lookups behind such a code)
                if (max_len > 15u) w = fine_window(col, q);
                const uint32_t s0 = fine_single<true>(tb, static_cast<uint32_t>(w >> Tables32::stale), max_len);
                w = fine_window(col, q + entry_len(s0));
                const uint32_t s1 = fine_single<true>(tb, static_cast<uint32_t>(w >> Tables32::stale), max_len);
                used = entry_len(s1);
                len = entry_len(s0) + used;
                val = bf16_of(entry_sym(s0) & 15u, zf) | (bf16_of(entry_sym(s1) & 15u, zf) << 16);
            }
            q += len;
            g.v[0] = i == 0 ? val : g.v[0];
            g.v[1] = i == 1 ? val : g.v[1];
            g.v[FineGroup<PAIR>::kVals - 2] = i == 2 ? val : g.v[FineGroup<PAIR>::kVals - 2];
            g.v[FineGroup<PAIR>::kVals - 1] = i == 3 ? val : g.v[FineGroup<PAIR>::kVals - 1];
            w >>= used;
        } else {
            if (miss) {
                e = lookup_l2(tb, e, static_cast<uint32_t>(w >> Tables32::stale));
                if (__builtin_expect(e == 0, 0)) e = fine_search(tb, static_cast<uint32_t>(fine_window(col, q) >> Tables32::stale), kL1 + 1, max_len);
            }
            q += entry_len(e);
            val = bf16_of(entry_sym(e), zf);
            const uint32_t keep = (i & 1u) ? 0x0000ffffu : 0xffff0000u, put = (i & 1u) ? val << 16 : val;
            g.v[0] = i < 2u ? (g.v[0] & keep) | put : g.v[0];
            g.v[1] = i >= 2u ? (g.v[1] & keep) | put : g.v[1];
            w >>= entry_len(e);
        }
        if (++i == 4u) return q;
        if (miss && (!PAIR || max_len > 15u)) w = fine_window(col, q);
        e = lut_at(tb, static_cast<uint32_t>(w) & (kL1Mask << Tables32::stale));
    }
}

// One group of either chain, without a branch per lookup, the chains' round trips side by side.
template <bool PAIR>
__device__ __forceinline__ void fine_groups(lds_v32 col, const Tables32 &tb, uint32_t max_len, float zf, uint32_t &qa, uint32_t &qb,
                                            FineGroup<PAIR> &ga, FineGroup<PAIR> &gb) {
    constexpr uint32_t kMask = kL1Mask << Tables32::stale, M = FineGroup<PAIR>::kLenMask;
    uint64_t wa = fine_window(col, qa), wb = fine_window(col, qb);
    uint32_t a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a[i] = lut_at(tb, static_cast<uint32_t>(wa) & kMask);
        b[i] = lut_at(tb, static_cast<uint32_t>(wb) & kMask);
        if (i < 3) {
            wa >>= (a[i] & M);
            wb >>= (b[i] & M);
        }
    }
    uint32_t na, nb;
    if constexpr (PAIR) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ga.v[i] = a[i] & ~M;
            gb.v[i] = b[i] & ~M;
        }
        na = qa + (a[0] & M) + (a[1] & M) + (a[2] & M) + (a[3] & M);
        nb = qb + (b[0] & M) + (b[1] & M) + (b[2] & M) + (b[3] & M);
    } else {
        ga.v[0] = __builtin_amdgcn_perm(a[1], a[0], 0x07060302u);
        ga.v[1] = __builtin_amdgcn_perm(a[3], a[2], 0x07060302u);
        gb.v[0] = __builtin_amdgcn_perm(b[1], b[0], 0x07060302u);
        gb.v[1] = __builtin_amdgcn_perm(b[3], b[2], 0x07060302u);
        na = qa + ((a[0] + a[1] + a[2] + a[3]) & 0xffu);
        nb = qb + ((b[0] + b[1] + b[2] + b[3]) & 0xffu);
    }
    const bool ma = (a[3] & M) == 0, mb = (b[3] & M) == 0;      // (a miss entry's length stays until the group's end)
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(ma || mb) != 0, 0)) {
        // (one copy of the careful code for both chains)
#pragma unroll 1
        for (int c = 0; c < 2; ++c) {
            if (c ? mb : ma) {
                FineGroup<PAIR> g;
#pragma unroll
                for (int i = 0; i < FineGroup<PAIR>::kVals; ++i) g.v[i] = c ? gb.v[i] : ga.v[i];
                const uint32_t q = fine_careful<PAIR>(col, tb, max_len, zf, c ? qb : qa, c ? wb : wa, c ? b[0] : a[0], c ? b[1] : a[1],
                                                      c ? b[2] : a[2], c ? b[3] : a[3], g);
#pragma unroll
                for (int i = 0; i < FineGroup<PAIR>::kVals; ++i) {
                    ga.v[i] = c ? ga.v[i] : g.v[i];
                    gb.v[i] = c ? g.v[i] : gb.v[i];
                }
                na = c ? na : q;
                nb = c ? q : nb;
            }
        }
    }
    qa = na;
    qb = nb;
}

__device__ __forceinline__ float dot2(uint32_t v, uint32_t x, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v), __builtin_bit_cast(bf16x2, x), acc, false);
}

// `N` pieces of sixteen bytes of the stream, from absolute bit `pos` on, into the dwords that `col` is the first of.  Returns the
// position of that bit, as if they were dwords 1 and up of the lane's column.
template <uint32_t N>
__device__ __forceinline__ uint32_t fine_fill(const DevTensor &t, lds_v32 col, uint64_t pos) {
    const uint32_t at = static_cast<uint32_t>(pos >> 5) << 2, last = t.stream_bytes - 16u;
    u32x4 v[N];
#pragma unroll
    for (uint32_t i = 0; i < N; ++i) {
        const uint32_t off = at + 16u * i;
        v[i] = *(global_u4a4_ptr)(t.stream + (off < last ? off : last));
    }
#pragma unroll
    for (uint32_t j = 0; j < 4u * N; ++j) col[j * 64u] = v[j / 4][j % 4];
    return (static_cast<uint32_t>(pos) & 31u) + 32u - Tables32::stale;
}

// Half a column, dwords 1 to 8 or 9 to 16, filled behind a dword's end holds a group of the longest codes: four of 32 bits, or
// eight of 28 (fine_fits).  Does what is left of it, from position q on, hold one?
constexpr uint32_t kFineHalf = 8;
template <bool PAIR>
__device__ __forceinline__ bool fine_short(uint32_t q, uint32_t max_len) {
    return q + (PAIR ? 8u : 4u) * max_len > 32u * (kFineHalf + 1u) - Tables32::stale;
}

// The position behind the group of four lookups that begins at q.
template <bool PAIR>
__device__ __forceinline__ uint32_t fine_skip(lds_v32 col, const Tables32 &tb, uint32_t max_len, uint32_t q) {
    constexpr uint32_t M = FineGroup<PAIR>::kLenMask;
    uint64_t w = fine_window(col, q);
    uint32_t bits = 0, len = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        len = lut_at(tb, static_cast<uint32_t>(w) & (kL1Mask << Tables32::stale)) & M;
        w >>= len;
        bits += len;
    }
    if (__builtin_expect(len == 0, 0)) {                 // (a code that the first level does not hold ends the others' advance)
        bits = 0;
#pragma unroll 1
        for (int i = 0; i < (PAIR ? 8 : 4); ++i)
            bits += entry_len(fine_single<PAIR>(tb, static_cast<uint32_t>(fine_window(col, q + bits) >> Tables32::stale), max_len));
    }
    return q + bits;
}

// A unit whose noted places do not hold: its pieces are walked from the tensor's own tables, a lane each, and the places are noted
// anew.  Where the lane's two chains begin, in bits from the unit's first, is returned in a and b.  The stream comes through the
// first half of a lane's column; places lie in the second.
//   The lanes that are left over walk `ahead` - 1 units more, `stride` apart, that this workgroup has yet to come to, and note their
// places: buffers that have been given other contents have them all over.  A launch behind other contents, symbol by symbol from
// memory -> now: 16.8 M symbols of 3.6 bits in pieces of 256 121 -> 61 us, 58.7 M 367 -> 102.
template <bool PAIR>
__device__ __forceinline__ void fine_walk(const DevTensor &t, const Tables32 &tb, lds_v32 col, uint32_t max_len, uint32_t unit, uint32_t stride,
                                          uint32_t ahead, uint32_t &a, uint32_t &b) {
    constexpr uint32_t SPG = PAIR ? 8u : 4u;             // symbols of a group
    const uint32_t lane = threadIdx.x & 63u, P = t.chunk_symbols, L = t.fine_len, per = t.fine_pieces;
    uint32_t j = lane / per, of_unit = lane - j * per;
    const bool live = j < ahead && (j + 1u) * per <= 64u && (unit + j * stride) * per + of_unit < t.n_chunks;
    j = live ? j : 0u;                                   // (a lane without a piece walks the unit's first and notes nothing)
    of_unit = live ? of_unit : 0u;
    const uint32_t u = unit + j * stride, k = u * per + of_unit;
    const uint64_t left = t.n - static_cast<uint64_t>(k) * P, base = seg_start(t, u * per);
    const uint32_t nsym = !live ? 0u : left < P ? static_cast<uint32_t>(left) : P;
    const lds_v32 place = col - lane + (kFineHalf + 1u) * 64u;
    uint16_t *index = reinterpret_cast<uint16_t *>(t.fine_index) + 128u * static_cast<uint64_t>(u);
    uint32_t at = of_unit * P / L, i = of_unit * P - at * L, from = 0, q = 0;
    uint64_t pos = seg_start(t, k);
    wave_sync_lds();
#pragma unroll 1
    for (uint32_t s = 0; s < P; s += SPG) {
        if (s == 0 || __builtin_amdgcn_ballot_w64(fine_short<PAIR>(q, max_len)) != 0) {
            pos += q - from;
            from = q = fine_fill<kFineHalf / 4u>(t, col + 64u, pos);
        }
        if (s < nsym && (i == 0 || i == t.fine_first)) {
            const uint32_t bits = static_cast<uint32_t>(pos - base) + q - from, chain = i ? 1u : 0u;
            if (j == 0) place[chain * 64u + at] = bits;
            index[2u * at + chain] = fine_note(bits);
        }
        q = fine_skip<PAIR>(col, tb, max_len, q);
        i += SPG;
        at += i == L ? 1u : 0u;
        i = i == L ? 0u : i;
    }
    wave_sync_lds();
    a = place[lane];
    b = place[64u + lane];
    wave_sync_lds();
}

// Code by code through the stream from bit `start` behind `base` on, four of them a step, until every lane is at `limit` or behind:
// each(where a code begins, its length).  (A lane that is there goes on until the others are.)
template <bool PAIR, class F>
__device__ __forceinline__ void fine_codes(const DevTensor &t, const Tables32 &tb, lds_v32 col, uint32_t max_len, uint64_t base, uint32_t start,
                                           uint32_t limit, F each) {
    uint32_t at = start, q = 0;
    bool fill = true;
#pragma unroll 1
    while (__builtin_amdgcn_ballot_w64(at < limit) != 0) {
        if (fill || __builtin_amdgcn_ballot_w64(fine_short<PAIR>(q, max_len)) != 0) q = fine_fill<kFineHalf / 4u>(t, col + 64u, base + at);
        fill = false;
        uint64_t w = fine_window(col, q);
        uint32_t len[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t v = static_cast<uint32_t>(w >> Tables32::stale);
            len[i] = entry_len(PAIR ? tb.lut2[v & ((1u << kSingleBits) - 1u)] : tb.lut[v & kL1Mask]);
            w >>= len[i];
        }
        if (__builtin_expect(len[3] == 0, 0)) {          // (a code that the first level does not hold ends the others' advance)
            uint32_t to = q;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                len[i] = entry_len(fine_single<PAIR>(tb, static_cast<uint32_t>(fine_window(col, to) >> Tables32::stale), max_len));
                to += len[i];
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            each(at, len[i]);
            at += len[i];
            q += len[i];
        }
    }
}

// The same places, found with all lanes where a piece is many lanes' symbols: as in k_shared every lane counts the codes that begin
// in an equal stretch of its piece's bits, from a guessed one; a lane whose neighbour ended elsewhere than it began counts again
// from there, until all agree.  Then every lane knows which symbols are its own, and notes the places among them.  False (and
// nothing is noted) where lanes do not agree soon, or the counts are not the pieces'.
//   A launch behind other contents, fine_walk -> this, 8 bits: 16.8 M symbols in pieces of 4096 397 -> 71 us, of 1024 120 -> 65, of 512
// 79 -> 68, 58.7 M in pieces of 4096 747 -> 192; 4 bits: 9.4 M in pieces of 4096 210 -> 59, of 1024 72 -> 46, 25 M of 512 49 -> 92.
constexpr int kFineRounds = 6;
constexpr uint32_t kFineFind = 1024;                     // symbols of such a piece, and more
template <bool PAIR>
__device__ __forceinline__ bool fine_find(const DevTensor &t, const Tables32 &tb, lds_v32 col, uint32_t max_len, uint32_t unit, uint64_t base,
                                          uint32_t &a, uint32_t &b) {
    const uint32_t lane = threadIdx.x & 63u, P = t.chunk_symbols, L = t.fine_len, per = t.fine_pieces, of_piece = 64u / per;
    const uint32_t piece = lane / of_piece, j = lane - piece * of_piece, k = unit * per + piece;
    const bool live = piece < per && k < t.n_chunks;
    uint32_t start = 0, limit = 0, nsym = 0;
    bool fits = true;
    if (live) {
        const uint64_t left = t.n - static_cast<uint64_t>(k) * P, from = seg_start(t, k) - base;
        // (behind the last piece there is no entry point to read)
        const uint64_t to = (k + 1u < t.n_chunks ? seg_start(t, k + 1u) : ((global_u64_ptr)t.offsets)[(k >> t.sub_shift) + 1u]) - base;
        nsym = left < P ? static_cast<uint32_t>(left) : P;
        fits = to >= from && to - from <= 32u * nsym && from <= 32u * 64u * L;
        const uint32_t bits = fits ? static_cast<uint32_t>(to - from) : 0u;
        start = static_cast<uint32_t>(from) + bits * j / of_piece;
        limit = static_cast<uint32_t>(from) + bits * (j + 1u) / of_piece;
    }
    if (__builtin_amdgcn_ballot_w64(!fits) != 0) return false;
    uint32_t count = 0;
#pragma unroll 1
    for (int round = 0;; ++round) {
        uint32_t end = start;
        count = 0;
        fine_codes<PAIR>(t, tb, col, max_len, base, start, limit, [&](uint32_t at, uint32_t len) __attribute__((always_inline)) {
            count += at < limit ? 1u : 0u;
            end = at < limit ? at + len : end;
        });
        const uint32_t before = __shfl_up(end, 1, 64);
        const bool moves = live && j != 0 && before != start;
        if (__builtin_amdgcn_ballot_w64(moves) == 0) break;
        if (round == kFineRounds) return false;
        start = moves ? before : start;
    }
    uint32_t upto = count;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const uint32_t y = __shfl_up(upto, m, 64);
        upto += lane >= static_cast<uint32_t>(m) ? y : 0u;
    }
    const uint32_t first = live ? piece * of_piece : lane, before = __shfl(upto - count, first, 64);
    const bool whole = !live || j + 1u != of_piece || upto - before == nsym;
    if (__builtin_amdgcn_ballot_w64(!whole) != 0) return false;
    const uint32_t symbol = piece * P + upto - count - before;
    const lds_v32 place = col - lane + (kFineHalf + 1u) * 64u;
    uint16_t *index = reinterpret_cast<uint16_t *>(t.fine_index) + 128u * static_cast<uint64_t>(unit);
    uint32_t to = symbol / L, i = symbol - to * L, mine = count;     // (no more than were counted, whatever is read now)
    wave_sync_lds();
    fine_codes<PAIR>(t, tb, col, max_len, base, start, limit, [&](uint32_t at, uint32_t) __attribute__((always_inline)) {
        if (mine != 0 && (i == 0 || i == t.fine_first)) {
            const uint32_t chain = i ? 1u : 0u;
            place[chain * 64u + to] = at;
            index[2u * to + chain] = fine_note(at);
        }
        mine -= mine != 0 ? 1u : 0u;
        ++i;
        to += i == L ? 1u : 0u;
        i = i == L ? 0u : i;
    });
    wave_sync_lds();
    a = place[lane];
    b = place[64u + lane];
    wave_sync_lds();
    return true;
}

// The sum of a lane whose chains begin a and b bits behind the unit's first, whatever their length: half of its column for either
// chain, filled where that may not hold the next group.  a and b become where the chains end.  Groups, values and sums come in the
// order that k_fine's own loop has them in, so that a unit's sums are the same to the last bit, however its places have been found.
//   For units of lanes with more bits than a column, and those of walked pieces.  Rows of log-normal spread (0.8) at 4.8 bits a symbol
// on average, walked in every launch -> now: 16.8 M symbols 120 -> 29 us, 58.7 M 219 -> 54; a lane per piece takes 96 and 127.
template <bool PAIR, class X>
__device__ __forceinline__ float fine_again(const DevTensor &t, const Tables32 &tb, lds_v32 col, uint32_t max_len, float zf, uint64_t base,
                                            uint32_t &a, uint32_t &b, X activations) {
    const uint32_t pieces = t.fine_len / 8u, steps = (pieces + 1u) / 2u;
    uint32_t from = 0, from_b = 0, qa = 0, qb = 0, end_b = 0;
    uint64_t pos_a = base + a, pos_b = base + b;
    float acc = 0.0f;
#pragma unroll 1
    for (uint32_t s = 0; s < steps; ++s) {
        const u32x4 xa = activations(s);
        u32x4 xb = activations(steps + s < pieces ? steps + s : 0u);
        if (steps + s >= pieces) xb = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int h = 0; h < (PAIR ? 1 : 2); ++h) {
            if ((s == 0 && h == 0) ||
                __builtin_amdgcn_ballot_w64(fine_short<PAIR>(qa, max_len) || fine_short<PAIR>(qb - 32u * kFineHalf, max_len)) != 0) {
                pos_a += qa - from;
                pos_b += qb - from_b;
                from = qa = fine_fill<kFineHalf / 4u>(t, col + 64u, pos_a);
                from_b = qb = fine_fill<kFineHalf / 4u>(t, col + (kFineHalf + 1u) * 64u, pos_b) + 32u * kFineHalf;
            }
            FineGroup<PAIR> ga, gb;
            fine_groups<PAIR>(col, tb, max_len, zf, qa, qb, ga, gb);
#pragma unroll
            for (int v = 0; v < FineGroup<PAIR>::kVals; ++v) {
                acc = dot2(ga.v[v], xa[(PAIR ? 0 : 2 * h) + v], acc);
                acc = dot2(gb.v[v], xb[(PAIR ? 0 : 2 * h) + v], acc);
            }
        }
        if (steps + s < pieces) end_b = static_cast<uint32_t>(pos_b - base) + qb - from_b;
    }
    a = static_cast<uint32_t>(pos_a - base) + qa - from;
    b = end_b;
    return acc;
}

template <bool F32>
__device__ __forceinline__ void fine_store(const DevTensor &t, uint32_t row, float sum) {
    const float y = sum * t.scale;
    if (F32) reinterpret_cast<float *>(t.out)[row] = y;
    else reinterpret_cast<uint16_t *>(t.out)[row] = static_cast<uint16_t>(bf16_bits(y));
}

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_of(float v) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, ROWS, 0xf, true));
}

// The lanes' sums become rows.
template <bool F32>
__device__ __forceinline__ void fine_sums(const DevTensor &t, uint32_t quantum, uint32_t unit, float sum) {
    const uint32_t lane = threadIdx.x & 63u, fl = unit * 64u + lane, rl = t.row_lanes;
    const bool valid = fl < t.fine_n;
    float v = valid ? sum : 0.0f;
    if (t.fine_rows == kFineParts) {
        // lanes of a row side by side: running sums from the row's first lane in the unit, of which the last one counts
        const uint32_t row = fl / rl, in_row = fl - row * rl;
        const uint32_t run = in_row < lane ? in_row : lane;          // lanes of the row in front of this one in the unit
#pragma unroll
        for (uint32_t m = 1; m < 64u; m <<= 1) {
            const float up = __shfl_up(v, m, 64);
            v += run >= m ? up : 0.0f;
        }
        const bool row_ends = in_row + 1u == rl;
        if (valid && (row_ends || lane == 63u)) {
            if (row_ends && run == in_row) fine_store<F32>(t, row, v);
            else t.partials[2 * static_cast<uint64_t>(unit) + (run == lane ? 0 : 1)] = v;     // (the unit's first row or another)
        }
        return;
    }
    // a power of two of lanes side by side: their last one ends up with the sum
    const uint32_t across = t.fine_rows == kFineUnits ? 64u : rl;
    if (across > 1u) v += dpp_of<0x111, 0xf>(v);         // row_shr:1, 2, 4, 8: from the lane that far in front, in rows of sixteen
    if (across > 2u) v += dpp_of<0x112, 0xf>(v);
    if (across > 4u) v += dpp_of<0x114, 0xf>(v);
    if (across > 8u) v += dpp_of<0x118, 0xf>(v);
    if (across > 16u) v += dpp_of<0x142, 0xa>(v);        // row_bcast:15: a row's last lane to the next row
    if (across > 32u) v += dpp_of<0x143, 0xc>(v);        // row_bcast:31: lane 31 to the upper half
    if (valid && (lane & (across - 1u)) == across - 1u)
        fine_store<F32>(t, t.fine_rows == kFineUnits ? quantum : fl >> __builtin_ctz(rl), v);
}

// The column of the lane's first symbol.
__device__ __forceinline__ uint32_t fine_column(const DevTensor &t, uint32_t unit, uint32_t of_row) {
    const uint32_t lane = threadIdx.x & 63u, fl = unit * 64u + lane;
    if (t.fine_rows == kFineUnits) return (of_row * 64u + lane) * t.fine_len;
    if (t.fine_rows == kFineRow) return (lane & (t.row_lanes - 1u)) * t.fine_len;
    return fl % t.row_lanes * t.fine_len;
}

// Where piece j of the activations lies: turned within its eight where lanes are an even number of pieces apart (turn 7; else 0),
// so that eight lanes beside each other find theirs in different banks.
__device__ __forceinline__ uint32_t fine_x_at(uint32_t j, uint32_t turn) { return (j & ~7u) | ((j + ((j >> 3) & turn)) & 7u); }
__device__ __forceinline__ uint32_t fine_x_from(uint32_t j, uint32_t turn) { return (j & ~7u) | ((j - ((j >> 3) & turn)) & 7u); }

template <bool PAIR, bool F32>
__global__ __launch_bounds__(64 * kFineWaves) void k_fine(const DevTensor *__restrict__ tensors, const WorkItem *__restrict__ items,
                                                          uint32_t each, uint32_t rest) {
    __shared__ FineMem sm;
    constexpr uint32_t kTableVecs = sizeof(Tables32) / 16u, kTableSteps = (kTableVecs + 1023u) / 1024u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    const lds_v32 col = (lds_v32)(sm.col + wave * (kFineData * 64u) + lane);
    // the items [b * n / G, (b + 1) * n / G), n = each * G + rest (a 64-bit division takes longer than the whole prologue)
    const uint32_t lo = blockIdx.x * each + blockIdx.x * rest / gridDim.x;
    const uint32_t hi = (blockIdx.x + 1u) * each + (blockIdx.x + 1u) * rest / gridDim.x;
    for (uint32_t i = lo; i < hi;) {
        const WorkItem it = items[i];
        const DevTensor &t = tensors[it.tensor];
        const uint32_t left = t.fine_quanta - it.first, item_quanta = t.fine_item;
        const uint64_t share = static_cast<uint64_t>(hi - i) * item_quanta;
        const uint32_t n_quanta = left < share ? left : static_cast<uint32_t>(share);
        // The first unit by the wavefront's number.  Its places, its codes and its activations are asked for with the tables.
        uint32_t g = wave, of_row = 0;
        const bool some = g < n_quanta;
        uint32_t unit = (it.first + (some ? g : 0u)) * t.fine_units;
        FineUnit u;
        fine_ask(t, unit, u);
        // Tables and activations (of rows that fit) go straight to LDS.  Through registers the tables' pieces took twenty of them, and
        // some were spilled as they came; activations asked for by each lane where it needs them took 64 lines an instruction.
        const uint32_t x_pieces = t.cols / 8u, turn = (t.fine_len / 8u) & 1u ? 0u : 7u;
        const bool x_here = t.cols <= kFineX;
        if (i != lo) __syncthreads();                    // nobody reads the previous tables or the counter any more
#pragma unroll
        for (uint32_t s = 0; s < kTableSteps; ++s) {
            const uint32_t j = s * 1024u + threadIdx.x;
            if (j < kTableVecs)
                __builtin_amdgcn_global_load_lds((global_void_ptr)(static_cast<const u32x4 *>(t.tables) + j),
                                                 (lds_void_ptr)(reinterpret_cast<u32x4 *>(&sm.tb) + s * 1024u + wave * 64u), 16, 0, 0);
        }
        if (x_here) {
#pragma unroll
            for (uint32_t s = 0; s < 2; ++s) {
                const uint32_t j = s * 1024u + threadIdx.x, from = fine_x_from(j, turn);
                if (s * 1024u < x_pieces && from < x_pieces)
                    __builtin_amdgcn_global_load_lds((global_void_ptr)(reinterpret_cast<const u32x4 *>(t.x) + from),
                                                     (lds_void_ptr)(sm.x + s * 1024u + wave * 64u), 16, 0, 0);
            }
        }
        fine_load(t, u);
        if (threadIdx.x == 0) sm.next = kFineWaves;
        __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0): what goes to LDS is there
        __syncthreads();
        const uint32_t max_len = t.max_len, steps = (t.fine_len + 15u) / 16u, pieces = t.fine_len / 8u;
        const float zf = static_cast<float>(t.zero_point);
        auto activations = [&](uint32_t j) __attribute__((always_inline)) {          // piece j of them
            return x_here ? sm.x[fine_x_at(j, turn)] : *(global_u4_ptr)(reinterpret_cast<const char *>(t.x) + 16u * j);
        };
        u32x4 x[8];
        uint32_t x_col = 0xffffffffu;                    // the column that x holds
        float sum = 0.0f;
        bool more = some;
        while (more) {
#pragma unroll
            for (uint32_t j = 0; j < kFineData; ++j) col[(1u + j) * 64u] = u.data[j / 4][j % 4];
            const uint32_t here = unit * 64u + lane < t.fine_n ? fine_column(t, unit, of_row) : 0u;
            if (__builtin_amdgcn_ballot_w64(here != x_col) != 0) {
                // pieces of eight activations: the first `steps` of them are the first chain's, the others the second one's (zeros
                // where that is a piece shorter: it decodes on into nothing)
#pragma unroll
                for (uint32_t p = 0; p < 8; ++p) {
                    const uint32_t at = p < 4u ? p : steps + p - 4u;
                    x[p] = activations(here / 8u + (at < pieces ? at : 0u));
                }
#pragma unroll
                for (uint32_t p = 5; p < 8; ++p)
                    if (steps + p - 4u == pieces) x[p] = u32x4{0u, 0u, 0u, 0u};
                x_col = here;
            }
            // what comes next: the row's next unit, or one of another quantum
            const bool row_done = of_row + 1u == t.fine_units;
            uint32_t g_next = g;
            if (row_done) {
                if (lane == 0) g_next = atomicAdd(&sm.next, 1u);
                g_next = __builtin_amdgcn_readfirstlane(g_next);
                more = g_next < n_quanta;
            }
            const uint32_t unit_next = !row_done ? unit + 1u : more ? (it.first + g_next) * t.fine_units : unit;
            const uint32_t a = u.places & 0xffffu, b = u.places >> 16, next = u.next;
            const uint32_t q0 = u.q;
            fine_ask(t, unit_next, u);
            // Lanes whose codes do not fit their columns, as far as noted (which says nothing of the last lane): the unit is left to
            // fine_again.  By no steps rather than a branch around all of them, which made a step over 32 layers 1 % longer.
            const uint32_t q_mid = q0 + (b - a), q_next = q0 + (next - a);
            const bool longer = __builtin_amdgcn_ballot_w64(q_next > kFineEnd - Tables32::stale) != 0;
            const uint32_t steps_here = longer ? 0u : steps;
            uint32_t qa = q0, qb = q_mid, end_b = qb;
            float acc = 0.0f;
#pragma unroll
            for (uint32_t s = 0; s < 4; ++s) {
                if (s < steps_here) {
#pragma unroll
                    for (int h = 0; h < (PAIR ? 1 : 2); ++h) {
                        FineGroup<PAIR> ga, gb;
                        fine_groups<PAIR>(col, sm.tb, max_len, zf, qa, qb, ga, gb);
                        if constexpr (PAIR) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                acc = dot2(ga.v[v], x[s][v], acc);
                                acc = dot2(gb.v[v], x[4 + s][v], acc);
                            }
                        } else {
#pragma unroll
                            for (int v = 0; v < 2; ++v) {
                                acc = dot2(ga.v[v], x[s][2 * h + v], acc);
                                acc = dot2(gb.v[v], x[4 + s][2 * h + v], acc);
                            }
                        }
                    }
                    end_b = steps + s < pieces ? qb : end_b;
                }
                if (s == 0) fine_load(t, u);
            }
            // every chain ends where the next one begins, and the unit's first begins at its first bit
            const uint32_t fl = unit * 64u + lane;
            const bool last_lane = lane == 63u || fl + 1u >= t.fine_n;
            // (no short circuits, which are branches; a longer unit's qa stays q0, and not all of its lanes' chains are empty)
            const bool end_good = last_lane ? end_b <= kFineEnd - Tables32::stale : end_b == q_next;
            const bool good = (qa == q_mid) & end_good & ((lane != 0) | (a == 0));
            if (__builtin_expect(__builtin_amdgcn_ballot_w64((fl < t.fine_n) & !good) != 0, 0)) {
                bool walk = !longer && __builtin_amdgcn_ballot_w64(fl < t.fine_n && !good && !last_lane) != 0;
                const uint64_t base = seg_start(t, unit * t.fine_pieces);
                const uint64_t anew = __builtin_amdgcn_ballot_w64(!last_lane && next < a);
                uint32_t from_a = a + (__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(anew >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(anew), 0u)) << 16);
                uint32_t from_b = from_a + ((b - a) & 0xffffu);
                const uint32_t next_a = from_a + ((next - a) & 0xffffu);
#pragma unroll 1
                for (;; walk = true) {
                    if (walk) {
                        const bool one = t.fine_units == 1u;
                        if (t.chunk_symbols < kFineFind || !fine_find<PAIR>(t, sm.tb, col, max_len, unit, base, from_a, from_b))
                            fine_walk<PAIR>(t, sm.tb, col, max_len, unit, one ? kFineWaves : 1u,
                                            one ? (n_quanta - g + kFineWaves - 1u) / kFineWaves : t.fine_units - of_row, from_a, from_b);
                    }
                    uint32_t end_a = from_a, end_b = from_b;
                    acc = fine_again<PAIR>(t, sm.tb, col, max_len, zf, base, end_a, end_b,
                                           [&](uint32_t j) __attribute__((always_inline)) { return activations(here / 8u + j); });
                    const bool good = end_a == from_b && (last_lane || end_b == next_a) && (lane != 0 || from_a == 0);
                    if (walk || __builtin_amdgcn_ballot_w64(fl < t.fine_n && !good) == 0) break;
                }
                // (what a wavefront holds for its next unit is asked for again: kept over all this, some of it is spilled)
#pragma unroll
                for (uint32_t p = 0; p < 8; ++p) x[p] = u32x4{0u, 0u, 0u, 0u};
                x_col = 0xffffffffu;
                fine_ask(t, unit_next, u);
                fine_load(t, u);
            }
            sum += acc;
            if (row_done) {
                fine_sums<F32>(t, it.first + g, unit, sum);
                sum = 0.0f;
            }
            g = g_next;
            of_row = row_done ? 0u : of_row + 1u;
            unit = unit_next;
        }
        i += (n_quanta + item_quanta - 1u) / item_quanta;
    }
}

// ------------------------------------------------------------------ host glue
thread_local std::string g_last_error;

bool hip_ok(hipError_t e, const char *what) {
    if (e == hipSuccess) return true;
    g_last_error = std::string(what) + ": " + hipGetErrorString(e);
    return false;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool dtype_ok(entro_op op, entro_dtype d, int bits) {
    if (op == ENTRO_OP_DECODE) return d == ENTRO_U8 || (d == ENTRO_U4_PACKED && bits == 4);
    return d == ENTRO_F32 || d == ENTRO_BF16;
}

// Re-derive the canonical codes from the lengths and compare: the kernels
// rebuild the code from lengths alone, so the two must agree.
entro_status check_codebook(const entro_codebook *cb) {
    if (!cb) return ENTRO_ERR_NULL;
    if (cb->bits != 4 && cb->bits != 8) return ENTRO_ERR_BITS;
    entro_codebook ref;
    entro_status st = entro_codebook_from_lengths(cb->len, cb->bits, &ref);
    if (st != ENTRO_OK) return st == ENTRO_ERR_SIZE ? ENTRO_ERR_CORRUPT : st;
    for (int s = 0; s < (1 << cb->bits); ++s)
        if (ref.code[s] != cb->code[s]) return ENTRO_ERR_CORRUPT;
    for (int s = (1 << cb->bits); s < ENTRO_MAX_SYMBOLS; ++s)
        if (cb->len[s]) return ENTRO_ERR_CORRUPT;
    if (ref.max_len != cb->max_len) return ENTRO_ERR_CORRUPT;
    return ENTRO_OK;
}

// log2 of the entry points per segment of a tensor (0: none inside the segments)
uint32_t sub_levels(const entro_tensor &t) {
    if (!t.sub_symbols || !t.chunk_symbols || t.chunk_symbols % t.sub_symbols) return 0;
    uint32_t per = t.chunk_symbols / t.sub_symbols, lg = 0;
    while ((1u << lg) < per) ++lg;
    return lg;
}

// Symbols a lane takes of this tensor when pieces are merged `level` times pairwise (at most up to whole segments).
uint64_t lane_symbols_at(const entro_tensor &t, uint32_t level) {
    if (!t.sub_symbols) return t.chunk_symbols;
    return static_cast<uint64_t>(t.sub_symbols) << std::min(level, sub_levels(t));
}

// How coarse the lanes of a launch over these tensors are: as coarse as still gives every lane slot of the
// device (`lane_slots`) a lane -- a lane's work is serial, so small launches are cut as fine as the entry
// points allow, and large ones as coarse as their segments, which costs the least per symbol.
uint32_t choose_level(const entro_tensor *ts, uint32_t count, uint64_t lane_slots) {
    uint32_t top = 0;
    for (uint32_t i = 0; i < count; ++i) top = std::max(top, sub_levels(ts[i]));
    for (uint32_t level = top; level > 0; --level) {
        uint64_t lanes = 0;
        for (uint32_t i = 0; i < count; ++i)
            if (ts[i].chunk_symbols) lanes += (ts[i].n + lane_symbols_at(ts[i], level) - 1) / lane_symbols_at(ts[i], level);
        if (lanes * 8 >= lane_slots * 7) return level;        // (seven eighths of the slots: one unit per wavefront beats two for most)
    }
    return 0;
}

entro_status fill_dev_tensor(const entro_tensor *t, entro_op op, entro_dtype d, uint32_t level, DevTensor *dt) {
    if (!t || !t->stream || !t->offsets || !t->out || !t->cb) return ENTRO_ERR_NULL;
    entro_status st = check_codebook(t->cb);
    if (st != ENTRO_OK) return st;
    const int bits = t->cb->bits;
    if (!dtype_ok(op, d, bits)) return ENTRO_ERR_SCHEME;
    if (t->n == 0 || t->chunk_symbols == 0 || t->chunk_symbols > kMaxChunkSymbols) return ENTRO_ERR_SIZE;
    if (d == ENTRO_U4_PACKED && (t->chunk_symbols & 1u)) return ENTRO_ERR_SIZE;
    // offsets into the stream are 32-bit numbers in the kernels, with room for a line or two past the end
    if (t->stream_bytes < 32 || (t->stream_bytes & 15u) || t->stream_bytes >= (uint64_t{1} << 32) - 65536)
        return ENTRO_ERR_SIZE;
    // the symbols one lane decodes: 2^level pieces, where the tensor has entry points inside its segments
    uint32_t lane_symbols = t->chunk_symbols, sub_shift = 0, sub_merge = 0;
    if (t->sub_symbols) {
        if (!t->sub_bits) return ENTRO_ERR_NULL;
        if (reinterpret_cast<uintptr_t>(t->sub_bits) & 3u) return ENTRO_ERR_ALIGN;
        if (t->chunk_symbols % t->sub_symbols != 0) return ENTRO_ERR_SIZE;
        const uint32_t per = t->chunk_symbols / t->sub_symbols;
        if (per > ENTRO_MAX_SUB_PER_CHUNK || (per & (per - 1u)) != 0) return ENTRO_ERR_SIZE;
        if (d == ENTRO_U4_PACKED && (t->sub_symbols & 1u)) return ENTRO_ERR_SIZE;
        sub_merge = std::min(level, sub_levels(*t));
        sub_shift = sub_levels(*t) - sub_merge;
        lane_symbols = t->sub_symbols << sub_merge;
    }
    const uint64_t n_chunks = entro_num_chunks(t->n, lane_symbols);
    if (n_chunks >= (uint64_t{1} << 32) - 1024) return ENTRO_ERR_SIZE;
    if (!aligned16(t->stream) || !aligned16(t->offsets) || !aligned16(t->out)) return ENTRO_ERR_ALIGN;
    if (op != ENTRO_OP_DECODE && t->qp.bits != bits) return ENTRO_ERR_BITS;
    // the kernels subtract the zero-point in fp32, which must represent it exactly
    if (op != ENTRO_OP_DECODE && (t->qp.zero_point > (1 << 24) || t->qp.zero_point < -(1 << 24))) return ENTRO_ERR_RANGE;
    if (op == ENTRO_OP_GEMV) {
        if (!t->x) return ENTRO_ERR_NULL;
        if (!aligned16(t->x)) return ENTRO_ERR_ALIGN;
        if (t->rows == 0 || t->cols == 0 || static_cast<uint64_t>(t->rows) * t->cols != t->n)
            return ENTRO_ERR_SIZE;
    }
    std::memset(dt, 0, sizeof(*dt));
    dt->stream = static_cast<const uint8_t *>(t->stream);
    dt->offsets = t->offsets;
    dt->out = t->out;
    dt->x = static_cast<const uint16_t *>(t->x);
    dt->n = t->n;
    dt->stream_bytes = static_cast<uint32_t>(t->stream_bytes);
    dt->chunk_symbols = dt->fix_symbols = lane_symbols;
    dt->n_chunks = static_cast<uint32_t>(n_chunks);
    dt->sub = sub_shift ? t->sub_bits : nullptr;
    dt->sub_shift = sub_shift;
    dt->sub_merge = sub_merge;
    dt->rows = t->rows;
    dt->cols = t->cols;
    dt->bits = static_cast<uint32_t>(bits);
    dt->scale = t->qp.scale;
    dt->zero_point = t->qp.zero_point;
    dt->max_len = static_cast<uint32_t>(t->cb->max_len);
    dt->need_fix = (op == ENTRO_OP_GEMV && (lane_symbols % t->cols) != 0) ? 1u : 0u;
    // rows cut into a power of two of lanes (at most a wavefront's 64) that all go through the kernels' block
    // path: the wavefront adds the row up itself
    if (dt->need_fix && t->cols % lane_symbols == 0 && lane_symbols % 128u == 0) {
        const uint32_t per_row = t->cols / lane_symbols;
        if (per_row <= 64u && (per_row & (per_row - 1u)) == 0) {
            dt->row_lanes = per_row;
            dt->need_fix = 0;
        }
    }
    std::memcpy(dt->len, t->cb->len, 256);
    return ENTRO_OK;
}

template <class F>
void dispatch_mode(int mode, F f) {
    switch (mode) {
        case kModeU8: f(std::integral_constant<int, kModeU8>{}); break;
        case kModeU4: f(std::integral_constant<int, kModeU4>{}); break;
        case kModeF32: f(std::integral_constant<int, kModeF32>{}); break;
        case kModeBF16: f(std::integral_constant<int, kModeBF16>{}); break;
        case kModeGemvF32: f(std::integral_constant<int, kModeGemvF32>{}); break;
        case kModeU8P: f(std::integral_constant<int, kModeU8P>{}); break;
        case kModeF32P: f(std::integral_constant<int, kModeF32P>{}); break;
        case kModeBF16P: f(std::integral_constant<int, kModeBF16P>{}); break;
        case kModeGemvF32P: f(std::integral_constant<int, kModeGemvF32P>{}); break;
        case kModeGemvBF16P: f(std::integral_constant<int, kModeGemvBF16P>{}); break;
        case kModeGemvF32W: f(std::integral_constant<int, kModeGemvF32W>{}); break;
        case kModeGemvBF16W: f(std::integral_constant<int, kModeGemvBF16W>{}); break;
        default: f(std::integral_constant<int, kModeGemvBF16>{}); break;
    }
}

// Lanes (= segments) per workgroup of the main kernel of a mode.
unsigned wg_of(int mode) {
    unsigned wg = 64;
    dispatch_mode(mode, [&](auto m) { wg = 64u * Cfg<decltype(m)::value>::waves; });
    return wg;
}

// Symbols per block of a mode's kernel: lanes must be whole blocks to go through its fast path.
unsigned spb_of(int mode) {
    unsigned spb = 64;
    dispatch_mode(mode, [&](auto m) { spb = Cfg<decltype(m)::value>::spb; });
    return spb;
}

// Does the GEMV of this tensor fit the wide tables?
bool wide_ok(const DevTensor &dt) { return dt.bits == 8 && dt.zero_point >= -1 && dt.zero_point <= 256; }

// `pairs`: every tensor of the launch holds 4-bit symbols, so the tables can hold two codes per entry.
// `wide`: a GEMV all of whose tensors hold 8-bit symbols with a zero-point in [-1, 256] (symbol - zero_point is a
// bf16 then, which the wide tables hold ready for use).
int mode_of(entro_op op, entro_dtype d, bool pairs, bool wide = false) {
    if (op == ENTRO_OP_GEMV) {
        if (pairs) return d == ENTRO_F32 ? kModeGemvF32P : kModeGemvBF16P;
        if (wide) return d == ENTRO_F32 ? kModeGemvF32W : kModeGemvBF16W;
        return d == ENTRO_F32 ? kModeGemvF32 : kModeGemvBF16;
    }
    switch (d) {
        case ENTRO_U8: return pairs ? kModeU8P : kModeU8;
        case ENTRO_U4_PACKED: return kModeU4;
        case ENTRO_F32: return pairs ? kModeF32P : kModeF32;
        default: return pairs ? kModeBF16P : kModeBF16;
    }
}


// Workgroups of the batched kernel of `mode` that the current device holds at once
// (its LDS footprint decides); 0 if the device cannot be asked.
unsigned resident_workgroups(int mode) {
    thread_local int cached_dev = -1, cached_cus = 0;
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev), "hipGetDevice")) return 0;
    if (dev != cached_dev) {
        int n = 0;
        if (!hip_ok(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev), "hipDeviceGetAttribute")) return 0;
        cached_dev = dev;
        cached_cus = n;
    }
    const int cus = cached_cus;
    size_t smem = 1;
    dispatch_mode(mode, [&](auto m) { smem = sizeof(SmemFor<decltype(m)::value>); });
    const unsigned per_cu = static_cast<unsigned>((160u * 1024u) / smem);
    return static_cast<unsigned>(cus) * (per_cu ? per_cu : 1u);
}

// Does decoding from a wrong bit fall into step soon?  Not where (nearly) all codes have one length, or lengths with
// a common divisor.  Judged by the spread of the lengths as the code itself weighs them (a code of l bits: 2^-l): at
// least half a squared bit.  Weights have one or two, symbols spread evenly over the grid about a tenth.
bool falls_into_step(const entro_codebook *cb) {
    uint32_t symbols[ENTRO_MAX_CODE_LEN + 1] = {}, divisor = 0;
    for (int s = 0; s < ENTRO_MAX_SYMBOLS; ++s) ++symbols[cb->len[s]];
    double weight = 0, mean = 0, square = 0;
    for (uint32_t l = 1; l <= ENTRO_MAX_CODE_LEN; ++l) {
        if (!symbols[l]) continue;
        const double p = std::ldexp(static_cast<double>(symbols[l]), -static_cast<int>(l));
        weight += p;
        mean += p * l;
        square += p * l * l;
        divisor = std::gcd(divisor, l);
    }
    mean /= weight;
    return divisor == 1 && square / weight - mean * mean >= 0.5;
}

// Is this a code of nearly one length (ring_trip_flat)?  Symbols spread evenly over the grid have one, norm gains for instance.
bool flat_code(const entro_codebook *cb, DevTensor *dt) {
    uint32_t symbols[ENTRO_MAX_CODE_LEN + 1] = {}, least = ENTRO_MAX_CODE_LEN;
    for (int s = 0; s < ENTRO_MAX_SYMBOLS; ++s) {
        ++symbols[cb->len[s]];
        if (cb->len[s]) least = std::min<uint32_t>(least, cb->len[s]);
    }
    if (least == 0 || cb->max_len > kL1 || static_cast<uint32_t>(cb->max_len) > least + 3u) return false;
    uint64_t space = 0;                                      // taken by the codes of up to l bits, in units of 2^-32
    for (uint32_t l = least; l < least + 4u; ++l) {
        if (l <= ENTRO_MAX_CODE_LEN) space += static_cast<uint64_t>(symbols[l]) << (ENTRO_MAX_CODE_LEN - l);
        if (l < least + 3u) dt->flat_last[l - least] = static_cast<uint32_t>(space - 1u);
    }
    dt->flat_len = least;
    return space == uint64_t{1} << 32;
}

// Segments without entry points that leave most lanes of the device without work: 2^sub_shift lanes per segment that find their
// pieces' starts themselves (find_start), as many as the device has lanes for.  For segments longer than k_shared holds
// (kShareMost), and for those of more than half of that where it is the faster of the two (launch_single).
// A lane then decodes its share three times, two of them symbol by symbol, which pays from eight lanes per segment on (4-bit
// symbols, decoded two a lookup but searched one at a time: sixteen).  The pieces must be whole blocks of the kernel.
// Measured when shorter segments came here too: 4096 x 4096 in segments of 4096 to bf16 318 us with a lane per segment, 47 us
// with 64; 8192 x 4096 in segments of 1024, which got eight, 115 -> 98 us.
bool cut_segments(entro_op op, int mode, uint64_t lane_slots, const entro_tensor *t, DevTensor *dt) {
    if (op == ENTRO_OP_GEMV || t->sub_symbols) return false;
    const uint32_t block = spb_of(mode);
    const uint32_t least = dt->bits == 4 ? 4u : 3u;
    for (uint32_t sh = 6; sh >= least; --sh) {
        if ((static_cast<uint64_t>(dt->n_chunks) << sh) > lane_slots || dt->chunk_symbols % (block << sh) != 0) continue;
        if (!falls_into_step(t->cb)) return false;               // (asked last: a pass over the code's lengths)
        dt->chunk_symbols >>= sh;
        dt->sub_shift = sh;
        dt->n_chunks = static_cast<uint32_t>(entro_num_chunks(dt->n, dt->chunk_symbols));
        return true;
    }
    return false;
}

// Stream bits of a symbol on average (as far as the rules below use them: at most the symbol's own).
double stream_bits(uint32_t bits, uint64_t stream_bytes, uint64_t n) {
    return std::min(static_cast<double>(bits), 8.0 * static_cast<double>(stream_bytes) / static_cast<double>(n));
}
double stream_bits(const DevTensor &dt) { return stream_bits(dt.bits, dt.stream_bytes, dt.n); }

// A tensor in few segments, or few pieces between entry points: 4 to 64 lanes share one (k_shared), at about 64 symbols a
// lane.  A wavefront's share of LDS is what its unit's symbols take, and its part of the stream at the tensor's mean rate and
// a thirty-second more (a unit with more is read straight from memory).
// share_fits: whether the tensor's form goes there at all; describes its units and says how much LDS one takes.
// Pieces of 256 symbols come here up to 4 bits a symbol (2048 x 4096: 33.7 -> 28.4 us and 26.7 -> 21.8, but the more bits a symbol
// takes, the fewer a lookup answers: at 5.0 bits 35.6 -> 36.1, and the product 34.2 -> 36.1).  Pieces of 128 do not: 20.9
// against 26.2 (256 x 4096).
bool share_fits(entro_op op, const entro_tensor *t, DevTensor *dt, uint32_t *wave_bytes) {
    const uint32_t S = dt->chunk_symbols;
    if (dt->sub_merge != 0 || S % 128u != 0 || S < (t->sub_symbols ? 4u : 8u) * kShareSymbols || S > kShareMost) return false;
    if (op == ENTRO_OP_GEMV && dt->cols % 8u != 0) return false;
    const double rate = stream_bits(*dt);
    if (t->sub_symbols && S < 8u * kShareSymbols && rate > 4.0) return false;
    if (!falls_into_step(t->cb)) return false;
    uint32_t sh = 1;
    while (sh < 6u && (kShareSymbols << (sh + 1u)) <= S) ++sh;
    uint32_t per = 64u >> sh;
    // units of whole rows need no second stage: up to a quarter of the lanes is left idle for it
    for (uint32_t p = per; op == ENTRO_OP_GEMV && 4u * p >= 3u * (64u >> sh); --p)
        if (S * p % dt->cols == 0) {
            per = p;
            break;
        }
    dt->share_shift = sh;
    dt->share_per = per;
    dt->share_units = (dt->n_chunks + per - 1u) / per;
    dt->fix_symbols = S * per;
    dt->row_lanes = 0;
    dt->need_fix = (op == ENTRO_OP_GEMV && dt->fix_symbols % dt->cols != 0) ? 1u : 0u;
    const uint32_t copy = static_cast<uint32_t>(S * per * rate / 8.0 * 33.0 / 32.0) + 16u;
    *wave_bytes = share_symbol_bytes(S * per) + (copy + 15u) / 16u * 16u + 32u;
    return true;
}

uint32_t share_waves(uint32_t wave_bytes) { return std::min<uint32_t>(kShareWaves, sizeof(ShareMem::pool) / wave_bytes); }

// Whether sharing pays is decided by what the launches take, in microseconds, as measured on 3000 calls of 3.3 to 7.5 (8 bits)
// and 1.5 to 3.6 (4 bits) bits a symbol, segments and pieces of 256 to 8192 symbols, 512 to 49152 of them; the estimates are
// within 10 to 20 % of the times, beside what the launches have in common.
// A lane per segment: a lane's serial chain, whatever their number while wavefronts have their SIMDs to themselves; that is up to
// three sixteenths of the lanes, and launches of more segments are not shared.  A product takes a shorter last segment symbol by
// symbol behind that (4096 segments of 4096 in rows of 11008: 864 us, 298 without one).
// Shared: rounds of units, one a wavefront.  A round's time goes with the bits (more of them, fewer codes a lookup; 4-bit symbols
// leave a lookup's four codes as the limit), with the symbols of a unit, and less than in proportion with the wavefronts.
// Searched (find_start): every piece is decoded three times, slower the more bits a symbol has; up to 4096 symbols a segment the
// search gives up on dense codes and has cost a lane per segment then (4096 x 4096 at 7.5 bits to bf16 296 us, 86 shared).
// Measured, a lane per segment -> shared, at the places where the choice turns.  Prepared products of 8 bits: 40960 segments of
// 512 symbols at 3.5 bits 48 -> 42 us, at 5.4 54.7 -> 57.1, at 7.5 46 -> 80; of 4096 at 5.2 338 -> 363; 28672 of 4096 at 6.5
// 396 -> 292, at 7.5 314 -> 346.  Of 4 bits: 40960 of 1024 44.3 -> 53.5, 28672 43.1 -> 37.8.  Single calls to bytes: 28672 of
// 8192 at 3.3 bits searched 631, shared 295.
bool few_segments(uint64_t segments, uint64_t lane_slots) { return segments * 16u <= lane_slots * 3u; }

double lane_us(entro_op op, entro_dtype d, uint32_t bits, const DevTensor &dt) {
    const double each = op == ENTRO_OP_GEMV ? (bits == 4 ? 0.038 : 0.072) : d == ENTRO_F32 ? (bits == 4 ? 0.045 : 0.098)
                        : d == ENTRO_BF16   ? (bits == 4 ? 0.039 : 0.080) : (bits == 4 ? 0.034 : 0.080);
    return 2.0 + each * dt.chunk_symbols + (op == ENTRO_OP_GEMV ? 0.18 * (dt.n % dt.chunk_symbols) : 0.0);
}

// `units`: of the workgroup that has most of them.
double share_us(entro_op op, entro_dtype d, const DevTensor &dt, uint32_t units, uint32_t waves) {
    const double out = op == ENTRO_OP_GEMV ? 4.0 : d == ENTRO_F32 ? 1.5 : 0.0;
    const double full = (dt.bits == 4 ? 12.0 : 4.9 * stream_bits(dt)) + out;      // 16 wavefronts, 4096 symbols each
    const double by_size = full * dt.chunk_symbols * dt.share_per / 4096.0;
    const uint32_t rounds = units / waves, last = units % waves;
    return by_size / 30.0 * (rounds * (14.0 + waves) + (last ? 14.0 + last : 0.0));
}

double find_us(const DevTensor &dt, double rate) { return 3.0 * dt.chunk_symbols * (0.04 + 0.04 * rate); }

// A prepared launch gives workgroup b of G the items [b * n / G, (b + 1) * n / G): the longest time that `cost` makes of a
// workgroup's stretches (items of one tensor side by side), with the time to load a stretch's tables.
template <class Items, class Cost>
double busiest_us(uint32_t count, uint32_t slots, Items items, Cost cost) {
    uint64_t n = 0;
    for (uint32_t i = 0; i < count; ++i) n += items(i);
    const uint64_t groups = std::min<uint64_t>(n, slots);
    double most = 0;
    uint64_t left = items(0), carried = 0;
    uint32_t i = 0;
    for (uint64_t b = 0; b < groups; ++b) {
        carried += n % groups;
        uint64_t share = n / groups + (carried >= groups ? 1u : 0u);
        carried -= carried >= groups ? groups : 0u;
        double us = 0;
        while (share != 0) {
            const uint64_t here = std::min(share, left);
            us += cost(i, here) + 3.0;
            share -= here;
            left -= here;
            if (left == 0 && i + 1u < count) left = items(++i);
        }
        most = std::max(most, us);
    }
    return most;
}

uint64_t items_of(uint64_t units, uint64_t per_item) { return (units + per_item - 1u) / per_item; }

// Units of a work item where a lane takes a segment (or piece): what a workgroup takes in one round when the launch is large, and
// less when the launch would not give every compute unit an item otherwise.
uint32_t lane_item_units(uint64_t units, uint32_t slots, uint32_t waves) {
    return static_cast<uint32_t>(std::min<uint64_t>(waves, std::max<uint64_t>(1, units / slots)));
}

entro_status launch_fix_single(entro_dtype d, const DevTensor &dt, hipStream_t s) {
    const unsigned grid = (dt.rows + kFixRows - 1) / kFixRows;
    if (d == ENTRO_F32) hipLaunchKernelGGL(k_fix_single<kModeGemvF32>, dim3(grid), dim3(kFixWG), 0, s, dt);
    else hipLaunchKernelGGL(k_fix_single<kModeGemvBF16>, dim3(grid), dim3(kFixWG), 0, s, dt);
    return hip_ok(hipGetLastError(), "launch row-sum kernel") ? ENTRO_OK : ENTRO_ERR_DEVICE;
}

// Wavefronts of a workgroup that take units in a launch over one tensor.
uint32_t share_launch_waves(const DevTensor &dt, uint32_t wave_bytes, unsigned cus) {
    return std::min<uint32_t>(share_waves(wave_bytes), (dt.share_units + cus - 1u) / cus);
}

entro_status launch_shared(entro_op op, entro_dtype d, const DevTensor &dt, uint32_t wave_bytes, unsigned cus, hipStream_t s) {
    const unsigned waves = share_launch_waves(dt, wave_bytes, cus);
    const unsigned grid = std::min<unsigned>(cus, (dt.share_units + waves - 1u) / waves);
    dispatch_mode(mode_of(op, d, false), [&](auto m) {
        constexpr int M = decltype(m)::value;
        if constexpr (M <= kModeGemvBF16)
            hipLaunchKernelGGL(k_shared<M>, dim3(grid), dim3(64u * kShareWaves), 0, s, dt, static_cast<uint32_t>(waves), wave_bytes);
    });
    if (!hip_ok(hipGetLastError(), "launch decode kernel")) return ENTRO_ERR_DEVICE;
    return dt.need_fix ? launch_fix_single(d, dt, s) : ENTRO_OK;
}

entro_status launch_single(const entro_tensor *t, entro_op op, entro_dtype d, float *partials,
                           void *hip_stream) {
    // all argument checks first, on the host alone; then the device is asked how many lanes it holds, which
    // decides how fine the lanes are cut
    DevTensor dt;
    entro_status st = fill_dev_tensor(t, op, d, 0, &dt);
    if (st != ENTRO_OK) return st;
    const int mode = mode_of(op, d, dt.bits == 4, wide_ok(dt));
    const unsigned wg = wg_of(mode);
    const unsigned slots = resident_workgroups(mode);
    if (slots == 0) return ENTRO_ERR_DEVICE;
    st = fill_dev_tensor(t, op, d, choose_level(t, 1, static_cast<uint64_t>(slots) * wg), &dt);
    if (st != ENTRO_OK) return st;
    dt.partials = partials;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const uint64_t lane_slots = static_cast<uint64_t>(slots) * wg;
    // a unit per wavefront when the tensor is large; fewer units per workgroup, down to one, when
    // that would leave compute units without a workgroup
    unsigned wg_units = 1, grid = 1;
    auto cut_units = [&](const DevTensor &of) {
        const unsigned units = (of.n_chunks + kUnit - 1) / kUnit;
        wg_units = std::min(wg / 64u, std::max(1u, units / slots));
        grid = (units + wg_units - 1) / wg_units;
        return (grid + slots - 1u) / slots;                      // rounds of workgroups
    };
    bool find = false;
    DevTensor shared = dt;
    uint32_t wave_bytes = 0;
    if (few_segments(dt.n_chunks, lane_slots) && share_fits(op, t, &shared, &wave_bytes)) {
        const uint32_t waves = share_launch_waves(shared, wave_bytes, slots);
        const uint32_t rounds = (shared.share_units + slots * waves - 1u) / (slots * waves);
        const double share = share_us(op, d, shared, rounds * waves, waves);
        const double lane = lane_us(op, d, dt.bits, dt) * cut_units(dt);
        DevTensor found = dt;
        if (dt.bits == 8 && dt.chunk_symbols > kShareMost / 2u && cut_segments(op, mode, lane_slots, t, &found)) {
            const double search = find_us(found, stream_bits(dt)) * cut_units(found);
            find = search < share && search < lane;
        }
        if (!find && share <= lane) return launch_shared(op, d, shared, wave_bytes, slots, s);
        if (find) dt = found;
    } else {
        find = cut_segments(op, mode, lane_slots, t, &dt);
    }
    cut_units(dt);
    dispatch_mode(mode, [&](auto m) {
        constexpr int M = decltype(m)::value;
        if constexpr (!is_gemv(M)) {
            if (find) {
                hipLaunchKernelGGL((k_single<M, true, false>), dim3(grid), dim3(wg), 0, s, dt, static_cast<uint32_t>(wg_units));
                return;
            }
        }
        if constexpr (short_ring(M)) {
            // Up to a wavefront for each compute unit, which waits for its own chain alone.  Lookups in the chain -> none, pieces of 256
            // to fp32, us a call: 1 wavefront 26.0 -> 25.5, 64 27.0 -> 26.3, 256 28.4 -> 27.7; 512 30.0 -> 30.3 (to bf16 27.1 -> 28.1).
            if ((dt.n_chunks + kUnit - 1u) / kUnit <= slots && flat_code(t->cb, &dt)) {
                hipLaunchKernelGGL((k_single<M, false, true>), dim3(grid), dim3(wg), 0, s, dt, static_cast<uint32_t>(wg_units));
                return;
            }
        }
        hipLaunchKernelGGL((k_single<M, false, false>), dim3(grid), dim3(wg), 0, s, dt, static_cast<uint32_t>(wg_units));
    });
    if (!hip_ok(hipGetLastError(), "launch decode kernel")) return ENTRO_ERR_DEVICE;
    return dt.need_fix ? launch_fix_single(d, dt, s) : ENTRO_OK;
}

// Device address of `scratch` on the current device, looked up once per device; nullptr if the
// lookup fails (the error text is kept for entro_last_device_error).
float *static_scratch() {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static float *ptrs[kMaxDevices] = {};
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev), "hipGetDevice")) return nullptr;
    if (dev < 0 || dev >= kMaxDevices) {
        g_last_error = "device index beyond the static scratch table";
        return nullptr;
    }
    std::lock_guard<std::mutex> guard(mu);
    if (!ptrs[dev]) {
        void *p = nullptr;
        if (!hip_ok(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)")) return nullptr;
        ptrs[dev] = static_cast<float *>(p);
    }
    return ptrs[dev];
}

uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

// Symbols one lane decodes of this tensor (what the work list and the partial sums are counted in).
uint32_t lane_symbols_of(const entro_tensor &t) { return t.sub_symbols ? t.sub_symbols : t.chunk_symbols; }

// How k_fine cuts a tensor, by its shape alone (the workspace is laid out from it): lanes of `len` symbols (0: not at all), a
// unit of 64 of them in whole pieces, every lane inside one row.  Shapes whose units hold whole rows, or whose rows are whole
// units, need no second stage and come first; up to 64 symbols, the longest lane that gives one of those.
struct FineShape {
    uint32_t len, rows;
};
FineShape fine_shape(const entro_tensor &t) {
    const uint32_t P = lane_symbols_of(t);
    if (P == 0 || P % 64u != 0 || t.cols == 0 || t.cols > (1u << 30) || t.cols % 8u != 0 || static_cast<uint64_t>(t.rows) * t.cols != t.n) return {0, 0};
    for (uint32_t len = 64; len >= 32; len -= 8) {
        if (64u * len % P != 0 || t.cols % len != 0) continue;
        const uint32_t row_lanes = t.cols / len;
        if (row_lanes <= 64u && (row_lanes & (row_lanes - 1u)) == 0) return {len, kFineRow};
        if (row_lanes % 64u == 0 && row_lanes <= 64u * 16u) return {len, kFineUnits};
    }
    for (uint32_t len = 64; len >= 32; len -= 16)
        if (64u * len % P == 0 && t.cols % len == 0) return {len, kFineParts};
    return {0, 0};
}

// Does this product go to k_fine?  Its lanes have to hold the stream of their symbols (at the tensor's mean rate and 80 bits more,
// where rows are alike six standard deviations of a lane's bits; lanes that do not take longer), its tables the symbols' values:
// integers of at most 256 in magnitude, or 16 for 4-bit symbols.
// (Asked before the tensor has been looked at, by the calls that only say how much room a launch takes.)
bool fine_fits(const entro_tensor &t) {
    const FineShape f = fine_shape(t);
    if (f.len == 0 || t.n / f.len >= (uint64_t{1} << 31) || check_codebook(t.cb) != ENTRO_OK) return false;
    const bool four = t.cb->bits == 4;
    if (t.qp.zero_point < -1 || t.qp.zero_point > (four ? 16 : 256)) return false;
    if (four && t.cb->max_len > 28) return false;            // (fine_again: eight codes and a dword's end in half a column)
    return stream_bits(static_cast<uint32_t>(t.cb->bits), t.stream_bytes, t.n) * f.len + 31.0 + 80.0 <= 32.0 * kFineData;
}

// Does a prepared launch go there: every tensor's form allows it, and all have the same alphabet?
bool fine_launch(const entro_tensor *ts, uint32_t count, entro_op op) {
    if (op != ENTRO_OP_GEMV) return false;
    for (uint32_t i = 0; i < count; ++i)
        if (!fine_fits(ts[i]) || ts[i].cb->bits != ts[0].cb->bits) return false;
    return true;
}

// Describes a tensor (already described with a lane per piece) to k_fine.
void fine_describe(const entro_tensor &t, uint32_t *index, DevTensor *dt) {
    const FineShape f = fine_shape(t);
    const uint32_t row_lanes = t.cols / f.len;
    dt->fine_index = index;
    dt->fine_len = f.len;
    dt->fine_first = (f.len + 15u) / 16u * 8u;
    dt->fine_n = static_cast<uint32_t>(t.n / f.len);
    dt->fine_pieces = 64u * f.len / dt->chunk_symbols;
    dt->fine_rows = f.rows;
    dt->fine_units = f.rows == kFineUnits ? row_lanes / 64u : 1u;
    dt->fine_quanta = f.rows == kFineUnits ? t.rows : (dt->fine_n + 63u) / 64u;
    dt->row_lanes = row_lanes;
    dt->fix_symbols = 64u * f.len;
    dt->need_fix = f.rows == kFineParts && dt->fix_symbols % t.cols != 0 ? 1u : 0u;
}

struct Layout {
    uint64_t off_tensors, off_items, off_fix, off_partials, off_tables, off_index, total;
    uint32_t n_items, n_fix;
};
// room for one tensor's lookup tables in the workspace (the larger kind, whichever the launch uses)
constexpr uint64_t kTablesStride = (sizeof(Tables32) + 255) / 256 * 256;

constexpr uint64_t kFineItems = 16384;

// Workspace layout shared by entro_workspace_bytes and entro_plan_init.  `fine`: of a launch that goes to k_fine (fine_launch).
bool plan_layout(const entro_tensor *ts, uint32_t count, entro_op op, bool fine, Layout *L) {
    uint64_t items = 0, fix = 0, partial_floats = 0, fine_items = 0, index_bytes = 0;
    for (uint32_t i = 0; i < count; ++i) {
        if (ts[i].chunk_symbols == 0 || ts[i].n == 0) return false;
        const uint64_t nc = entro_num_chunks(ts[i].n, lane_symbols_of(ts[i]));
        items += (nc + kUnit - 1) / kUnit;
        if (op == ENTRO_OP_GEMV && ts[i].cols && (lane_symbols_of(ts[i]) % ts[i].cols) != 0) {
            fix += (static_cast<uint64_t>(ts[i].rows) + kFixRows - 1) / kFixRows;
            partial_floats += 2 * nc;
        }
        if (fine) {
            index_bytes += align_up(sizeof(uint32_t) * (ts[i].n / fine_shape(ts[i]).len), 256);
            fine_items += ts[i].n / 2048u + 1u;              // (units have 2048 symbols at least)
        }
    }
    // (k_fine's items are units or rows at least, and larger where this many do not hold a launch)
    items = std::max(items, std::min<uint64_t>(fine_items, kFineItems + count));
    if (items >= (uint64_t{1} << 31) || fix >= (uint64_t{1} << 31)) return false;
    L->n_items = static_cast<uint32_t>(items);
    L->n_fix = static_cast<uint32_t>(fix);
    L->off_tensors = 0;
    L->off_items = align_up(sizeof(DevTensor) * 2 * static_cast<uint64_t>(count), 256);   // a tensor may be described at two lane sizes
    L->off_fix = L->off_items + align_up(sizeof(WorkItem) * items, 256);
    L->off_partials = L->off_fix + align_up(sizeof(WorkItem) * fix, 256);
    L->off_tables = L->off_partials + align_up(sizeof(float) * partial_floats, 256);
    L->off_index = L->off_tables + kTablesStride * count;
    L->total = L->off_index + index_bytes;
    return true;
}

}  // namespace

// for the library's other device source: record a failed HIP call for entro_last_device_error
void entro_detail_note_hip_error(const char *what, int hip_error) {
    hip_ok(static_cast<hipError_t>(hip_error), what);
}

extern "C" {

const char *entro_last_device_error(void) { return g_last_error.c_str(); }

entro_status entro_decode(const entro_tensor *t, entro_dtype out_type, void *hip_stream) {
    return launch_single(t, ENTRO_OP_DECODE, out_type, nullptr, hip_stream);
}

entro_status entro_decode_dequant(const entro_tensor *t, entro_dtype out_type, void *hip_stream) {
    return launch_single(t, ENTRO_OP_DEQUANT, out_type, nullptr, hip_stream);
}

uint64_t entro_gemv_workspace_bytes(const entro_tensor *t) {
    if (!t || t->chunk_symbols == 0 || t->cols == 0) return 0;
    if ((lane_symbols_of(*t) % t->cols) == 0) return 0;
    return align_up(2 * sizeof(float) * entro_num_chunks(t->n, lane_symbols_of(*t)), 256);
}

entro_status entro_decode_gemv(const entro_tensor *t, entro_dtype y_type, void *workspace,
                               uint64_t workspace_bytes, void *hip_stream) {
    if (!t) return ENTRO_ERR_NULL;
    const uint64_t need = entro_gemv_workspace_bytes(t);
    if (need) {
        if (!workspace) return ENTRO_ERR_NULL;
        if (workspace_bytes < need) return ENTRO_ERR_CAPACITY;
        if (!aligned16(workspace)) return ENTRO_ERR_ALIGN;
    }
    return launch_single(t, ENTRO_OP_GEMV, y_type, static_cast<float *>(workspace), hip_stream);
}

entro_status entro_decode_gemv_static(const entro_tensor *t, entro_dtype y_type, void *hip_stream) {
    if (!t) return ENTRO_ERR_NULL;
    float *partials = nullptr;
    if (entro_gemv_workspace_bytes(t)) {
        if (entro_num_chunks(t->n, lane_symbols_of(*t)) > ENTRO_STATIC_GEMV_MAX_SEGMENTS) return ENTRO_ERR_CAPACITY;
        partials = static_scratch();
        if (!partials) return ENTRO_ERR_DEVICE;
    }
    return launch_single(t, ENTRO_OP_GEMV, y_type, partials, hip_stream);
}

uint64_t entro_workspace_bytes(const entro_tensor *ts, uint32_t count, entro_op op) {
    Layout L;
    if (!ts || count == 0 || !plan_layout(ts, count, op, fine_launch(ts, count, op), &L)) return 0;
    return L.total;
}

// Validate, lay the table out in `host` (L.off_partials bytes) and fill in the plan; nothing touches the device.
// `fine`: the launch goes to k_fine.
static entro_status build_plan(entro_plan *plan, const entro_tensor *ts, uint32_t count, entro_op op, entro_dtype out_type,
                               void *workspace, uint64_t workspace_bytes, const Layout &L, unsigned char *host, bool fine) {
    std::memset(host, 0, L.off_partials);
    DevTensor *dts = reinterpret_cast<DevTensor *>(host + L.off_tensors);
    WorkItem *items = reinterpret_cast<WorkItem *>(host + L.off_items);
    WorkItem *fix = reinterpret_cast<WorkItem *>(host + L.off_fix);
    uint64_t n_items = 0, n_fix = 0, partial_floats = 0, total_units = 0;
    bool pairs = true;                                       // every tensor 4-bit: two codes per table entry
    bool multirow = false;                                   // GEMV: a tensor's segments are longer than its rows
    float *partials_base = reinterpret_cast<float *>(static_cast<unsigned char *>(workspace) + L.off_partials);
    // how fine the lanes are cut is decided for the launch as a whole (all its tensors are 4-bit, or the
    // tables take single codes: the kernel and with it the lane slots are known before the tensors are looked at)
    // (all argument checks come first, on the host alone)
    bool all4 = true, wide = true;
    for (uint32_t i = 0; i < count; ++i) {
        entro_status st = fill_dev_tensor(&ts[i], op, out_type, 0, &dts[i]);
        if (st != ENTRO_OK) return st;
        all4 = all4 && dts[i].bits == 4;
        wide = wide && wide_ok(dts[i]);
    }
    const int mode0 = mode_of(op, out_type, all4, wide);
    const unsigned slots0 = resident_workgroups(mode0);
    if (slots0 == 0) return ENTRO_ERR_DEVICE;
    const uint64_t lane_slots = static_cast<uint64_t>(slots0) * wg_of(mode0);
    // Launches whose segments or pieces are so few that lanes share them (k_shared_batch), by the rule of the single calls.
    // Measured, prepared launches, before -> now.  2048 x 2048 matrices, 8 bits, pieces of 512: one to bf16 47.6 -> 22.7 us, its
    // product 46.8 -> 23.9; five 90.2 -> 48.8, 85.0 -> 47.8.  Pieces of 1024: 86.2 -> 26.4, 82.4 -> 27.7.  4 bits, pieces of 512:
    // 27.8 -> 15.2, five 53.1 -> 32.3.
    // Without entry points, 4096 x 4096 in segments of 4096: 8 bits to bf16 319 -> 86 us, to bytes 303 -> 80, 4 bits to nibbles
    // 135 -> 55.  4-bit products whose rows a wavefront adds up itself, pieces of 512: 2048 x 4096 25.3 -> 15.7 us; of 256 they
    // are not shared: 4096 x 1024 at 1.5 bits a symbol 15.3 us, and 17.0 shared, at 3.6 bits 14.9 and 17.3.
    uint64_t segments = 0;
    for (uint32_t i = 0; i < count; ++i) segments += dts[i].n_chunks;
    bool shared = few_segments(segments, lane_slots);
    uint32_t wave_bytes = 1;
    for (uint32_t i = 0; shared && i < count; ++i) {
        uint32_t bytes = 0;
        shared = !(op == ENTRO_OP_GEMV && dts[i].bits == 4 && dts[i].row_lanes && dts[i].chunk_symbols < 512u) && share_fits(op, &ts[i], &dts[i], &bytes);
        wave_bytes = std::max(wave_bytes, bytes);
    }
    if (shared) {
        // what the busiest workgroup takes: its stretches, one after the other, with the tables of each
        const uint32_t take = share_waves(wave_bytes), have = static_cast<uint32_t>(wg_of(mode0) / 64u);
        uint64_t units = 0;
        for (uint32_t i = 0; i < count; ++i) units += (dts[i].n_chunks + kUnit - 1u) / kUnit;
        const uint32_t item_units = lane_item_units(units, slots0, have);
        const double share = busiest_us(count, slots0, [&](uint32_t i) { return items_of(dts[i].share_units, share_item_units(dts[i].share_per)); },
                                        [&](uint32_t i, uint64_t items) {
                                            const uint64_t n = std::min<uint64_t>(dts[i].share_units, items * share_item_units(dts[i].share_per));
                                            return share_us(op, out_type, dts[i], static_cast<uint32_t>(n), take);
                                        });
        const double lane = busiest_us(count, slots0, [&](uint32_t i) { return items_of((dts[i].n_chunks + kUnit - 1u) / kUnit, item_units); },
                                       [&](uint32_t i, uint64_t items) {
                                           return lane_us(op, out_type, all4 ? 4u : 8u, dts[i]) * ((items * item_units + have - 1u) / have);
                                       });
        shared = share <= lane;
    }
    // (products that go to k_fine do so whether their pieces are few or not)
    shared = shared && !fine;
    uint64_t index_at = L.off_index;
    const uint32_t level = shared || fine ? 0u : choose_level(ts, count, lane_slots);
    for (uint32_t i = 0; i < count; ++i) {
        entro_status st = fill_dev_tensor(&ts[i], op, out_type, level, &dts[i]);
        if (st != ENTRO_OK) return st;
        uint32_t bytes;
        if (shared) share_fits(op, &ts[i], &dts[i], &bytes);
        if (fine) {
            fine_describe(ts[i], reinterpret_cast<uint32_t *>(static_cast<unsigned char *>(workspace) + index_at), &dts[i]);
            index_at += align_up(sizeof(uint32_t) * static_cast<uint64_t>(dts[i].fine_n), 256);
        }
        dts[i].tables = static_cast<unsigned char *>(workspace) + L.off_tables + kTablesStride * i;
        total_units += (dts[i].n_chunks + kUnit - 1) / kUnit;
        pairs = pairs && dts[i].bits == 4;
        multirow = multirow || (op == ENTRO_OP_GEMV && dts[i].cols < dts[i].chunk_symbols);
        if (dts[i].need_fix) {
            dts[i].partials = partials_base + partial_floats;
            partial_floats += 2 * static_cast<uint64_t>(shared ? dts[i].share_units : fine ? dts[i].fine_quanta : dts[i].n_chunks);
            for (uint32_t r = 0; r < dts[i].rows; r += kFixRows) fix[n_fix++] = WorkItem{i, r};
        }
    }
    // A work item is what a workgroup takes in one round when the launch is large (a unit per
    // wavefront: stretches of whole items end for all wavefronts together), and less when the launch
    // would not give every compute unit an item otherwise.
    const int mode = mode0;
    const unsigned slots = slots0;
    const uint64_t waves = wg_of(mode) / 64u;
    uint32_t item_units = lane_item_units(total_units, slots, static_cast<uint32_t>(waves));
    // Tensors with entry points inside their segments are described a second time, with lanes up to
    // 2^kTailShift times finer (as fine as still tiles into the kernel's blocks): the kernel draws what
    // is left over behind the last whole round of a stretch from that description.  (Not for the GEMV: its partial sums are laid out per lane.)
    uint32_t n_desc = count;
    const uint32_t block = spb_of(mode);
    for (uint32_t i = 0; i < count && op != ENTRO_OP_GEMV && !shared; ++i) {
        uint32_t finer = std::min<uint32_t>(dts[i].sub_merge, kTailShift);
        while (finer > 0 && ((dts[i].chunk_symbols >> finer) % block) != 0) --finer;
        if (finer == 0 || dts[i].chunk_symbols % block != 0) continue;
        entro_status st = fill_dev_tensor(&ts[i], op, out_type, dts[i].sub_merge - finer, &dts[n_desc]);
        if (st != ENTRO_OK) return st;
        dts[n_desc].tables = dts[i].tables;
        dts[i].fine = n_desc++;
        dts[i].fine_shift = finer;
    }
    // where every tensor has that second description a stretch may end anywhere at little cost: the
    // workgroups' shares are made equal to within one unit
    if (n_desc == 2 * count) item_units = 1;
    if (fine) {
        // Where every tensor is worth eight workgroups or more, each gets workgroups of its own, an item each: a workgroup whose share
        // goes from one tensor to the next loads tables twice and comes in last (6144 rows of 4096 in three tensors, 25 M symbols:
        // 23 -> 21 us).  Otherwise about sixteen items of as many symbols for every workgroup (not of as many rows: 224 products
        // of rows of 4096 and 14336 in one launch took 195 us a layer).
        uint64_t all = 0, least = UINT64_MAX, used = 0;
        for (uint32_t i = 0; i < count; ++i) {
            all += dts[i].fine_n;
            least = std::min<uint64_t>(least, dts[i].fine_n);
        }
        if (least * slots >= 8u * all) {
            for (uint32_t i = 0; i < count; ++i) {
                const uint64_t groups = dts[i].fine_n * static_cast<uint64_t>(slots) / all;
                dts[i].fine_item = static_cast<uint32_t>(items_of(dts[i].fine_quanta, groups));
                used += items_of(dts[i].fine_quanta, dts[i].fine_item);
            }
            // (shares are rounded down: what is left goes to the tensor whose workgroups have most to do)
            for (bool more = true; more;) {
                uint32_t top = 0;
                for (uint32_t i = 1; i < count; ++i)
                    if (static_cast<uint64_t>(dts[i].fine_item) * dts[i].fine_units > static_cast<uint64_t>(dts[top].fine_item) * dts[top].fine_units) top = i;
                const uint32_t smaller = dts[top].fine_item - 1u;
                const uint64_t now = items_of(dts[top].fine_quanta, dts[top].fine_item);
                more = smaller != 0 && used - now + items_of(dts[top].fine_quanta, smaller) <= slots;
                if (more) {
                    used += items_of(dts[top].fine_quanta, smaller) - now;
                    dts[top].fine_item = smaller;
                }
            }
        } else {
            uint64_t symbols = 0;
            for (uint32_t i = 0; i < count; ++i) symbols += ts[i].n;
            uint64_t step = std::max<uint64_t>(4096, symbols / (16u * static_cast<uint64_t>(slots)));
            for (;; step *= 2) {
                uint64_t n = 0;
                for (uint32_t i = 0; i < count; ++i) {
                    const uint64_t quantum = static_cast<uint64_t>(dts[i].fix_symbols) * dts[i].fine_units;
                    dts[i].fine_item = static_cast<uint32_t>(std::max<uint64_t>(1, step / quantum));
                    n += items_of(dts[i].fine_quanta, dts[i].fine_item);
                }
                if (n <= L.n_items) break;
            }
        }
        item_units = dts[0].fine_item;
    }
    for (uint32_t i = 0; i < count; ++i) {
        const uint64_t end = shared ? dts[i].share_units : fine ? dts[i].fine_quanta : dts[i].n_chunks;
        const uint64_t step = shared ? share_item_units(dts[i].share_per) : fine ? dts[i].fine_item : static_cast<uint64_t>(item_units) * kUnit;
        for (uint64_t c = 0; c < end; c += step) {
            if (n_items >= L.n_items) return ENTRO_ERR_SIZE;     // (the layout counts the same units: cannot happen)
            items[n_items++] = WorkItem{i, static_cast<uint32_t>(c)};
        }
    }
    plan->workspace = workspace;
    plan->workspace_bytes = workspace_bytes;
    plan->op = op;
    plan->out = out_type;
    plan->count = count;
    plan->n_items = static_cast<uint32_t>(n_items);
    plan->n_fix = static_cast<uint32_t>(n_fix);
    plan->item_units = item_units;
    plan->pair_tables = pairs ? 1u : 0u;
    plan->wide_tables = fine ? 2u : (op == ENTRO_OP_GEMV && !pairs && wide) ? 1u : 0u;
    plan->gemv_multirow = multirow ? 1u : 0u;
    plan->shared_wave_bytes = shared ? wave_bytes : 0u;
    plan->off_tensors = L.off_tensors;
    plan->off_items = L.off_items;
    plan->off_partials = L.off_partials;
    plan->off_fix = L.off_fix;
    return ENTRO_OK;
}

// `once`: the launch is prepared for one run, which a walk through the streams (k_fine) would not pay for.  Others go to k_fine
// where they fit and workspace and staging memory hold what it keeps beside the tables; with less they go the ways of a lane per
// piece or of shared ones, whose room is all that they have to have.
static entro_status plan_checks(entro_plan *plan, const entro_tensor *ts, uint32_t count, entro_op op, void *workspace,
                                uint64_t workspace_bytes, const void *staging, uint64_t staging_bytes, bool once, Layout *L, bool *fine) {
    if (!plan || !ts || !workspace) return ENTRO_ERR_NULL;
    if (count == 0) return ENTRO_ERR_SIZE;
    if (op != ENTRO_OP_DECODE && op != ENTRO_OP_DEQUANT && op != ENTRO_OP_GEMV) return ENTRO_ERR_SCHEME;
    if (!aligned16(workspace)) return ENTRO_ERR_ALIGN;
    *fine = !once && fine_launch(ts, count, op) && plan_layout(ts, count, op, true, L) && workspace_bytes >= L->total &&
            staging_bytes >= L->off_partials;
    if (*fine) return staging ? ENTRO_OK : ENTRO_ERR_NULL;
    if (!plan_layout(ts, count, op, false, L)) return ENTRO_ERR_SIZE;
    if (workspace_bytes < L->total) return ENTRO_ERR_CAPACITY;
    if (!staging) return ENTRO_ERR_NULL;
    return staging_bytes < L->off_partials ? ENTRO_ERR_CAPACITY : ENTRO_OK;
}

// Enqueue the kernel that builds every tensor's lookup tables into the workspace (behind the copy of the
// descriptor table on the same stream).
static entro_status enqueue_tables(const entro_plan *plan, hipStream_t s, bool with_items = false) {
    const DevTensor *dts = reinterpret_cast<const DevTensor *>(static_cast<const unsigned char *>(plan->workspace) + plan->off_tensors);
    if (plan->wide_tables == 2u) {
        // (workgroups without a piece of their tensor end at once; tensors in x, which may be more than 65535)
        const dim3 index_grid(plan->count, std::max(8u, 512u / plan->count));
        if (plan->pair_tables) {
            hipLaunchKernelGGL(k_fine_pairs, dim3(plan->count), dim3(1024), 0, s, dts);
            hipLaunchKernelGGL(k_fine_index<true>, index_grid, dim3(1024), 0, s, dts);
        } else {
            hipLaunchKernelGGL(k_tables<kModeGemvF32W>, dim3(plan->count), dim3(wg_of(kModeGemvF32W)), 0, s, dts, plan->count, nullptr, 0u, 1u);
            hipLaunchKernelGGL(k_fine_index<false>, index_grid, dim3(1024), 0, s, dts);
        }
        return hip_ok(hipGetLastError(), "launch table kernels") ? ENTRO_OK : ENTRO_ERR_DEVICE;
    }
    if (plan->shared_wave_bytes) {                           // (its items have come with the table)
        hipLaunchKernelGGL(k_share_tables, dim3(plan->count), dim3(64u * kShareWaves), 0, s, dts);
        return hip_ok(hipGetLastError(), "launch table kernel") ? ENTRO_OK : ENTRO_ERR_DEVICE;
    }
    const int mode = mode_of(static_cast<entro_op>(plan->op), static_cast<entro_dtype>(plan->out), plan->pair_tables != 0,
                             plan->wide_tables != 0);
    WorkItem *items = reinterpret_cast<WorkItem *>(static_cast<unsigned char *>(plan->workspace) + plan->off_items);
    const unsigned wg = wg_of(mode), writers = with_items ? (plan->n_items + wg - 1u) / wg : 0u;
    dispatch_mode(mode, [&](auto m) {
        constexpr int M = decltype(m)::value;
        hipLaunchKernelGGL(k_tables<M>, dim3(plan->count + writers), dim3(wg), 0, s, dts, plan->count, items, plan->n_items,
                           plan->item_units * kUnit);
    });
    return hip_ok(hipGetLastError(), "launch table kernel") ? ENTRO_OK : ENTRO_ERR_DEVICE;
}

uint64_t entro_plan_staging_bytes(const entro_tensor *ts, uint32_t count, entro_op op) {
    Layout L;
    if (!ts || count == 0 || !plan_layout(ts, count, op, fine_launch(ts, count, op), &L)) return 0;
    return L.off_partials;
}

entro_status entro_plan_init_staged(entro_plan *plan, const entro_tensor *ts, uint32_t count, entro_op op,
                                    entro_dtype out_type, void *workspace, uint64_t workspace_bytes, void *staging,
                                    uint64_t staging_bytes, void *hip_stream) {
    Layout L;
    bool fine;
    entro_status st = plan_checks(plan, ts, count, op, workspace, workspace_bytes, staging, staging_bytes, false, &L, &fine);
    if (st != ENTRO_OK) return st;
    st = build_plan(plan, ts, count, op, out_type, workspace, workspace_bytes, L, static_cast<unsigned char *>(staging), fine);
    if (st != ENTRO_OK) return st;
    if (!hip_ok(hipMemcpyAsync(workspace, staging, L.off_partials, hipMemcpyHostToDevice, static_cast<hipStream_t>(hip_stream)),
                "copy plan table"))
        return ENTRO_ERR_DEVICE;
    return enqueue_tables(plan, static_cast<hipStream_t>(hip_stream));
}

// The table of a launch that is prepared and run in one call travels as arguments of a few small kernels, and its work list is written
// beside the lookup tables (k_tables) unless lanes share segments: a copy from pageable memory has to be waited for, with everything
// in front of it on the stream.  Measured: seven tensors of 218 M symbols to bf16, two such kernels, 187 -> 169 us a call.  Larger
// tables are copied: such a kernel takes 5 us, the copy and the wait about 25 (a call with more of them than three 65.5 -> 68.7).
constexpr uint64_t kMostPuts = 3;

static bool put_table(const entro_plan &plan, const unsigned char *host, hipStream_t s) {
    const DevTensor *dts = reinterpret_cast<const DevTensor *>(host + plan.off_tensors);
    uint32_t n_desc = plan.count;
    for (uint32_t i = 0; i < plan.count; ++i) n_desc = std::max(n_desc, dts[i].fine + 1u);
    const struct {
        uint64_t at, words;
    } parts[3] = {{plan.off_tensors, sizeof(DevTensor) / 4u * static_cast<uint64_t>(n_desc)},
                  {plan.off_items, plan.shared_wave_bytes ? sizeof(WorkItem) / 4u * static_cast<uint64_t>(plan.n_items) : 0u},
                  {plan.off_fix, sizeof(WorkItem) / 4u * static_cast<uint64_t>(plan.n_fix)}};
    static_assert(sizeof(DevTensor) % 4 == 0 && sizeof(WorkItem) % 4 == 0, "whole words");
    uint64_t puts = 0;
    for (const auto &part : parts) puts += items_of(part.words, PutWords::most);
    if (puts > kMostPuts) return false;
    for (const auto &part : parts)
        for (uint64_t from = 0; from < part.words; from += PutWords::most) {
            PutWords words;
            const uint32_t n = static_cast<uint32_t>(std::min<uint64_t>(PutWords::most, part.words - from));
            std::memcpy(words.w, host + part.at + 4u * from, 4u * n);
            std::memset(words.w + n, 0, 4u * (PutWords::most - n));
            hipLaunchKernelGGL(k_put, dim3(1), dim3(PutWords::most), 0, s,
                               reinterpret_cast<uint32_t *>(static_cast<unsigned char *>(plan.workspace) + part.at + 4u * from), n, words);
        }
    return true;
}

static entro_status plan_init(entro_plan *plan, const entro_tensor *ts, uint32_t count, entro_op op, entro_dtype out_type,
                              void *workspace, uint64_t workspace_bytes, bool once, void *hip_stream) {
    Layout L;
    bool fine;
    entro_status st = plan_checks(plan, ts, count, op, workspace, workspace_bytes, plan, UINT64_MAX, once, &L, &fine);
    if (st != ENTRO_OK) return st;
    std::vector<unsigned char> host(L.off_partials);
    st = build_plan(plan, ts, count, op, out_type, workspace, workspace_bytes, L, host.data(), fine);
    if (st != ENTRO_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (once && put_table(*plan, host.data(), s))
        return hip_ok(hipGetLastError(), "launch table kernel") ? enqueue_tables(plan, s, true) : ENTRO_ERR_DEVICE;
    if (!hip_ok(hipMemcpyAsync(workspace, host.data(), host.size(), hipMemcpyHostToDevice, s), "copy plan table"))
        return ENTRO_ERR_DEVICE;
    // the staging vector dies with this call, so wait for the copy
    if (!hip_ok(hipStreamSynchronize(s), "wait for plan table")) return ENTRO_ERR_DEVICE;
    return enqueue_tables(plan, s);
}

entro_status entro_plan_init(entro_plan *plan, const entro_tensor *ts, uint32_t count, entro_op op,
                             entro_dtype out_type, void *workspace, uint64_t workspace_bytes,
                             void *hip_stream) {
    return plan_init(plan, ts, count, op, out_type, workspace, workspace_bytes, false, hip_stream);
}

entro_status entro_plan_run(const entro_plan *plan, void *hip_stream) {
    if (!plan || !plan->workspace) return ENTRO_ERR_NULL;
    if (plan->n_items == 0 || plan->item_units == 0) return ENTRO_ERR_SIZE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const unsigned char *ws = static_cast<const unsigned char *>(plan->workspace);
    const DevTensor *dts = reinterpret_cast<const DevTensor *>(ws + plan->off_tensors);
    const WorkItem *items = reinterpret_cast<const WorkItem *>(ws + plan->off_items);
    const WorkItem *fix = reinterpret_cast<const WorkItem *>(ws + plan->off_fix);
    const int mode = mode_of(static_cast<entro_op>(plan->op), static_cast<entro_dtype>(plan->out), plan->pair_tables != 0,
                             plan->wide_tables != 0);
    const unsigned slots = resident_workgroups(mode);
    if (slots == 0) return ENTRO_ERR_DEVICE;
    const unsigned grid = plan->n_items < slots ? plan->n_items : slots;
    if (plan->wide_tables == 2u) {
        const bool f32 = gemv_f32(mode);
        const auto kernel = plan->pair_tables ? (f32 ? k_fine<true, true> : k_fine<true, false>) : (f32 ? k_fine<false, true> : k_fine<false, false>);
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64u * kFineWaves), 0, s, dts, items, plan->n_items / grid, plan->n_items % grid);
    } else if (plan->shared_wave_bytes) {
        const uint32_t waves = share_waves(plan->shared_wave_bytes);
        dispatch_mode(mode_of(static_cast<entro_op>(plan->op), static_cast<entro_dtype>(plan->out), false), [&](auto m) {
            constexpr int M = decltype(m)::value;
            if constexpr (M <= kModeGemvBF16)
                hipLaunchKernelGGL(k_shared_batch<M>, dim3(grid), dim3(64u * kShareWaves), 0, s, dts, items, plan->n_items, waves,
                                   plan->shared_wave_bytes);
        });
    } else dispatch_mode(mode, [&](auto m) {
        constexpr int M = decltype(m)::value;
        hipLaunchKernelGGL(k_batch<M>, dim3(grid), dim3(wg_of(mode)), 0, s, dts, items, plan->n_items, plan->item_units);
    });
    if (!hip_ok(hipGetLastError(), "launch batched decode kernel")) return ENTRO_ERR_DEVICE;
    if (plan->n_fix) {
        if (gemv_f32(mode)) hipLaunchKernelGGL(k_fix_batch<kModeGemvF32>, dim3(plan->n_fix), dim3(kFixWG), 0, s, dts, fix);
        else hipLaunchKernelGGL(k_fix_batch<kModeGemvBF16>, dim3(plan->n_fix), dim3(kFixWG), 0, s, dts, fix);
        if (!hip_ok(hipGetLastError(), "launch batched row-sum kernel")) return ENTRO_ERR_DEVICE;
    }
    return ENTRO_OK;
}

static entro_status run_batch(const entro_tensor *ts, uint32_t count, entro_op op, entro_dtype d,
                              void *workspace, uint64_t workspace_bytes, void *hip_stream) {
    entro_plan plan;
    // (run once: a walk through the streams beforehand would not pay)
    entro_status st = plan_init(&plan, ts, count, op, d, workspace, workspace_bytes, true, hip_stream);
    if (st != ENTRO_OK) return st;
    return entro_plan_run(&plan, hip_stream);
}

entro_status entro_decode_batch(const entro_tensor *ts, uint32_t count, entro_dtype out_type,
                                void *workspace, uint64_t workspace_bytes, void *hip_stream) {
    return run_batch(ts, count, ENTRO_OP_DECODE, out_type, workspace, workspace_bytes, hip_stream);
}

entro_status entro_decode_dequant_batch(const entro_tensor *ts, uint32_t count, entro_dtype out_type,
                                        void *workspace, uint64_t workspace_bytes, void *hip_stream) {
    return run_batch(ts, count, ENTRO_OP_DEQUANT, out_type, workspace, workspace_bytes, hip_stream);
}

entro_status entro_decode_gemv_batch(const entro_tensor *ts, uint32_t count, entro_dtype y_type,
                                     void *workspace, uint64_t workspace_bytes, void *hip_stream) {
    return run_batch(ts, count, ENTRO_OP_GEMV, y_type, workspace, workspace_bytes, hip_stream);
}

}  // extern "C"
