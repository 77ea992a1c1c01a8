// The device's search for starts inside segments (find_start) as host code: a lane is a thread, and what lanes do
// together (ballots, shuffles, barriers) is a rendezvous of the 64 of them.  "search.inc" is the device source's own
// text, cut out by the test that builds this.
#include <barrier>
#include <cstdint>
#include <cstring>
#include <thread>
#include <type_traits>
#include <vector>

#define ENTRO_MAX_CODE_LEN 32
#define __device__
#define __forceinline__ inline
#define __noinline__

namespace {

thread_local struct { uint32_t x; } threadIdx;
std::barrier<> *wavefront;
uint64_t said[64];                       // what every lane brings to a ballot or a shuffle

void wave_sync_lds() { wavefront->arrive_and_wait(); }

template <class F>
auto together(uint64_t mine, F f) {
    said[threadIdx.x] = mine;
    wave_sync_lds();
    const auto res = f();
    wave_sync_lds();
    return res;
}

uint64_t ballot(bool b) {
    return together(b, [] {
        uint64_t m = 0;
        for (int l = 0; l < 64; ++l) m |= said[l] << l;
        return m;
    });
}

uint32_t shuffle(uint32_t v, uint32_t from) {
    return together(v, [&] { return static_cast<uint32_t>(said[from & 63u]); });
}

uint32_t bits_reversed(uint32_t v) {
    uint32_t r = 0;
    for (int i = 0; i < 32; ++i) r |= (v >> i & 1u) << (31 - i);
    return r;
}

#define __builtin_amdgcn_ballot_w64 ballot
#define __builtin_amdgcn_ubfe(v, at, n) (((v) >> (at)) & ((1u << (n)) - 1u))
#define __shfl_up(v, d, width) shuffle(v, threadIdx.x >= (d) ? threadIdx.x - (d) : threadIdx.x)
#define __shfl(v, l, width) shuffle(v, l)
#define __brev bits_reversed
#define __hip_atomic_fetch_or(p, v, order, scope) __atomic_fetch_or(p, v, __ATOMIC_RELAXED)

#include "search.inc"

// Canonical tables straight from the definition; longer codes than the table's are left to the canonical search.
template <bool PAIR>
void fill_tables(Tables &tb, const uint8_t *len, int n_len) {
    std::memset(&tb, 0, sizeof(tb));
    for (int s = 0; s < n_len; ++s)
        if (len[s]) ++tb.cnt[len[s]];
    uint32_t code = 0, off = 0;
    for (uint32_t b = 1; b <= ENTRO_MAX_CODE_LEN; ++b) {
        tb.first[b] = code;
        tb.offs[b] = off;
        for (int s = 0; s < n_len; ++s)
            if (len[s] == b) tb.sorted[off++] = static_cast<uint8_t>(s);
        code = (code + tb.cnt[b]) << 1;
    }
    const uint32_t bits = PAIR ? kSingleBits : kL1;
    for (uint32_t i = 0; i < (1u << bits); ++i) {
        uint32_t e = PAIR ? 0u : 7u << 8;
        for (uint32_t l = 1; l <= bits; ++l) {
            const uint32_t d = (bits_reversed(i) >> (32 - l)) - tb.first[l];
            if (d < tb.cnt[l]) e = pack_entry(tb.sorted[tb.offs[l] + d], l);
        }
        (PAIR ? tb.lut2[i] : tb.lut[i]) = static_cast<uint16_t>(e);
    }
}

template <bool PAIR>
int all_starts(const DevTensor &t, const uint8_t *len, int n_len, uint64_t *starts) {
    static Tables tb;
    static uint32_t ring[kRing2Dwords * 64];
    fill_tables<PAIR>(tb, len, n_len);
    int given_up = 0;
    for (uint32_t first = 0; first < t.n_chunks; first += 64) {
        for (uint32_t &r : ring) r = 0xdeadbeefu;
        std::barrier<> meet(64);
        wavefront = &meet;
        Unit unit[64];
        uint64_t start[64];
        std::vector<std::thread> lanes;
        for (uint32_t l = 0; l < 64; ++l)
            lanes.emplace_back([&, l] {
                threadIdx.x = l;
                unit[l] = {first, t.n_chunks, t.chunk_symbols};
                start[l] = find_start<PAIR>(t, tb, ring, unit[l]);
            });
        for (std::thread &lane : lanes) lane.join();
        const Unit &u = unit[0];
        const bool found = u.symbols == t.chunk_symbols;
        for (uint32_t l = 0; l < 64; ++l) {
            if (std::memcmp(&unit[l], &u, sizeof(u))) return -1;          // the lanes must agree on what they work on
            if (u.first + l < u.end) starts[(u.first + l) << (found ? 0u : t.sub_shift)] = start[l];
        }
        given_up += !found;
    }
    return given_up;
}

}  // namespace

// Start bits of a tensor's pieces of chunk >> shift symbols, as the wavefronts find them; only those of whole segments
// where a wavefront gives up.  Returns how many did (-1: lanes of a wavefront disagree).
extern "C" int host_starts(const uint8_t *stream, uint32_t stream_bytes, const uint64_t *offsets, uint64_t n, uint32_t chunk, uint32_t shift,
                           const uint8_t *len, int n_len, int max_len, uint64_t *starts) {
    DevTensor t = {};
    t.stream = stream;
    t.stream_bytes = stream_bytes;
    t.offsets = offsets;
    t.n = n;
    t.max_len = static_cast<uint32_t>(max_len);
    t.chunk_symbols = chunk >> shift;
    t.sub_shift = shift;
    t.n_chunks = static_cast<uint32_t>((n + t.chunk_symbols - 1) / t.chunk_symbols);
    return n_len == 16 ? all_starts<true>(t, len, n_len, starts) : all_starts<false>(t, len, n_len, starts);
}
