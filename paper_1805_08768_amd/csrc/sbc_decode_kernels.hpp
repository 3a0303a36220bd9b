// Server step: parallel Golomb position decoding (the supplement's Alg. 4) fused with the
// scaled accumulation of Alg. 1's averaging line.
//
// Alg. 4 is a bit-serial state machine.  At a bit boundary its state is either "reading
// the unary part" (state 0) or "j remainder bits still to read" (state j, 1 <= j <= b).
// A stream is cut into 64-bit segments, one per thread.  For every segment and every one of the b+1
// entry states the exit state is looked up, a byte of the stream at a time, in a table of 256
// functions; an inclusive scan under function composition over the segments gives each segment its
// true entry state.  A position is then a linear function of what precedes its terminating zero:
//     position_i = 2^b * (#unary ones before the zero) + (sum of remainders up to code i) + i
// so prefix sums over segments (unary ones, zeros that end a unary part, remainders)
// place every code without any sequential dependence.
//
//   k_decode          one workgroup per stream, or several that each decode it and share out the updates;
//                     further workgroups compose the functions of the tiles of long streams
//   k_dec_tile_sums,  (tensors that keep very many entries): what k_decode carries from tile to tile in
//   k_dec_tile_place  registers goes through small per-tile arrays there
//   k_decode_generic  b > 15: functions over more than 16 states, as byte arrays in LDS
#pragma once

#include <type_traits>

#include "sbc_device.hpp"

namespace sbc {

constexpr int kDecThreads = 512;
constexpr int kDecWaves = kDecThreads / 64;
constexpr int kMaxB = 30;
constexpr int kStates = kMaxB + 1;
constexpr int kPackedMaxB = 15;               // up to 16 states: functions over them as bytes of four registers

constexpr int kTileWords = 2 * kDecThreads;   // stream words covered by one tile of segments
constexpr int kTileSlack = 2;                 // a remainder may reach this many words past the tile

// What a workgroup of k_decode works on.
struct alignas(8) DecBlock {
    float* out;
    uint32_t n;
    uint32_t t;                               // tensor
    uint32_t share, shares;                   // it applies every shares-th wavefront's updates, from share on
};

struct DecWide {
    float* out;
    uint64_t seg0;        // first segment of this stream in the segment arrays
    uint32_t n;
    uint32_t t;           // tensor
    uint32_t tile0;       // first tile of this stream in the tile arrays
    uint32_t max_tiles;   // tiles reserved for it (from the worst-case stream length)
};
constexpr int kMaxWideDec = 32;               // streams per call that the tile kernels take
struct DecWides { DecWide w[kMaxWideDec]; int count; };      // (a kernel argument)
struct NoWides {};                            // (of a call that has none)

__device__ __forceinline__ void add_to(gfloat_ptr p, float v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// First zero bit of `w` (bit 0 = most significant) at or after offset x (< 64); 64 if none.
__device__ __forceinline__ int first_zero_from(unsigned long long w, int x) {
    const unsigned long long zz = (~w) & (~0ull >> x);
    return zz ? __clzll((long long)zz) : 64;
}

// ---------------------------------------------------------- state functions ----

// A function over 4 D states, one byte per state: D = 2, 3 or 4 for b <= 7, 11 or 15.
template <int D>
struct StateFn { uint32_t v[D]; };

template <int D>
__device__ __forceinline__ StateFn<D> identity_fn() {
    StateFn<D> f;
#pragma unroll
    for (int i = 0; i < D; ++i) f.v[i] = 0x03020100u + 0x04040404u * (uint32_t)i;
    return f;
}

// later o earlier: every byte of `earlier` picks a byte of `later`.  (Byte permutes: 2 to 36 instructions
// for all states, where shifting 4-bit fields took about ten per state and a wavefront's scan 2 us.)
template <int D>
__device__ __forceinline__ StateFn<D> compose(const StateFn<D>& later, const StateFn<D>& earlier) {
    StateFn<D> r;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        const uint32_t e = earlier.v[i];
        if constexpr (D == 2) {
            r.v[i] = __builtin_amdgcn_perm(later.v[1], later.v[0], e);
        } else {
            const uint32_t low = e & 0x07070707u, one = (e >> 3) & 0x01010101u, high = (one << 8) - one;
            const uint32_t a = __builtin_amdgcn_perm(later.v[1], later.v[0], low);
            const uint32_t b = __builtin_amdgcn_perm(later.v[D - 1], later.v[2], low);
            r.v[i] = (b & high) | (a & ~high);
        }
    }
    return r;
}

// f(s) for a state s that is the same in the whole wavefront
template <int D>
__device__ __forceinline__ uint32_t apply_uniform(const StateFn<D> f, uint32_t s) {
    const unsigned long long lo = ((unsigned long long)f.v[1] << 32) | f.v[0];
    unsigned long long hi = 0ull;
    if constexpr (D >= 3) hi = f.v[2];
    if constexpr (D >= 4) hi |= (unsigned long long)f.v[D - 1] << 32;
    const unsigned long long mask = s & 8u ? ~0ull : 0ull;
    return (uint32_t)(((hi & mask) | (lo & ~mask)) >> (8u * (s & 7u))) & 0xFFu;
}

// Inclusive scan under composition over the lanes of a wavefront (ROWS = 4) or of its first row of
// 16 (ROWS = 1); steps as in wave_incl_sum, a lane without a source lane sees the identity.
template <int D, int CTRL, int ROW_MASK>
__device__ __forceinline__ void scan_step(StateFn<D>& f) {
    const StateFn<D> id = identity_fn<D>();
    StateFn<D> o;
#pragma unroll
    for (int i = 0; i < D; ++i)
        o.v[i] = (uint32_t)__builtin_amdgcn_update_dpp((int)id.v[i], (int)f.v[i], CTRL, ROW_MASK, 0xf, false);
    f = compose<D>(f, o);
}
template <int D, int ROWS>
__device__ __forceinline__ void scan_fns(StateFn<D>& f) {
    scan_step<D, 0x111, 0xf>(f);
    scan_step<D, 0x112, 0xf>(f);
    scan_step<D, 0x114, 0xf>(f);
    scan_step<D, 0x118, 0xf>(f);
    if constexpr (ROWS == 4) {
        scan_step<D, 0x142, 0xa>(f);
        scan_step<D, 0x143, 0xc>(f);
    }
}

template <int D>
struct DecShared {
    uint32_t fn[256][D];                      // exit state per entry state for every byte of the stream
    uint32_t wave_fn[kDecWaves][D];
    unsigned long long sums[2][kDecWaves];
};

// The table entry of byte value v.  With g(x) the exit state when Alg. 4 is in its unary state at
// bit x (bit 0 = most significant): g(x) = x - 8 for 8 <= x <= 8 + b, and for x < 8 g(x) = g(x + 1)
// if bit x is a one (one more unary bit), g(x + b + 1) if it is a zero (the code ends b bits later).
// The values are kept as 4-bit fields of one word while x runs from 7 down to 0; entry state s of the
// byte (its first s bits finish a remainder) then exits as field s.
template <int D>
__device__ __forceinline__ void build_table(uint32_t (*fn)[D], uint32_t v, int b) {
    unsigned long long g = 0xFEDCBA9876543210ull;
    const int top = 4 * b;
#pragma nounroll
    for (int i = 0; i < 8; ++i) {
        const unsigned long long one = g & 15ull, zero = (g >> top) & 15ull;
        g = (g << 4) | (((v >> i) & 1u) ? one : zero);
    }
#pragma unroll
    for (int i = 0; i < D; ++i) {
        const uint32_t x = (uint32_t)(g >> (16 * i)) & 0xFFFFu;
        const uint32_t y = (x | (x << 8)) & 0x00FF00FFu;
        fn[v][i] = (y | (y << 4)) & 0x0F0F0F0Fu;
    }
}

// Function of a 64-bit segment, byte by byte.
template <int D>
__device__ __forceinline__ StateFn<D> segment_fn(const uint32_t (*fn)[D], uint32_t hi, uint32_t lo) {
    StateFn<D> f = identity_fn<D>();
#pragma nounroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t w = h ? lo : hi;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t v = (w >> (24 - 8 * i)) & 0xFFu;
            StateFn<D> t;
#pragma unroll
            for (int j = 0; j < D; ++j) t.v[j] = fn[v][j];
            f = compose<D>(t, f);
        }
    }
    return f;
}

// A segment and the word after it (a remainder reaches at most 15 bits into that).
struct Segment {
    uint32_t hi, lo, next;
    __device__ __forceinline__ unsigned long long bits() const { return ((unsigned long long)hi << 32) | lo; }
    // b bits (0 <= b <= 15) from bit x (1 <= x <= 64)
    __device__ __forceinline__ uint32_t field(int x, int b) const {
        const unsigned long long w = x < 32 ? bits() : x < 64 ? ((unsigned long long)lo << 32) | next : (unsigned long long)next << 32;
        return (uint32_t)(((w << (x & 31)) >> 32) >> (32 - b));          // (64-bit shifts: b may be 0)
    }
};

// Word w of a stream of bit_len bits; bits at or past its end read as ones (never a terminator).
__device__ __forceinline__ uint32_t stream_word(const uint32_t* __restrict__ words, unsigned long long w, unsigned long long n_words,
                                                unsigned long long bit_len) {
    if (w >= n_words) return 0xFFFFFFFFu;
    const unsigned long long valid = bit_len - 32ull * w;
    uint32_t v = words[w];
    if (valid < 32ull) v |= 0xFFFFFFFFu >> valid;
    return v;
}
__device__ __forceinline__ Segment stream_segment(const uint32_t* __restrict__ words, unsigned long long seg, unsigned long long n_words,
                                                  unsigned long long bit_len) {
    Segment s;
    s.hi = stream_word(words, 2ull * seg, n_words, bit_len);
    s.lo = stream_word(words, 2ull * seg + 1ull, n_words, bit_len);
    s.next = stream_word(words, 2ull * seg + 2ull, n_words, bit_len);
    return s;
}

// Unary ones, codes and remainders of a segment entered in state `entry`, packed: ones in bits 0..15,
// codes in 16..31, remainders from 32 (a tile of 512 segments holds at most 2^15 of the first two and
// remainders below 2^32 in all).  bits_left: stream bits from the segment's first on; a code that
// would run past them sets bad.  last_end: the bit after the segment's last code, from its first.
__device__ __forceinline__ unsigned long long walk_segment(const Segment& s, int entry, int b, unsigned long long bits_left,
                                                           uint32_t& last_end, bool& bad) {
    const unsigned long long w = s.bits();
    uint32_t ones = 0u, codes = 0u, rem = 0u;
    int x = entry;
    while (x < 64) {
        const int z = first_zero_from(w, x);
        ones += (uint32_t)(z - x);
        if (z == 64) break;
        x = z + b + 1;
        if ((unsigned long long)x > bits_left) { bad = true; break; }
        rem += s.field(z + 1, b);
        ++codes;
        last_end = (uint32_t)x;
    }
    return (unsigned long long)ones | ((unsigned long long)codes << 16) | ((unsigned long long)rem << 32);
}

// The codes of a segment one after another, given the unary ones, codes and remainders of the stream
// before it: next() is the position of the next one (0xFFFFFFFF: none, x is 64 then).
struct CodeWalk {
    const Segment& s;
    unsigned long long ones, codes, rem, bits_left;
    int x, b;
    uint32_t n, nnz;
    bool& bad;
    __device__ __forceinline__ uint32_t next() {
        const int z = first_zero_from(s.bits(), x);
        ones += (unsigned)(z - x);
        x = z == 64 ? 64 : z + b + 1;
        // (a code that runs past the stream's end has been reported by walk_segment)
        if (z == 64 || (unsigned long long)x > bits_left) { x = 64; return 0xFFFFFFFFu; }
        rem += s.field(z + 1, b);
        const unsigned long long pos = (ones << b) + rem + codes;
        if (pos >= n || codes >= nnz) { bad = true; x = 64; return 0xFFFFFFFFu; }
        ++codes;
        return (uint32_t)pos;                          // (below n, so below 0xFFFFFFFF)
    }
};

struct StreamInfo {
    bool ok;
    float mu;
    uint32_t nnz;
    unsigned long long bit_len, word_off, n_words, n_seg;
    const uint32_t* words;
};

// Header and table entry of tensor t, validated.  (The host has checked that the message holds the
// header and T table entries, so all loads go out together.)
__device__ __forceinline__ StreamInfo stream_info(const uint8_t* __restrict__ msg, unsigned long long msg_bytes,
                                                  uint32_t n, int T, int b, int t) {
    StreamInfo si;
    const uint32_t* h = reinterpret_cast<const uint32_t*>(msg);
    const unsigned long long table_end = 32ull + 24ull * (unsigned)T;
    const uint8_t* e = msg + 32 + 24ull * (unsigned)t;
    const uint32_t h0 = h[0], h1 = h[1], h2 = h[2], h3 = h[3];
    const unsigned long long payload_words = *reinterpret_cast<const unsigned long long*>(msg + 16);
    si.mu = *reinterpret_cast<const float*>(e);
    si.nnz = *reinterpret_cast<const uint32_t*>(e + 4);
    si.bit_len = *reinterpret_cast<const unsigned long long*>(e + 8);
    si.word_off = *reinterpret_cast<const unsigned long long*>(e + 16);
    si.ok = msg_bytes >= table_end && h0 == 0x31434253u && h1 == 1u && h2 == (uint32_t)T && h3 == (uint32_t)b;
    si.n_words = (si.bit_len + 31ull) >> 5;
    si.n_seg = (si.bit_len + 63ull) >> 6;
    if (si.ok) {
        const unsigned long long max_words = (msg_bytes - table_end) >> 2;
        si.ok = payload_words <= max_words && si.bit_len <= (max_words << 5) &&
                si.word_off <= payload_words && si.n_words <= payload_words - si.word_off &&
                si.nnz <= n && (unsigned long long)si.nnz * (unsigned)(b + 1) <= si.bit_len &&
                (si.nnz != 0u || si.bit_len == 0ull);
    }
    si.words = reinterpret_cast<const uint32_t*>(msg + table_end) + si.word_off;
    return si;
}

// Where the errors of a decode call go: an error word, or (context-free calls) the caller's status.
__device__ __forceinline__ void report_corrupt(ResultBlock* result, int32_t* status) {
    if (result) atomicOr(&result->err, kErrCorrupt);
    else *status = -4;                        // SBC_ECORRUPT (whoever raises it stores the same value)
}

// --------------------------------------------------------------------------
// One validated stream, tile after tile, by NW wavefronts: a whole workgroup, or one wavefront by
// itself (NW = 1; it then meets no barrier), up to segment seg_end.  f(walk, active, count) is called by
// every lane of a wavefront for which mine(tile) is true and that has a segment of the stream: walk gives the codes of the lane's segment
// (only if `active`), the codes of a wavefront's lanes follow one another, and there are `count` of them;
// bad: the stream is corrupt.  sh.fn must have been built (with NW > 1 a barrier follows before it is read).
// Returns the smallest position that a further code would have.
// --------------------------------------------------------------------------
template <int D, int NW, typename Mine, typename F>
__device__ __forceinline__ unsigned long long decode_codes(DecShared<D>& sh, const StreamInfo& si, uint32_t n, int b,
                                                                 unsigned long long seg_end, Mine mine, bool& bad, F f) {
    const int lane = threadIdx.x & 63, wave = NW > 1 ? (int)(threadIdx.x >> 6) : 0;
    uint32_t carry_state = 0u;
    unsigned long long carry_ones = 0ull, carry_codes = 0ull, carry_rem = 0ull;      // of the tiles so far
    int parity = 0;
    Segment ahead;                                     // of the next tile, on its way during this one
    ahead.hi = ahead.lo = ahead.next = 0xFFFFFFFFu;
    if ((unsigned)(wave * 64) < si.n_seg) ahead = stream_segment(si.words, (unsigned)(wave * 64 + lane), si.n_words, si.bit_len);
    uint32_t tile_no = 0u;
    for (unsigned long long seg0 = 0; seg0 < seg_end; seg0 += 64 * NW, ++tile_no) {
        const unsigned long long seg = seg0 + (unsigned)(wave * 64 + lane);
        const bool busy = seg0 + (unsigned)(wave * 64) < si.n_seg;     // the same for the whole wavefront
        const Segment s = ahead;
        if (seg0 + (unsigned)(64 * NW + wave * 64) < si.n_seg) ahead = stream_segment(si.words, seg + 64 * NW, si.n_words, si.bit_len);
        if (NW > 1) __syncthreads();                   // the table; the tile before this one is done with LDS
        SBC_TS(2, 2);
        StateFn<D> fn = identity_fn<D>();
        if (busy) {
            fn = segment_fn<D>(sh.fn, s.hi, s.lo);
            scan_fns<D, 4>(fn);
        }
        // state in which this wavefront is entered, from the functions of those before it
        uint32_t entry_wave = carry_state;
        if constexpr (NW > 1) {
            if (lane == 63) {
#pragma unroll
                for (int i = 0; i < D; ++i) sh.wave_fn[wave][i] = fn.v[i];
            }
            __syncthreads();
            SBC_TS(2, 3);
            StateFn<D> g = identity_fn<D>();
            if (lane < NW) {
#pragma unroll
                for (int i = 0; i < D; ++i) g.v[i] = sh.wave_fn[lane][i];
            }
            scan_fns<D, 1>(g);
            const uint32_t through = apply_uniform<D>(g, carry_state);     // lane w: after wavefronts 0..w
            if (wave) entry_wave = (uint32_t)__builtin_amdgcn_readlane((int)through, wave - 1);
            carry_state = (uint32_t)__builtin_amdgcn_readlane((int)through, NW - 1);
        }
        const uint32_t up_to = apply_uniform<D>(fn, entry_wave);           // after this lane's segment
        if constexpr (NW == 1) carry_state = last_lane(up_to);
        const uint32_t before = __shfl_up(up_to, 1, 64);
        const int entry = lane ? (int)before : (int)entry_wave;
        const unsigned long long bits_left = si.bit_len > 64ull * seg ? si.bit_len - 64ull * seg : 0ull;
        uint32_t last_end = 0u;
        unsigned long long own = 0ull;
        if (seg < si.n_seg) own = walk_segment(s, entry, b, bits_left, last_end, bad);
        const unsigned long long inc = wave_incl_sum(own);
        unsigned long long tile = last_lane(inc), ex = inc - own;
        if constexpr (NW > 1) {
            if (lane == 63) sh.sums[parity][wave] = inc;
            __syncthreads();
            SBC_TS(2, 4);
            const unsigned long long ws = wave_incl_sum(lane < NW ? sh.sums[parity][lane] : 0ull);
            tile = last_lane(ws);
            if (wave) ex += ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(ws >> 32), wave - 1) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ws, wave - 1);
            parity ^= 1;
        }
        const unsigned long long codes = carry_codes + ((ex >> 16) & 0xFFFFull);
        const uint32_t n_own = (uint32_t)(own >> 16) & 0xFFFFu;
        // the stream's last code ends the stream exactly
        if (n_own && codes + n_own == si.nnz && (unsigned long long)last_end != bits_left) bad = true;
        if (busy && mine(tile_no)) {
            CodeWalk w = {s, carry_ones + (ex & 0xFFFFull), codes, carry_rem + (ex >> 32), bits_left, entry, b, n, si.nnz, bad};
            f(w, seg < si.n_seg && !bad, (uint32_t)(last_lane(inc) >> 16) & 0xFFFFu);
        }
        carry_ones += tile & 0xFFFFull; carry_codes += (tile >> 16) & 0xFFFFull; carry_rem += tile >> 32;
        SBC_TS(2, 5);
    }
    if (seg_end >= si.n_seg && carry_codes != si.nnz) bad = true;      // identical in every thread
    return (carry_ones << b) + carry_rem + carry_codes;
}

// A stream's updates.  An update out[j] += fl32(scale * mu) is an atomic that returns nothing: one access
// per entry instead of a load and a store, and no wait, for a compute unit sustains only about one
// scattered access per 3 ns (ResNet-50 shape: k_decode 8.4 us, 11.3 with loads and stores at p = 0.001).
// Positions of a message are distinct, so each address sees one rounded fp32 addition either way.
template <int D>
__device__ __forceinline__ void decode_stream(DecShared<D>& sh, const uint8_t* __restrict__ msg, unsigned long long msg_bytes,
                                              const DecBlock& blk, int T, int b, float scale, ResultBlock* result, int32_t* status) {
    const int tid = threadIdx.x, wave = tid >> 6;
    const StreamInfo si = stream_info(msg, msg_bytes, blk.n, T, b, (int)blk.t);
    if (tid < 256) build_table<D>(sh.fn, (uint32_t)tid, b);            // (while the header is on its way)
    SBC_TS(2, 1);
    if (!si.ok) {
        if (tid == 0) report_corrupt(result, status);
        return;
    }
    if (si.nnz == 0u) return;
    const float addend = scale * si.mu;
    const gfloat_ptr out = as_global(blk.out);
    bool bad = false;
    const bool mine = (uint32_t)wave % blk.shares == blk.share;
    decode_codes<D, kDecWaves>(sh, si, blk.n, b, si.n_seg, [&](uint32_t) { return mine; }, bad, [&](CodeWalk& w, bool active, uint32_t) {
        if (active)
            while (w.x < 64) {
                const uint32_t at = w.next();
                if (at != 0xFFFFFFFFu) add_to(out + at, addend);
            }
    });
    if (bad) report_corrupt(result, status);
    SBC_TS(2, 6);
}

// Where the workgroups of a decode kernel find what to work on: a table in memory, or (context-free
// calls) the kernel's arguments.
struct MemBlocks {
    const DecBlock* table;
    ResultBlock* result;
    ResultBlock* next_result;                 // left clean for the next call
    __device__ __forceinline__ DecBlock at(uint32_t i) const { return table[i]; }
    __device__ __forceinline__ ResultBlock* errors() const { return result; }
    __device__ __forceinline__ int32_t* status_word() const { return nullptr; }
    __device__ __forceinline__ void begin() const {
        if (blockIdx.x == 0 && threadIdx.x == 0) next_result->err = 0u;
    }
};

// Tile `tile` of long stream w: its segments' functions composed, for the tiles after it.
template <int D>
__device__ __forceinline__ void tile_function(DecShared<D>& sh, const uint8_t* __restrict__ msg, unsigned long long msg_bytes,
                                              const DecWide& w, uint32_t tile, int T, int b, uint4* __restrict__ tile_fn,
                                              ResultBlock* result) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const StreamInfo si = stream_info(msg, msg_bytes, w.n, T, b, (int)w.t);
    if (tid < 256) build_table<D>(sh.fn, (uint32_t)tid, b);
    const unsigned long long n_tiles = (si.n_seg + kDecThreads - 1) / kDecThreads;
    if (!si.ok || n_tiles > w.max_tiles) {                // a valid stream never exceeds its worst case
        if (tile == 0 && tid == 0) report_corrupt(result, nullptr);
        return;
    }
    if (tile + 1u >= n_tiles) return;                     // (nobody asks for the last one's)
    const Segment s = stream_segment(si.words, (unsigned long long)tile * kDecThreads + (unsigned)tid, si.n_words, si.bit_len);
    __syncthreads();
    StateFn<D> f = segment_fn<D>(sh.fn, s.hi, s.lo);
    scan_fns<D, 4>(f);
    if (lane == 63) {
#pragma unroll
        for (int i = 0; i < D; ++i) sh.wave_fn[wave][i] = f.v[i];
    }
    __syncthreads();
    if (tid >= 64) return;
    StateFn<D> g = identity_fn<D>();
    if (lane < kDecWaves) {
#pragma unroll
        for (int i = 0; i < D; ++i) g.v[i] = sh.wave_fn[lane][i];
    }
    scan_fns<D, 1>(g);
    if (lane == kDecWaves - 1) {
        uint32_t v[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < D; ++i) v[i] = g.v[i];
        tile_fn[w.tile0 + tile] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

__device__ __forceinline__ int stream_of_tile(const DecWides& dw, uint32_t tile) {
    int which = 0;
#pragma nounroll
    for (int i = 1; i < dw.count; ++i) if (tile >= dw.w[i].tile0) which = i;      // (the streams' tiles lie one after another)
    return which;
}

// The first n_blocks workgroups decode short streams whole; the others take the tiles of the long ones.
template <int D, typename Blocks, typename Wides>
__global__ __launch_bounds__(kDecThreads) void k_decode(const uint8_t* __restrict__ msg, unsigned long long msg_bytes,
                                                        const Blocks blocks, uint32_t n_blocks, int T, int b, float scale,
                                                        const Wides dw, uint4* __restrict__ tile_fn) {
    __shared__ __attribute__((aligned(16))) DecShared<D> sh;
    SBC_TS(2, 0);
    blocks.begin();
    if (blockIdx.x < n_blocks) {
        const DecBlock blk = blocks.at(blockIdx.x);
        decode_stream<D>(sh, msg, msg_bytes, blk, T, b, scale, blocks.errors(), blocks.status_word());
    } else if constexpr (std::is_same_v<Wides, DecWides>) {
        const uint32_t tile = blockIdx.x - n_blocks;
        const DecWide& w = dw.w[stream_of_tile(dw, tile)];
        tile_function<D>(sh, msg, msg_bytes, w, tile - w.tile0, T, b, tile_fn, blocks.errors());
    }
}

// --------------------------------------------------------------------------
// Long streams.  k_dec_tile_sums, per tile: the state in which the tile is entered, from the functions
// of the tiles before it (every tile folds them by itself: a few hundred small values, cheaper than a
// launch in between); then per segment its entry state and the unary ones, codes and remainders before
// it in the tile (seg_pack: as walk_segment packs them, the state from bit 58), and the tile's totals.
// --------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kDecThreads) void k_dec_tile_sums(
        const uint8_t* __restrict__ msg, unsigned long long msg_bytes, const DecWides dw, int T, int b,
        const uint4* __restrict__ tile_fn, unsigned long long* __restrict__ seg_pack,
        unsigned long long* __restrict__ tile_sum, ResultBlock* __restrict__ result) {
    __shared__ __attribute__((aligned(16))) DecShared<D> sh;
    __shared__ uint32_t before_fn[kDecWaves][D];
    const DecWide& w = dw.w[stream_of_tile(dw, blockIdx.x)];
    const uint32_t tile = blockIdx.x - w.tile0;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const StreamInfo si = stream_info(msg, msg_bytes, w.n, T, b, (int)w.t);
    if (tid < 256) build_table<D>(sh.fn, (uint32_t)tid, b);
    // the tiles before this one: a run of them per thread
    StateFn<D> p = identity_fn<D>();
    const uint32_t per = (tile + kDecThreads - 1) / kDecThreads;
    for (uint32_t j = 0; j < per; ++j) {
        const uint32_t i = (uint32_t)tid * per + j;
        if (i < tile) {
            const uint4 v = tile_fn[w.tile0 + i];
            const uint32_t a[4] = {v.x, v.y, v.z, v.w};
            StateFn<D> q;
#pragma unroll
            for (int k = 0; k < D; ++k) q.v[k] = a[k];
            p = compose<D>(q, p);
        }
    }
    const unsigned long long n_tiles = (si.n_seg + kDecThreads - 1) / kDecThreads;
    if (!si.ok || n_tiles > w.max_tiles || tile >= n_tiles) return;
    const unsigned long long seg = (unsigned long long)tile * kDecThreads + (unsigned)tid;
    const Segment s = stream_segment(si.words, seg, si.n_words, si.bit_len);
    scan_fns<D, 4>(p);
    if (lane == 63) {
#pragma unroll
        for (int i = 0; i < D; ++i) before_fn[wave][i] = p.v[i];
    }
    __syncthreads();
    StateFn<D> f = segment_fn<D>(sh.fn, s.hi, s.lo);
    scan_fns<D, 4>(f);
    if (lane == 63) {
#pragma unroll
        for (int i = 0; i < D; ++i) sh.wave_fn[wave][i] = f.v[i];
    }
    __syncthreads();
    StateFn<D> g = identity_fn<D>(), h = identity_fn<D>();
    if (lane < kDecWaves) {
#pragma unroll
        for (int i = 0; i < D; ++i) { g.v[i] = sh.wave_fn[lane][i]; h.v[i] = before_fn[lane][i]; }
    }
    scan_fns<D, 1>(h);
    const uint32_t state = (uint32_t)__builtin_amdgcn_readlane((int)apply_uniform<D>(h, 0u), kDecWaves - 1);
    scan_fns<D, 1>(g);
    const uint32_t through = apply_uniform<D>(g, state);
    const uint32_t entry_wave = wave ? (uint32_t)__builtin_amdgcn_readlane((int)through, wave - 1) : state;
    const uint32_t before = __shfl_up(apply_uniform<D>(f, entry_wave), 1, 64);
    const uint32_t entry = lane ? before : entry_wave;
    const unsigned long long bits_left = si.bit_len > 64ull * seg ? si.bit_len - 64ull * seg : 0ull;
    uint32_t last_end = 0u;
    bool bad = false;
    unsigned long long own = 0ull;
    if (seg < si.n_seg) own = walk_segment(s, (int)entry, b, bits_left, last_end, bad);
    if (bad) report_corrupt(result, nullptr);
    const unsigned long long inc = wave_incl_sum(own);
    if (lane == 63) sh.sums[0][wave] = inc;
    __syncthreads();
    const unsigned long long ws = wave_incl_sum(lane < kDecWaves ? sh.sums[0][lane] : 0ull);
    const unsigned long long ws_before =
        wave ? ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(ws >> 32), wave - 1) << 32) |
                   (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ws, wave - 1)
             : 0ull;
    seg_pack[w.seg0 + seg] = (ws_before + inc - own) | ((unsigned long long)entry << 58);
    if (tid == 63) tile_sum[w.tile0 + tile] = last_lane(ws);
}

// Positions, checks and updates; a workgroup takes a quarter of a tile, so that the scattered updates
// spread evenly over the compute units.  The last one of a stream checks the code count against nnz.
constexpr int kPlaceThreads = 128;
constexpr uint32_t kPlacePer = kDecThreads / kPlaceThreads;

__global__ __launch_bounds__(kPlaceThreads) void k_dec_tile_place(
        const uint8_t* __restrict__ msg, unsigned long long msg_bytes, const DecWides dw, int T, int b, float scale,
        const unsigned long long* __restrict__ seg_pack, const unsigned long long* __restrict__ tile_sum,
        ResultBlock* __restrict__ result) {
    __shared__ unsigned long long part[3][kPlaceThreads / 64];
    const uint32_t any_tile = blockIdx.x / kPlacePer;
    const DecWide& w = dw.w[stream_of_tile(dw, any_tile)];
    const uint32_t tile = any_tile - w.tile0;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const StreamInfo si = stream_info(msg, msg_bytes, w.n, T, b, (int)w.t);
    // unary ones, codes and remainders of the tiles before this one
    unsigned long long sum[3] = {0ull, 0ull, 0ull};
    for (uint32_t i = (uint32_t)tid; i < tile; i += kPlaceThreads) {
        const unsigned long long v = tile_sum[w.tile0 + i];
        sum[0] += v & 0xFFFFull; sum[1] += (v >> 16) & 0xFFFFull; sum[2] += v >> 32;
    }
    const unsigned long long n_tiles = (si.n_seg + kDecThreads - 1) / kDecThreads;
    if (!si.ok || n_tiles > w.max_tiles || tile >= n_tiles) return;
    const unsigned long long seg = (unsigned long long)tile * kDecThreads + (blockIdx.x % kPlacePer) * kPlaceThreads + (unsigned)tid;
    const Segment s = stream_segment(si.words, seg, si.n_words, si.bit_len);
    const unsigned long long pk = seg_pack[w.seg0 + seg];              // (the array holds whole tiles)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const unsigned long long x = wave_incl_sum(sum[j]);
        if (lane == 63) part[j][wave] = x;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        sum[j] = 0ull;
#pragma unroll
        for (int i = 0; i < kPlaceThreads / 64; ++i) sum[j] += part[j][i];
    }
    bool bad = false;
    if (tile + 1u == n_tiles && blockIdx.x % kPlacePer == 0u && tid == 0) {
        const unsigned long long v = tile_sum[w.tile0 + tile];
        if (sum[1] + ((v >> 16) & 0xFFFFull) != si.nnz) bad = true;
    }
    if (seg < si.n_seg) {
        const unsigned long long bits_left = si.bit_len - 64ull * seg;
        const unsigned long long ones = sum[0] + (pk & 0xFFFFull), codes = sum[1] + ((pk >> 16) & 0xFFFFull),
                                 rem = sum[2] + ((pk >> 32) & 0x3FFFFFFull);
        const int entry = (int)(pk >> 58);
        // the stream's last code ends the stream exactly
        uint32_t last_end = 0u;
        if (codes + 64u >= si.nnz) {                   // (only near its end: the codes of one segment)
            bool b2 = false;
            const unsigned long long own = walk_segment(s, entry, b, bits_left, last_end, b2);
            const uint32_t n_own = (uint32_t)(own >> 16) & 0xFFFFu;
            if (n_own && codes + n_own == si.nnz && (unsigned long long)last_end != bits_left) bad = true;
        }
        // Up to eight loads in flight, then their stores: updates spread over the chip are bound by the lines they
        // touch in memory (66e6 entries, 660,000 updates: 25.9 us, 36.0 with atomics).
        CodeWalk cw = {s, ones, codes, rem, bits_left, entry, b, w.n, si.nnz, bad};
        const gfloat_ptr o = as_global(w.out);
        const float addend = scale * si.mu;
        while (cw.x < 64) {
            uint32_t at[8];
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) at[j] = cw.x < 64 ? cw.next() : 0xFFFFFFFFu;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = at[j] != 0xFFFFFFFFu ? o[at[j]] : 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) if (at[j] != 0xFFFFFFFFu) o[at[j]] = v[j] + addend;
        }
    }
    if (bad) report_corrupt(result, nullptr);
}

// --------------------------------------------------------------------------
// b > 15 (p below about 1.5e-5): transition functions over up to 31 states, one byte per state in LDS.
// --------------------------------------------------------------------------
// b bits (MSB first, 0 <= b <= 30) starting at bit `pos` of the tile staged in LDS.
__device__ __forceinline__ uint32_t read_bits(const uint32_t* tile, uint32_t pos, int b) {
    if (b == 0) return 0u;
    const uint32_t w = pos >> 5;
    const int off = (int)(pos & 31u);
    const unsigned long long v = ((unsigned long long)tile[w] << 32) | tile[w + 1];
    return (uint32_t)((v >> (64 - off - b)) & ((1ull << b) - 1ull));
}

// State in which Alg. 4 leaves a 64-bit segment that it enters in state s (the first s bits
// finish a remainder).
__device__ __forceinline__ int exit_state_of(unsigned long long w64, int s, int b) {
    int x = s;
    while (true) {
        if (x >= 64) return x - 64;
        const int z = first_zero_from(w64, x);
        if (z == 64) return 0;
        x = z + b + 1;
    }
}

template <typename Blocks>
__global__ __launch_bounds__(kDecThreads) void k_decode_generic(const uint8_t* __restrict__ msg, unsigned long long msg_bytes,
                                                                const Blocks blocks, int T, int b, float scale) {
    __shared__ uint8_t fn[2][kStates][kDecThreads];       // transition functions, [state][segment]
    __shared__ unsigned long long scratch64[kDecWaves];
    __shared__ uint32_t s_state;
    __shared__ uint32_t tile[kTileWords + kTileSlack];    // words past the stream read as ones
    const int tid = threadIdx.x;
    blocks.begin();
    const DecBlock blk = blocks.at(blockIdx.x);
    const bool mine = ((uint32_t)tid % blk.shares) == blk.share;
    const StreamInfo si = stream_info(msg, msg_bytes, blk.n, T, b, (int)blk.t);
    if (!si.ok) {
        if (tid == 0) report_corrupt(blocks.errors(), blocks.status_word());
        return;
    }
    if (si.nnz == 0u) return;
    const float addend = scale * si.mu;
    const int S = b + 1;                                  // number of states
    int carry_state = 0;
    unsigned long long carry_U = 0ull, carry_T = 0ull, carry_R = 0ull;   // unary ones, codes, remainders so far
    bool bad = false;
    for (unsigned long long seg0 = 0; seg0 < si.n_seg; seg0 += kDecThreads) {
        const unsigned long long seg = seg0 + (unsigned)tid;
        __syncthreads();
        for (int i = tid; i < kTileWords + kTileSlack; i += kDecThreads)
            tile[i] = stream_word(si.words, 2ull * seg0 + (unsigned)i, si.n_words, si.bit_len);
        __syncthreads();
        const unsigned long long w64 = ((unsigned long long)tile[2 * tid] << 32) | tile[2 * tid + 1];
        // ---- exit state for every entry state ----
        int ex = exit_state_of(w64, 0, b);
        fn[0][0][tid] = (uint8_t)ex;
        for (int s = 1; s < S; ++s) {
            if (!((w64 >> (64 - s)) & 1ull)) ex = exit_state_of(w64, s, b);
            fn[0][s][tid] = (uint8_t)ex;
        }
        __syncthreads();
        // ---- inclusive scan under composition: fn[cur][.][i] = f_i o ... o f_0 ----
        int cur = 0;
        for (int dlt = 1; dlt < kDecThreads; dlt <<= 1) {
            for (int s = 0; s < S; ++s) {
                uint8_t v;
                if (tid >= dlt) v = fn[cur][fn[cur][s][tid - dlt]][tid];
                else v = fn[cur][s][tid];
                fn[cur ^ 1][s][tid] = v;
            }
            __syncthreads();
            cur ^= 1;
        }
        const int entry = (tid == 0) ? carry_state : (int)fn[cur][carry_state][tid - 1];
        if (tid == kDecThreads - 1) s_state = fn[cur][carry_state][tid];
        __syncthreads();
        carry_state = (int)s_state;
        // ---- unary ones, terminators and remainder sum of this segment ----
        uint32_t nU = 0u, nT = 0u;
        unsigned long long sR = 0ull, last_end = 0ull;
        if (seg < si.n_seg) {
            int x = entry;
            while (x < 64) {
                const int z = first_zero_from(w64, x);
                nU += (uint32_t)(z - x);
                if (z == 64) break;
                const unsigned long long end = seg * 64ull + (unsigned)z + 1ull + (unsigned)b;
                if (end > si.bit_len) { bad = true; break; }
                sR += read_bits(tile, (uint32_t)(tid * 64 + z + 1), b);
                ++nT;
                last_end = end;
                x = z + b + 1;
            }
        }
        unsigned long long tile_U, tile_T, tile_R;
        const unsigned long long exU = block_excl_sum<unsigned long long, kDecThreads>(nU, &tile_U, scratch64);
        const unsigned long long exT = block_excl_sum<unsigned long long, kDecThreads>(nT, &tile_T, scratch64);
        const unsigned long long exR = block_excl_sum<unsigned long long, kDecThreads>(sR, &tile_R, scratch64);
        // ---- place every code whose terminating zero lies in this segment ----
        if (seg < si.n_seg && !bad) {
            unsigned long long U = carry_U + exU, Tn = carry_T + exT, R = carry_R + exR;
            // the stream's last code ends the stream exactly
            if (nT > 0u && Tn + nT == (unsigned long long)si.nnz && last_end != si.bit_len) bad = true;
            int x = entry;
            while (mine && !bad && x < 64) {
                const int z = first_zero_from(w64, x);
                U += (unsigned)(z - x);
                if (z == 64) break;
                R += read_bits(tile, (uint32_t)(tid * 64 + z + 1), b);
                const unsigned long long pos = (U << b) + R + Tn;
                if (pos >= blk.n || Tn >= si.nnz) { bad = true; break; }
                add_to(as_global(blk.out) + pos, addend);
                ++Tn;
                x = z + b + 1;
            }
        }
        carry_U += tile_U; carry_T += tile_T; carry_R += tile_R;
    }
    if (carry_T != si.nnz) bad = true;         // identical in every thread
    if (bad) report_corrupt(blocks.errors(), blocks.status_word());
}

}  // namespace sbc
