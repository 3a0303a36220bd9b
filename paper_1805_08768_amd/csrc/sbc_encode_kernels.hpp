// The rest of the client step once the thresholds are known, a wavefront per chunk of 8192 entries:
//   k_emit_all : calls of few tensors and up to 3584 chunks, everything behind the streaming pass in one launch: the sides'
//                selection (select_side), Alg. 2's side decision, Alg. 1's residual line and Alg. 3, the message
//   k_apply    : the same steps as launches of their own, for calls of more chunks or tensors, for the second pass and behind
//                the streaming kernel that finishes tensors: side decision, residual line and Alg. 3 within the
//                chunk, from the chunk's run of candidates: the codes of all its kept entries but the first, whose
//                predecessor lies in another chunk, as a bit string of its own, and a summary
//   k_emit_scan : up to 4096 chunks: every workgroup scans the summaries of the call's chunks (predecessors, bit
//                offsets, the tensors' places in the payload), then every wavefront puts its chunk's first code and bit
//                string together, shifted to their place
//   k_tile_summary, k_tensor_scan, k_emit : more chunks: the scan over a tensor's chunks in tiles of 4096 (predecessors, bit
//                offsets), then every wavefront puts its chunk's first code and bit string together, shifted to their
//                place (into the message, or, behind the streaming kernel that finishes tensors, into the
//                tensors' staging words, from which k_finish_message assembles the message)
//
// Candidates of one chunk sit next to each other in their tensor's lists (a workgroup of the
// streaming kernel appends them as one run), so the chunk is the unit of work here and no kept
// position is ever sorted: a bitmap, in LDS, puts a chunk's in order, and chunks are in order.
//
// A word of the payload is written once, whole, by the chunk that its first bit belongs to, which adds
// the first bits of the chunks behind it (k_emit_all: its last bit, and the last bits of those before it): nothing
// has to be cleared beforehand, no word is shared through atomics and nothing is copied afterwards.
#pragma once

#include "sbc_device.hpp"
#include "sbc_threshold_kernels.hpp"

namespace sbc {

constexpr int kEncThreads = 256;
constexpr int kEncWaves = kEncThreads / 64;
static_assert(kChunkWords == 256, "four bitmap words per lane");

__device__ __forceinline__ uint32_t golomb_len(uint32_t gap, int b) { return (gap >> b) + 1u + (uint32_t)b; }

// LDS that only one wavefront touches needs no barrier: its LDS operations complete in order, and
// this keeps the compiler from moving them across.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive prefix maximum over a wavefront (identity 0); *total: the maximum.
__device__ __forceinline__ uint32_t wave_excl_max(uint32_t v, uint32_t* total) {
    const uint32_t inc = wave_incl_max(v);
    *total = last_lane(inc);
    const uint32_t prev = __shfl_up(inc, 1, 64);
    return (threadIdx.x & 63) ? prev : 0u;
}
// Does a pass of k_apply / k_emit work on a tensor with these state flags?  (kPassAll: behind k_emit_all, which
// leaves the scan over the chunks to the second pass, of every tensor that has been selected.)
constexpr int kPassAll = 2;
__device__ __forceinline__ bool encoded_in_pass(uint32_t flags, int pass) {
    if (pass == kPassAll) return (flags & kStFailed) == 0u;
    return pass == 0 ? (flags & (kStInlineDone | kStDeferred | kStFailed)) == 0u : (flags & (kStExact | kStDeferred)) != 0u;
}

__device__ __forceinline__ uint32_t word_of(const uint4& v, int j) { return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w; }

// f(position in the chunk) for every set bit of a lane's four bitmap words, ascending.  (One body,
// whatever the word: these kernels run their code once from a cold instruction cache.)
template <typename F>
__device__ __forceinline__ void for_bits(const uint4& words, uint32_t first_pos, F f) {
    unsigned long long m = ((unsigned long long)words.y << 32) | words.x, rest = ((unsigned long long)words.w << 32) | words.z;
    if (m == 0ull) { m = rest; rest = 0ull; first_pos += 64u; }
    while (m) {
        f(first_pos + (uint32_t)(__ffsll((long long)m) - 1));
        m &= m - 1ull;
        if (m == 0ull) { m = rest; rest = 0ull; first_pos += 64u; }
    }
}
// position + 1 of the last set bit (0: none)
__device__ __forceinline__ uint32_t last_bit_end(const uint4& w, uint32_t first_pos) {
    const int j = w.w ? 3 : w.z ? 2 : w.y ? 1 : 0;
    const uint32_t m = word_of(w, j);
    return m ? first_pos + (uint32_t)(32 * j) + 32u - (uint32_t)__clz((int)m) : 0u;
}


// ------------------------------------------------------- codes of a chunk ----

// A chunk's kept entries as each lane's four bitmap words, and where the lane's codes start.
struct ChunkCodes {
    uint4 words;
    uint32_t p0;          // position (in the chunk) of the lane's first bit
    uint32_t pe;          // position + 1 of the last kept entry before the lane's (0: none in the chunk)
    uint32_t start;       // bit of the chunk's bit string that the lane's codes start at
};

// Bits of the chunk's codes without the first entry's; first (0xFFFFFFFF: none) and last_end (position
// + 1 of the last): the same in the whole wavefront.
__device__ __forceinline__ ChunkCodes chunk_codes(const uint4& words, int b, uint32_t& inner_bits, uint32_t& first, uint32_t& last_end) {
    ChunkCodes c;
    c.words = words;
    c.p0 = (threadIdx.x & 63u) * 128u;
    uint32_t bits = 0u, mine = 0xFFFFFFFFu;
    c.pe = wave_excl_max(last_bit_end(words, c.p0), &last_end);
    uint32_t pe = c.pe;
    for_bits(words, c.p0, [&](uint32_t x) {
        if (pe) bits += golomb_len(x - pe, b);
        else mine = x;                                 // the only entry of the chunk without predecessor
        pe = x + 1u;
    });
    const uint32_t inc = wave_incl_sum(bits);
    c.start = inc - bits;
    inner_bits = last_lane(inc);
    const unsigned long long has = __ballot(mine != 0xFFFFFFFFu);
    first = (uint32_t)__builtin_amdgcn_readlane((int)mine, has ? __ffsll((long long)has) - 1 : 0);
    return c;
}

// nb bits (1 to 32) of val at bit pos of a bit string of which `to` (zeroed) holds words [w0, w0 + n).
__device__ __forceinline__ void put_bits(uint32_t* to, uint32_t w0, uint32_t n, uint32_t pos, uint32_t val, uint32_t nb) {
    const uint32_t w = (pos >> 5) - w0;
    const unsigned long long v = (unsigned long long)val << (64u - (pos & 31u) - nb);
    if (w < n) atomicOr(&to[w], (uint32_t)(v >> 32));
    if ((uint32_t)v && w + 1u < n) atomicOr(&to[w + 1u], (uint32_t)v);
}

// One code, of gap `gap`, at bit pos, which moves on.
__device__ __forceinline__ void put_code(uint32_t* to, uint32_t w0, uint32_t n, uint32_t& pos, uint32_t gap, int b) {
    const uint32_t rem = gap & ((1u << b) - 1u);
    uint32_t q = gap >> b;
    while (q + (uint32_t)b + 1u > 32u) {               // a long unary run, 16 ones at a time
        const uint32_t take = min(q, 16u);
        put_bits(to, w0, n, pos, (1u << take) - 1u, take);
        pos += take;
        q -= take;
    }
    put_bits(to, w0, n, pos, (((1u << q) - 1u) << (b + 1)) | rem, q + (uint32_t)b + 1u);
    pos += q + (uint32_t)b + 1u;
}

// The chunk's bit string, which fits kChunkWords words.
__device__ __forceinline__ void write_codes(const ChunkCodes& c, int b, uint32_t* to) {
    uint32_t pe = c.pe, pos = c.start;
    for_bits(c.words, c.p0, [&](uint32_t x) {
        if (pe) put_code(to, 0u, (uint32_t)kChunkWords, pos, x - pe, b);
        pe = x + 1u;
    });
}

// A chunk so crowded that its bit string does not fit its words: its bitmap as a word per lane in four rounds,
// so that no lane has more than 32 codes of a stretch (8192 kept entries at b = 6, 1800 words: k_emit_scan 25 us;
// 60 with 128 codes of a lane in each of seven stretches of 256 words.  k_emit_all has stretches of 256 words, for with 512
// or 1024 it takes as long: 2000 kept entries in one of 25 chunks 55 us, threshold, apply and emit by themselves 45).
constexpr int kRawRounds = kChunkWords / 64;
struct RawCodes {
    uint32_t word[kRawRounds], pe[kRawRounds], start[kRawRounds];      // the lane's: bits, end of the entry before, first bit of the codes
    uint32_t end[kRawRounds];                                          // the round's codes end there
};
__device__ __forceinline__ RawCodes raw_codes(const uint32_t* __restrict__ bitmap, int b) {
    const uint32_t lane = threadIdx.x & 63u;
    RawCodes c;
    uint32_t ended = 0u, bits_before = 0u;
#pragma unroll
    for (int r = 0; r < kRawRounds; ++r) c.word[r] = bitmap[r * 64 + lane];
#pragma unroll
    for (int r = 0; r < kRawRounds; ++r) {
        const uint32_t p0 = ((uint32_t)r * 64u + lane) * 32u;
        uint32_t round_end, bits = 0u;
        c.pe[r] = wave_excl_max(c.word[r] ? p0 + 32u - (uint32_t)__clz((int)c.word[r]) : 0u, &round_end);
        if (c.pe[r] == 0u) c.pe[r] = ended;
        uint32_t pe = c.pe[r];
        for (uint32_t m = c.word[r]; m; m &= m - 1u) {
            const uint32_t x = p0 + (uint32_t)__ffs((int)m) - 1u;
            if (pe) bits += golomb_len(x - pe, b);
            pe = x + 1u;
        }
        const uint32_t inc = wave_incl_sum(bits);
        c.start[r] = bits_before + inc - bits;
        bits_before += last_lane(inc);
        c.end[r] = bits_before;
        if (round_end) ended = round_end;
    }
    return c;
}
// The words [w0, w0 + n) of the bit string.
__device__ __forceinline__ void write_raw(const RawCodes& c, int b, uint32_t* to, uint32_t w0, uint32_t n) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (int r = 0; r < kRawRounds; ++r) {
        if (c.end[r] <= 32u * w0 || (r ? c.end[r - 1] : 0u) >= 32u * (w0 + n)) continue;     // uniform
        uint32_t pe = c.pe[r], pos = c.start[r];
        for (uint32_t m = c.word[r]; m && pos < 32u * (w0 + n); m &= m - 1u) {
            const uint32_t x = ((uint32_t)r * 64u + lane) * 32u + (uint32_t)__ffs((int)m) - 1u;
            if (pe) put_code(to, w0, n, pos, x - pe, b);
            pe = x + 1u;
        }
    }
}

// The first 32 bits of the bit string of such a chunk: few of its codes, all of them the first lanes'.
__device__ __forceinline__ void write_head(const ChunkCodes& c, int b, uint32_t* to) {
    uint32_t pe = c.pe, pos = c.start;
    if (pos >= 32u) return;
    unsigned long long m = ((unsigned long long)c.words.y << 32) | c.words.x, rest = ((unsigned long long)c.words.w << 32) | c.words.z;
    for (uint32_t p0 = c.p0; (m || rest) && pos < 32u; m &= m - 1ull) {
        if (!m) { m = rest; rest = 0ull; p0 += 64u; }
        const uint32_t x = p0 + (uint32_t)(__ffsll((long long)m) - 1);
        if (pe) put_code(to, 0u, 1u, pos, x - pe, b);
        pe = x + 1u;
    }
}

// 32 bits from bit x on of a chunk's codes: the first entry's (gap >> b ones, a zero, b bits), then the
// bit string, whose words are rest(i) (zero beyond its end).
template <typename F>
__device__ __forceinline__ uint32_t chunk_bits(uint32_t x, uint32_t gap, int b, F rest) {
    const uint32_t q = gap >> b, lead = q + 1u + (uint32_t)b;
    if (x >= lead) {
        const uint32_t y = x - lead;
        return (uint32_t)(((((unsigned long long)rest(y >> 5) << 32) | rest((y >> 5) + 1u)) << (y & 31u)) >> 32);
    }
    const uint32_t ones = x < q ? min(q - x, 32u) : 0u, left = lead - x;          // (left >= 1)
    const unsigned long long rem = gap & ((1u << b) - 1u);
    uint32_t v = ones ? 0xFFFFFFFFu << (32u - ones) : 0u;
    if (left <= 32u) v |= (uint32_t)(rem << (32u - left));
    else if (left < 64u) v |= (uint32_t)(rem >> (left - 32u));
    if (left < 32u) v |= rest(0u) >> left;
    return v;
}

// A chunk's codes from its bitmap in bm (LDS): the bit string in code (zeroed), or, if it does not fit that (raw), its
// first word there and the bitmap in bm as it was.  `bits` of the codes without the first entry's, that entry's
// position, the last one's position + 1 (0: no entries): the same in the whole wavefront.
struct ChunkDone { uint32_t bits, first, end; bool raw; uint4 words; };
constexpr uint32_t kFewKept = 2u * kChunkWords;        // (positions of 16 bits in the bitmap's place)
__device__ __forceinline__ ChunkDone encode_chunk(uint32_t* bm, uint32_t* code, int b) {
    const uint32_t lane = threadIdx.x & 63u;
    ChunkDone d;
    d.words = reinterpret_cast<const uint4*>(bm)[lane];
    const uint32_t own = (uint32_t)(__popc(d.words.x) + __popc(d.words.y) + __popc(d.words.z) + __popc(d.words.w));
    const uint32_t upto = wave_incl_sum(own), kept = last_lane(upto);
    if (kept > kFewKept) {                             // uniform
        const ChunkCodes c = chunk_codes(d.words, b, d.bits, d.first, d.end);
        d.raw = d.bits > 32u * (uint32_t)kChunkWords;
        if (d.raw) write_head(c, b, code);
        else write_codes(c, b, code);
        wave_lds_fence();
        return d;
    }
    uint16_t* const pos = reinterpret_cast<uint16_t*>(bm);
    wave_lds_fence();
    uint32_t at = upto - own;
    for_bits(d.words, lane * 128u, [&](uint32_t x) { pos[at++] = (uint16_t)x; });
    wave_lds_fence();
    d.bits = 0u; d.first = 0xFFFFFFFFu; d.end = 0u;
    for (uint32_t r0 = 0u; r0 < kept; r0 += 64u) {     // a code per lane
        const uint32_t r = r0 + lane;
        const bool in = r < kept;
        const uint32_t x = in ? pos[r] : 0u, before = in && r ? pos[r - 1u] + 1u : 0u;
        const uint32_t len = in && r ? golomb_len(x - before, b) : 0u;
        const uint32_t inc = wave_incl_sum(len);
        uint32_t to = d.bits + inc - len;
        if (len) put_code(code, 0u, (uint32_t)kChunkWords, to, x - before, b);
        d.bits += last_lane(inc);
        if (r0 == 0u) d.first = uniform(x);
        d.end = (uint32_t)__builtin_amdgcn_readlane((int)x, (int)min(kept - r0 - 1u, 63u)) + 1u;
    }
    d.raw = d.bits > 32u * (uint32_t)kChunkWords;
    if (__builtin_expect(d.raw, 0)) reinterpret_cast<uint4*>(bm)[lane] = d.words;
    wave_lds_fence();
    return d;
}

// --------------------------------------------------------------------------
// Side, residual update and codes.  Bound by three dependent round trips to memory and, where a chunk
// has hundreds of candidates, by the instructions for those and the scattered stores of the residual: 5.9
// us on 25.6e6 entries at p = 0.001 (3243 chunks), 12.3 us at p = 0.01, 4.3 us on 512 chunks; 88 us on 1.5e9
// entries (106 when it stored a bitmap of 1 KB per chunk, which the next kernel read, instead of the codes).
// --------------------------------------------------------------------------
// PAIRS: see k_threshold.
template <bool PAIRS>
__global__ __launch_bounds__(kEncThreads) void k_apply(
        const TensorDesc* __restrict__ desc, const uint2* __restrict__ chunk_tensor, const ChunkRun* __restrict__ runs,
        const TensorState* __restrict__ st, TensorState* res, const CandPtr cand,
        uint64_t cand_entries, uint32_t* __restrict__ codes, ChunkSummary* __restrict__ sum,
        uint32_t* __restrict__ heads, int b, int pass, uint32_t n_chunks, ResultBlock* __restrict__ result) {
    __shared__ __attribute__((aligned(16))) uint32_t bits_sh[kEncWaves][kChunkWords];
    __shared__ __attribute__((aligned(16))) uint32_t code_sh[kEncWaves][kChunkWords];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t c = blockIdx.x * (uint32_t)kEncWaves + (uint32_t)wave;
    if (c >= n_chunks) return;
    uint32_t* const bm = bits_sh[wave];
    const uint2 ct = chunk_tensor[c];                  // (tensor, its first chunk)
    const ChunkRun run = runs[c];
    const uint32_t t = ct.x, cc = c - ct.y;
    // the first entries of both sides' runs (usually all of them) are on their way before it is known
    // which side is wanted.  (The run of a tensor that was finished elsewhere, or whose lists overflowed,
    // may be anything: such a tensor is passed over below.)
    uint2 e0[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        e0[s] = make_uint2(0u, 0u);
        if (!PAIRS && (uint32_t)lane < run.cnt[s] && run.at[s] < cand_entries - 64u) e0[s] = cand.get(run.at[s] + (uint32_t)lane);
    }
    reinterpret_cast<uint4*>(bm)[lane] = make_uint4(0u, 0u, 0u, 0u);
    reinterpret_cast<uint4*>(code_sh[wave])[lane] = make_uint4(0u, 0u, 0u, 0u);
    const uint32_t n = desc[t].n;
    const gfloat_ptr R = as_global(desc[t].R);
    const uint32_t flags = st[t].flags;
    const double mean_p = st[t].mean[0], mean_n = st[t].mean[1];
    const uint32_t tau_p = st[t].tau[0], tau_n = st[t].tau[1], itau_p = st[t].itau[0], itau_n = st[t].itau[1];
    if (!encoded_in_pass(flags, pass)) {
        // (its error bit stops the call; cannot be missing: what is encoded below would be another call's)
        if (pass == kPassAll && lane == 0 && !(__hip_atomic_load(&result->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrStops))
            atomicOr(&result->err, kErrInternal);
        return;
    }
    // Alg. 2 compares the means (sums that differ may still give equal means: the positive side then)
    const int chosen = mean_p >= mean_n ? 0 : 1;
    const float mu32 = (float)(chosen ? mean_n : mean_p);
    const float mu_signed = chosen ? -mu32 : mu32;
    const uint32_t tau = chosen ? tau_n : tau_p, itau = chosen ? itau_n : itau_p;
    if (cc == 0u && lane == 0) {
        const uint32_t nnz = st[t].kc[chosen];
        res[t].side = chosen ? -1 : 1; res[t].mu_signed = mu_signed; res[t].nnz = nnz;
        if (nnz > desc[t].kcap) atomicOr(&result->err, kErrInternal);          // (cannot happen)
    }
    const CandPtr list = cand + run.at[chosen];
    const uint32_t cnt = run.cnt[chosen];
    const uint64_t off = desc[t].cand_off;
    const uint2* const pair = pairs_of(cand, off, chosen) + (run.at[chosen] - off - (chosen ? desc[t].cand_cap : 0u));
    const auto entry = [&](uint32_t i) { return PAIRS && (flags & kStDeferred) ? pair[i] : list.get(i); };
    wave_lds_fence();
    bool bad = false;
    auto keep = [&](const uint2& e) {
        if (!cand_kept(e.x, e.y, tau, itau)) return;
        if (e.y >= n || e.y / (uint32_t)kChunk != cc) { bad = true; return; }        // (cannot happen)
        const float a = __uint_as_float(bits_of_key(chosen ? ~e.x : e.x));
        R[e.y] = a - mu_signed;                        // Alg. 1: R <- dW - dW*
        atomicOr(&bm[(e.y % (uint32_t)kChunk) >> 5], 1u << (e.y & 31u));
    };
    // (at the very end of the array the first entries were not read ahead)
    const bool ahead = !PAIRS && run.at[chosen] < cand_entries - 64u;
    if (ahead && (uint32_t)lane < cnt) keep(chosen ? e0[1] : e0[0]);
    for (uint32_t i0 = ahead ? 64u : 0u; i0 < cnt; i0 += 256u) {
        uint2 e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t i = i0 + 64u * u + (uint32_t)lane;
            e[u] = entry(i < cnt ? i : 0u);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + 64u * u + (uint32_t)lane < cnt) keep(e[u]);
    }
    if (bad) atomicOr(&result->err, kErrInternal);
    wave_lds_fence();
    // (a chunk crowded with kept entries: the bitmap goes out instead, and of the codes only the first word)
    const ChunkDone done = encode_chunk(bm, code_sh[wave], b);
    uint4* const out = reinterpret_cast<uint4*>(codes + (uint64_t)c * kChunkWords) + lane;
    if (done.raw) *out = done.words;
    else if ((uint32_t)lane * 128u < done.bits) *out = reinterpret_cast<const uint4*>(code_sh[wave])[lane];
    if (lane == 0) {
        if (done.raw) heads[c] = code_sh[wave][0];
        sum[c] = make_summary(done.bits, done.first, done.end, done.raw, cc == 0u);
    }
}

constexpr int kScanThreads = 1024;
constexpr int kScanPer = 4;              // consecutive chunks per thread
constexpr uint32_t kScanTile = kScanThreads * kScanPer;   // chunks per workgroup of the scan

// What a tile of kScanTile consecutive chunks of a tensor contributes to the scan over all of
// the tensor's chunks.  The code of the tile's first kept entry depends on where the previous
// kept entry lies, which the tile does not know: its bits are left out and its position kept.
struct TileSummary {
    uint32_t end;              // position + 1 of the last kept entry in the tile (0: none)
    uint32_t first;            // position of the first one (if there is one)
    unsigned long long bits;   // code bits of all of them but the first
};

// Tiles of tensor t live at tiles[chunk0 / kScanTile + t ...]: tensors never overlap there
// (floor((a + n) / T) + 1 >= floor(a / T) + ceil(n / T)).
__device__ __forceinline__ uint32_t tile_base(const TensorDesc& d, int t) { return d.chunk0 / kScanTile + (uint32_t)t; }

// One tile's share of the scan, given what precedes the tile: the gap before each chunk's first
// kept entry, bit offset of each chunk.  WRITE = false only adds up the tile (first pass of a
// tensor of several tiles, carries unknown: pe == 0 marks the tile's first kept entry).
template <bool WRITE>
__device__ __forceinline__ void scan_tile(const TensorDesc& d, uint32_t tile, const ChunkSummary* __restrict__ sum,
                                          uint32_t carry_end, unsigned long long carry_bits, int b,
                                          uint32_t* __restrict__ chunk_gap, uint64_t* __restrict__ chunk_bitoff,
                                          uint32_t* scratch32, unsigned long long* scratch64,
                                          uint32_t& tile_end, unsigned long long& tile_bits,
                                          uint32_t& first_pos, bool& has_first) {
    const int tid = threadIdx.x;
    const uint32_t c0 = tile * kScanTile + (uint32_t)tid * kScanPer;
    ChunkSummary s[kScanPer];
    uint32_t gend[kScanPer], my_end = 0u;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        s[j].x = 0u; s[j].y = 0u;
        if (c0 + j < d.nchunks) s[j] = sum[d.chunk0 + c0 + j];
        gend[j] = sum_any(s[j]) ? (c0 + j) * (uint32_t)kChunk + sum_end(s[j]) : 0u;
        if (gend[j] > my_end) my_end = gend[j];
    }
    uint32_t pe = block_excl_max<uint32_t, kScanThreads>(my_end, &tile_end, scratch32);
    if (carry_end > pe) pe = carry_end;
    // gap before every chunk's first kept entry, and the chunk's code bits
    uint32_t gaps[kScanPer];
    unsigned long long bits[kScanPer], my_bits = 0ull;
    has_first = false; first_pos = 0u;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        gaps[j] = 0u;
        bits[j] = 0ull;
        if (sum_any(s[j])) {
            const uint32_t pos = (c0 + j) * (uint32_t)kChunk + sum_first(s[j]);
            bits[j] = (unsigned long long)sum_inner(s[j]);
            if (!WRITE && pe == 0u) { has_first = true; first_pos = pos; }      // (a kept entry's end is at least 1)
            else bits[j] += (unsigned long long)golomb_len(pos - pe, b);
            gaps[j] = pos - pe;
            pe = gend[j];
        }
        my_bits += bits[j];
    }
    unsigned long long off = carry_bits + block_excl_sum<unsigned long long, kScanThreads>(my_bits, &tile_bits, scratch64);
    if (WRITE) {
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            if (c0 + j < d.nchunks) {
                chunk_gap[d.chunk0 + c0 + j] = gaps[j];
                chunk_bitoff[d.chunk0 + c0 + j] = off;
            }
            off += bits[j];
        }
    }
}

// grid (T, tiles): first pass over a tensor of several tiles (tensors of one tile need none)
__global__ __launch_bounds__(kScanThreads) void k_tile_summary(const TensorDesc* __restrict__ desc,
                                                               const TensorState* __restrict__ st,
                                                               const ChunkSummary* __restrict__ sum,
                                                               TileSummary* __restrict__ tiles, int b, int pass) {
    __shared__ uint32_t scratch32[kScanThreads / 64];
    __shared__ unsigned long long scratch64[kScanThreads / 64];
    const int t = blockIdx.x, tid = threadIdx.x;
    const TensorDesc d = desc[t];
    if (!encoded_in_pass(st[t].flags, pass)) return;
    const uint32_t n_tiles = (d.nchunks + kScanTile - 1u) / kScanTile;
    if (n_tiles < 2u || blockIdx.y >= n_tiles) return;
    uint32_t tile_end, first_pos;
    unsigned long long tile_bits;
    bool has_first;
    scan_tile<false>(d, blockIdx.y, sum, 0u, 0ull, b, nullptr, nullptr, scratch32, scratch64, tile_end, tile_bits, first_pos, has_first);
    TileSummary* const out = tiles + tile_base(d, t) + blockIdx.y;
    if (has_first) out->first = first_pos;              // exactly one thread of a tile that holds entries
    if (tid == 0) { out->end = tile_end; out->bits = tile_bits; }
}

// grid (T, tiles): per tensor, scan over its chunks: every tile folds the summaries of the
// tiles before it, then scans its own chunks.
__global__ __launch_bounds__(kScanThreads) void k_tensor_scan(const TensorDesc* __restrict__ desc,
                                                              const ChunkSummary* __restrict__ sum,
                                                              const TileSummary* __restrict__ tiles,
                                                              uint32_t* __restrict__ chunk_gap,
                                                              uint64_t* __restrict__ chunk_bitoff,
                                                              TensorState* __restrict__ st, int b, int pass,
                                                              ResultBlock* __restrict__ result) {
    __shared__ uint32_t scratch32[kScanThreads / 64];
    __shared__ unsigned long long scratch64[kScanThreads / 64];
    const int t = blockIdx.x, tid = threadIdx.x;
    const TensorDesc d = desc[t];
    if (!encoded_in_pass(st[t].flags, pass)) return;
    const uint32_t n_tiles = (d.nchunks + kScanTile - 1u) / kScanTile;
    if (blockIdx.y >= n_tiles) return;
    uint32_t carry_end = 0u;                            // position+1 of the last kept entry so far (0: none)
    unsigned long long carry_bits = 0ull;
    const TileSummary* __restrict__ ts = tiles + tile_base(d, t);
    for (uint32_t j = 0; j < blockIdx.y; ++j) {         // (every thread: the same few loads)
        const TileSummary s = ts[j];
        if (s.end) {
            carry_bits += s.bits + (unsigned long long)golomb_len(s.first - carry_end, b);
            carry_end = s.end;                           // positions grow from tile to tile
        }
    }
    uint32_t tile_end, first_pos;
    unsigned long long tile_bits;
    bool has_first;
    scan_tile<true>(d, blockIdx.y, sum, carry_end, carry_bits, b, chunk_gap, chunk_bitoff, scratch32, scratch64,
                    tile_end, tile_bits, first_pos, has_first);
    if (tid == 0 && blockIdx.y == n_tiles - 1u) {
        const unsigned long long bit_len = carry_bits + tile_bits;
        st[t].bit_len = bit_len;
        // (cannot happen; said here, for k_emit sends the call's result before the streams are written)
        if (((bit_len + 31ull) >> 5) > d.bound_words) atomicOr(&result->err, kErrInternal);
    }
}

// ------------------------------------------------------------ the payload ----

// The chunk of the calling wavefront: its place in its tensor's stream (bit offset `at`, from a word
// boundary of `to` on), the gap before its first kept entry, and its bit string or bitmap in `win`.
struct ChunkStream {
    uint32_t c, gap, inner;
    bool any, raw;
    unsigned long long at;
};
// Words of LDS per wavefront for W words of a chunk's bit string (and zeros behind them).
template <uint32_t W>
constexpr uint32_t kWindow = W + 4u;

// The words of the stream that start in the chunk.  win: the bit string's words, zeros behind them (raw:
// anything).  after(f, gap, any): chunk f of the same tensor, or false if there is none.
template <uint32_t W, typename After>
__device__ __forceinline__ void write_chunk(const ChunkStream& s, int b, uint32_t* win, const ChunkSummary* __restrict__ sum,
                                            const uint32_t* __restrict__ codes, const uint32_t* __restrict__ heads,
                                            uint32_t* __restrict__ to, After after) {
    const uint32_t lane = threadIdx.x & 63u;
    if (!s.any) return;
    const uint32_t lead = golomb_len(s.gap, b), bits = lead + s.inner;
    const unsigned long long first = (s.at + 31ull) >> 5, end = (s.at + bits + 31ull) >> 5;
    RawCodes rc;
    if (__builtin_expect(s.raw, 0)) rc = raw_codes(codes + (uint64_t)s.c * kChunkWords, b);
    for (uint32_t i0 = 0u; ; i0 += W) {
        // the words that need the bit string's words i0 .. i0 + W (all, unless the chunk is raw)
        unsigned long long lo = first, hi = end;
        if (__builtin_expect(s.raw, 0)) {
            wave_lds_fence();
            for (uint32_t i = lane; i < kWindow<W>; i += 64u) win[i] = 0u;
            wave_lds_fence();
            write_raw(rc, b, win, i0, W + 1u);
            wave_lds_fence();
            const unsigned long long from = s.at + lead + 31ull;
            if (i0) lo = (from + 32ull * i0) >> 5;
            hi = min(hi, (from + 32ull * (i0 + W)) >> 5);
        }
        for (unsigned long long w = lo + lane; w < hi; w += 64u) {
            const uint32_t x = (uint32_t)(32ull * w - s.at);
            uint32_t v = chunk_bits(x, s.gap, b, [&](uint32_t i) { return win[i - i0]; });
            if (bits - x < 32u) {
                // the chunk ends in this word: the first bits of the chunks behind it
                uint32_t have = bits - x;
                for (uint32_t f = s.c + 1u; have < 32u; ++f) {
                    uint32_t gap;
                    bool any;
                    if (!after(f, gap, any)) break;
                    if (!any) continue;
                    const ChunkSummary fs = sum[f];
                    const uint32_t inner = sum_inner(fs);
                    const uint32_t head = !inner ? 0u : sum_raw(fs) ? heads[f] : codes[(uint64_t)f * kChunkWords];
                    v |= chunk_bits(0u, gap, b, [&](uint32_t) { return head; }) >> have;
                    have += min(golomb_len(gap, b), 32u) + min(inner, 32u);
                }
            }
            to[w] = v;
        }
        if (!s.raw || 32u * (i0 + W) >= s.inner) break;
    }
}

// The chunk's bit string, for write_chunk: asked for early (bits beyond it are zero in memory up to a
// multiple of four words), put into LDS when it has arrived.
__device__ __forceinline__ uint4 load_codes(const uint32_t* __restrict__ codes, uint32_t c, const ChunkSummary& s) {
    const uint32_t lane = threadIdx.x & 63u;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (lane * 128u < sum_inner(s)) v = reinterpret_cast<const uint4*>(codes + (uint64_t)c * kChunkWords)[lane];
    return v;
}
__device__ __forceinline__ void stage_codes(uint32_t* win, const uint4& v) {
    const uint32_t lane = threadIdx.x & 63u;
    reinterpret_cast<uint4*>(win)[lane] = v;
    if (lane == 0u) *reinterpret_cast<uint4*>(win + kChunkWords) = make_uint4(0u, 0u, 0u, 0u);
    wave_lds_fence();
}

// A tensor's table entry, and its state left clean for the next call.
__device__ __forceinline__ void finish_tensor(uint8_t* __restrict__ msg, TensorState* __restrict__ st,
                                              unsigned long long* __restrict__ counters, uint32_t t, float mu_signed, uint32_t nnz,
                                              unsigned long long bit_len, unsigned long long word_off) {
    uint8_t* e = msg + 32 + 24ull * t;
    *reinterpret_cast<float*>(e) = mu_signed;
    *reinterpret_cast<uint32_t*>(e + 4) = nnz;
    *reinterpret_cast<uint64_t*>(e + 8) = bit_len;
    *reinterpret_cast<uint64_t*>(e + 16) = word_off;
    st[t].bit_len = bit_len;
    st[t].cand_cnt[0] = 0u; st[t].cand_cnt[1] = 0u; st[t].flags = 0u; st[t].done = 0u; st[t].sorted_kept = 0u;
#pragma unroll
    for (uint32_t g = 0; g < kSegs; ++g) counters[((size_t)t * kSegs + g) * kCounterStride] = 0ull;
}
// The header, and the call's result for the host.
__device__ __forceinline__ void finish_call(uint8_t* __restrict__ msg, int T, int b, unsigned long long payload_words, uint32_t err,
                                            ResultBlock* __restrict__ next_result,
                                            unsigned long long* __restrict__ host_word, uint32_t seq) {
    const unsigned long long bytes = 32ull + 24ull * (unsigned)T + 4ull * payload_words;
    publish(host_word, seq, err, bytes);
    uint32_t* h = reinterpret_cast<uint32_t*>(msg);
    h[0] = 0x31434253u; h[1] = 1u; h[2] = (uint32_t)T; h[3] = (uint32_t)b;
    *reinterpret_cast<uint64_t*>(msg + 16) = payload_words;
    *reinterpret_cast<uint64_t*>(msg + 24) = 0ull;
    // the result block of the next call starts out clean
    next_result->err = 0u;
}

// --------------------------------------------------------------------------
// From the candidate lists to the message in one launch (k_emit_all), for calls of up to kEmitAllChunks chunks
// in up to kEmitAllTensors tensors.  The first 2 T workgroups each select one side of a tensor; the others take up to sixteen chunks
// each, a wavefront per chunk, and go through k_apply's work and the message's words.  They do not end between these steps but wait
// for what they need of one another's results, which go through memory as words that carry the call's number
// (StepFlow): every wait is for such a word to carry it.  A launch costs 2 us from the last workgroup of the one before
// to its first, and its first loads a round trip; a wait costs 0.9 to 1.4 us, and what a workgroup loads is there by then.
// Whole steps in us, threshold, apply and emit as three launches / in one: 328,000 entries in four tensors 40.9 / 36.6,
// one tensor of 2^20 35.2 / 31.8, 24 ragged tensors of 12e6 65.8 / 61.5, ResNet-50 shape (3243 chunks) at p = 0.001 83.3
// / 82.6, at p = 0.01, where the chunks of other tensors are done while the longest list is selected, 103.0 / 96.1.
// Beyond that the workgroups that wait get into the others' way: one tensor of 3500 chunks at p = 1e-4 86 / 86, of 3750
// 90 / 93, eight tensors of 3500 chunks 85 / 85, of 4000 93 / 96, 8060 chunks 162 / 171.  The chip holds 512 workgroups of
// this size; where sides take nearly all of these places, those with chunks start late: 200 tensors of 1000 chunks 42 / 42, 240
// 43 / 44, 512 47 / 49, 255 tensors of 300 chunks 30 / 32, 4000 of 4000 entries 157 / 168.  Nor does it pay where a chunk keeps
// more than kFewKept entries, for the workgroups that wait have only their first 256 candidates of either side at
// hand, and the residual's stores come last: one tensor of 4.2e6 entries at p = 0.05 57 / 57, 0.07 63 / 66, 0.2 93 / 110.
// --------------------------------------------------------------------------
constexpr uint32_t kEmitAllChunks = 3584, kEmitAllTensors = 200;
constexpr int kEmitThreads = kThThreads;
// Calls of up to so many chunks have eight per workgroup, else sixteen: what a workgroup looks at of all lower ones grows
// with their number (one tensor of 512 chunks, step: four each 39.1 us, eight 38.0, sixteen 37.6; 128 chunks 32.2, 31.8, 32.2).
constexpr uint32_t kEmitFew = 256;
constexpr uint32_t kEmitGroups = kEmitAllChunks / 16;                  // most workgroups that take chunks
static_assert(kEmitGroups <= kEmitThreads && kEmitFew / 8 <= kEmitGroups, "one workgroup's summary per thread");

// Where a launch's workgroups leave results for one another (agent-scope atomics, which are performed in memory: plain
// loads and stores of different compute-unit groups do not see one another within a kernel).  A word counts
// once its upper bits carry the call's number; the host clears all of them whenever the sixteen bits start over.
constexpr uint32_t kSideWords = 8;       // per tensor and side, values of 32 bits
enum SideWord { kSideTau = 0, kSideItau, kSideMeanLo, kSideMeanHi, kSideKept, kSideRaise, kSideUsed };
constexpr uint32_t kGroupWords = 4;      // per workgroup that takes chunks, values of 48 bits
constexpr uint32_t kTagMask = 0xFFFFu;
struct StepFlow {
    unsigned long long* groups;          // kGroupWords each: the first ones of all, then the second ones and so on (what one
                                         // workgroup looks at lies on few memory lines)
    unsigned long long* sides;           // kSideWords each
    uint32_t* started;                   // workgroups of all launches that have got on with selecting a side, and, behind
                                         // it, that have taken chunks
    uint32_t sides_before, taken;        // ... of the launches before this one
    uint32_t tag;                        // the call's number, 1 to 0xFFFF
};
__device__ __forceinline__ unsigned long long flow_load(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void flow_store(unsigned long long* p, unsigned long long v, uint32_t tag) {
    __hip_atomic_store(p, v | ((unsigned long long)tag << 48), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool flow_has(unsigned long long v, uint32_t tag) { return (uint32_t)(v >> 48) == tag; }

// What stops a call, and what the host is told of it, as a workgroup's summary carries it.
constexpr uint32_t kFlowStop = 1u, kFlowLoose = 2u, kFlowWide = 4u, kFlowLong = 8u, kFlowInternal = 16u, kFlowLeft = 32u;
__device__ __forceinline__ uint32_t flow_bits(uint32_t err) {
    return (err & kErrStops ? kFlowStop : 0u) | (err & kErrLoose ? kFlowLoose : 0u) | (err & kErrWide ? kFlowWide : 0u) |
           (err & kErrLong ? kFlowLong : 0u) | (err & kErrInternal ? kFlowInternal : 0u);
}
__device__ __forceinline__ uint32_t flow_err(uint32_t bits) {
    return (bits & kFlowLoose ? kErrLoose : 0u) | (bits & kFlowWide ? kErrWide : 0u) | (bits & kFlowLong ? kErrLong : 0u) |
           (bits & kFlowInternal ? kErrInternal : 0u) | (bits & kFlowLeft ? kErrDeferred : 0u);
}

// A stretch of the call's codes: bits before the first tensor that starts in it, words of the tensors that start
// and end in it, bits since the last start (or, if none starts, all its bits), and the last 32 of those, the
// last one in bit 0.  Stretches are put together from left to right; all zero is the empty one.
struct Stretch {
    uint32_t head, words, bits, tail;    // (words: and kStarts if a tensor starts)
};
constexpr uint32_t kStarts = 0x80000000u;
__device__ __forceinline__ Stretch joined(const Stretch& f, const Stretch& g) {
    const bool fs = f.words & kStarts, gs = g.words & kStarts;
    const uint32_t over = f.bits + (gs ? g.head : g.bits);             // what ends f and continues in g
    Stretch r;
    r.head = fs ? f.head : over;
    r.bits = gs ? g.bits : over;
    r.words = (f.words + (gs ? (g.words & ~kStarts) + (fs ? (over + 31u) >> 5 : 0u) : 0u)) | (g.words & kStarts);
    r.tail = gs || g.bits >= 32u ? g.tail : (f.tail << g.bits) | g.tail;
    return r;
}
// Inclusive over a row of 16 lanes, or (ROW = false) over the wavefront.
template <bool ROW>
__device__ __forceinline__ Stretch join_lanes(Stretch v) {
    auto step = [&](auto fetch) {
        Stretch f;
        f.head = fetch(v.head); f.words = fetch(v.words); f.bits = fetch(v.bits); f.tail = fetch(v.tail);
        v = joined(f, v);
    };
    step([](uint32_t x) { return dpp_fetch<0x111, 0xf>(x); });
    step([](uint32_t x) { return dpp_fetch<0x112, 0xf>(x); });
    step([](uint32_t x) { return dpp_fetch<0x114, 0xf>(x); });
    step([](uint32_t x) { return dpp_fetch<0x118, 0xf>(x); });
    if constexpr (!ROW) {
        step([](uint32_t x) { return dpp_fetch<0x142, 0xa>(x); });
        step([](uint32_t x) { return dpp_fetch<0x143, 0xc>(x); });
    }
    return v;
}
__device__ __forceinline__ Stretch stretch_of_lane(const Stretch& v, uint32_t lane) {
    Stretch r;
    r.head = (uint32_t)__builtin_amdgcn_readlane((int)v.head, (int)lane); r.words = (uint32_t)__builtin_amdgcn_readlane((int)v.words, (int)lane);
    r.bits = (uint32_t)__builtin_amdgcn_readlane((int)v.bits, (int)lane); r.tail = (uint32_t)__builtin_amdgcn_readlane((int)v.tail, (int)lane);
    return r;
}
// One code, and `inner` bits behind it of which `tail` holds the last 32.
__device__ __forceinline__ Stretch code_stretch(uint32_t gap, int b, uint32_t inner, uint32_t tail) {
    const uint32_t q = min(gap >> b, 32u), rem = gap & ((1u << b) - 1u);
    const uint32_t code = (uint32_t)((((1ull << q) - 1ull) << (b + 1)) | rem);        // (its last 32 bits)
    Stretch s;
    s.head = 0u; s.words = 0u;
    s.bits = golomb_len(gap, b) + inner;
    s.tail = inner >= 32u ? tail : (code << inner) | tail;
    return s;
}

// A chunk's part of a workgroup's summary, in LDS.
struct ChunkPart {
    uint32_t first, end, inner, tail;    // (positions in the chunk; end: 0 if there are no kept entries)
    uint32_t starts;
};

// ... and where its codes go, from all chunks before it.
struct ChunkPlace {
    uint32_t word_off, at, before, gap;  // its tensor's first word in the payload, bits of that stream before the chunk, the last of them
};

// The words that end in the chunk, and, if it is its tensor's last, the one that the tensor ends in.  before: the
// stream's last bits before the chunk, the last one in bit 0.  win: the bit string's words, zeros behind them
// (raw: anything); bitmap: in LDS.
template <uint32_t W>
__device__ __forceinline__ void write_words(const ChunkStream& s, uint32_t at, uint32_t before, bool ends, int b, uint32_t* win,
                                            const uint32_t* bitmap, uint32_t* __restrict__ to) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t lead = s.any ? golomb_len(s.gap, b) : 0u, bits = lead + s.inner;
    const uint32_t first = at >> 5, end = (at + bits + (ends ? 31u : 0u)) >> 5;
    RawCodes rc;
    if (__builtin_expect(s.raw, 0)) rc = raw_codes(bitmap, b);
    for (uint32_t i0 = 0u; ; i0 += W) {
        // the words that need the bit string's words i0 .. i0 + W (all, unless the chunk is raw)
        uint32_t lo = first, hi = end;
        if (__builtin_expect(s.raw, 0)) {
            wave_lds_fence();
            for (uint32_t i = lane; i < kWindow<W>; i += 64u) win[i] = 0u;
            wave_lds_fence();
            write_raw(rc, b, win, i0, W + 1u);
            wave_lds_fence();
            const uint32_t from = at + lead + 31u;
            if (i0) lo = (from + 32u * i0) >> 5;
            hi = min(hi, (from + 32u * (i0 + W)) >> 5);
        }
        for (uint32_t w = lo + lane; w < hi; w += 64u) {
            const uint32_t x = 32u * w - at;           // (first word: less than zero by the bits before the chunk)
            const bool shared = 32u * w < at;
            uint32_t v = s.any ? chunk_bits(shared ? 0u : x, s.gap, b, [&](uint32_t i) { return win[i - i0]; }) : 0u;
            if (shared) v = (before << (32u + x)) | (v >> (0u - x));
            to[w] = v;
        }
        if (!s.raw || 32u * (i0 + W) >= s.inner) break;
    }
}

struct StepSweeps { const WideState* ws; uint32_t* hist; const long long* acc; int on; };
struct StepChunks { const uint2* chunk_tensor; const ChunkRun* runs; uint32_t* codes; ChunkSummary* sum; uint32_t* heads; uint64_t cand_entries; };
struct StepSizes { int T, b; uint32_t n_chunks; int carry; uint32_t looks; };

// Looks at a missing word (a microsecond each at the most) before a workgroup gives up on sides that nobody has
// started to select, and before it takes a missing word for an invariant violated (seconds).
constexpr uint32_t kFlowLooks = 4096, kFlowMostLooks = 1u << 22;

// --------------------------------------------------------------------------
// Waits end: chunks are handed out by a counter, in order, to the workgroups as they start, each of which waits
// for lower chunks alone, that is, for workgroups that are running.  (That is why a word of the payload is written by
// the chunk that its last bit belongs to, with the last bits of the chunks before it, and not as in k_emit.)
// The sides' workgroups wait for nobody; they come first in the launch, but where others fill the compute units, those of
// other launches of this kernel among them, some may not have started: a workgroup waits for those a while
// and then leaves the call to the kernels of the second pass (kErrDeferred).
// --------------------------------------------------------------------------
template <uint32_t CPW>
__global__ __launch_bounds__(kEmitThreads, 8) void k_emit_all(
        const TensorDesc* __restrict__ desc, const uint32_t* __restrict__ order, TensorState* __restrict__ st,
        unsigned long long* __restrict__ counters, const CandPtr cand, const StepSweeps sweeps, const StepChunks chunks, const StepFlow flow,
        const StepSizes sizes, uint8_t* __restrict__ msg, uint64_t msg_capacity, ResultBlock* __restrict__ result, ResultBlock* __restrict__ next_result,
        unsigned long long* __restrict__ host_word, uint32_t seq) {
    constexpr uint32_t NW = kEmitThreads / 64, W = kChunkWords;
    static_assert(CPW <= NW && CPW <= 16, "a wavefront per chunk, a row of lanes");
    struct Chunks {
        __attribute__((aligned(16))) uint32_t bits[CPW][kChunkWords];
        __attribute__((aligned(16))) uint32_t code[CPW][kWindow<W>];
    };
    __shared__ __attribute__((aligned(16))) union { ThresholdShared select; Chunks chunk; } sh;
    __shared__ uint32_t side_sh[CPW][2 * kSideWords];
    __shared__ ChunkPart part_sh[CPW];
    __shared__ ChunkPlace place_sh[CPW];
    __shared__ Stretch wave_sh[NW];
    __shared__ uint32_t ends_sh[NW], next_item, flags_sh;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = uniform((uint32_t)tid >> 6);
    const int T = sizes.T, b = sizes.b;
    const uint32_t n_chunks = sizes.n_chunks, tag = flow.tag, n_sides = 2u * (uint32_t)T;
    SBC_TS(0, 0);
    if (blockIdx.x < n_sides) {                        // uniform
        select_side<false>(sh.select, blockIdx.x, desc, order, st, counters, cand, chunks.codes, sweeps.ws, sweeps.hist, sweeps.acc, 0, sweeps.on,
                           sizes.carry, result, [&]() { atomicAdd(flow.started, 1u); }, [&](int t, int s, const SideResult& r) {
            unsigned long long* const to = flow.sides + ((size_t)t * 2u + (uint32_t)s) * kSideWords;
            const unsigned long long mean = (unsigned long long)__double_as_longlong(r.mean);
            if (r.raise || !r.ok) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // (the error word has them before anybody can see this)
            flow_store(to + kSideTau, r.tau, tag); flow_store(to + kSideItau, r.itau, tag);
            flow_store(to + kSideMeanLo, (uint32_t)mean, tag); flow_store(to + kSideMeanHi, mean >> 32, tag);
            flow_store(to + kSideKept, r.ok ? r.kc : 0u, tag); flow_store(to + kSideRaise, flow_bits(r.raise), tag);
        });
        return;
    }
    // (1 us that there is to wait anyway: the sides' workgroups have the memory to themselves for their first loads.  With
    // 500 workgroups that take chunks those took 5.4 us, 1.3 so.)
    // (of the kernels before this one; sides of this one may have raised theirs there already.  A round trip to memory,
    // which the sides' workgroups would wait for: 1 us.)
    const uint32_t err_in = __hip_atomic_load(&result->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_sleep(32);
    if (tid == 0) { next_item = atomicAdd(flow.started + 1, 1u) - flow.taken; flags_sh = 0u; }
    __syncthreads();
    const uint32_t a = uniform(next_item), c = a * CPW + wave;
    if (a >= gridDim.x - n_sides) {                    // uniform; cannot happen (the host's count of launches is wrong)
        if (tid == 0) atomicOr(&result->err, kErrInternal);
        return;
    }
    const bool mine = wave < CPW && c < n_chunks;
    uint2 ct = make_uint2(0u, 0u);
    ChunkRun run;
    run.at[0] = run.at[1] = 0ull; run.cnt[0] = run.cnt[1] = 0u;
    constexpr int AHEAD = 4;                           // 64 entries each of both sides that are loaded before the side is known
    uint2 e[2][AHEAD];
    uint32_t n = 0u, nchunks = 0u, kcap = 0u;
    float* residual = nullptr;
    if (mine) {
        ct = chunks.chunk_tensor[c];
        run = chunks.runs[c];
        ct.x = uniform(ct.x); ct.y = uniform(ct.y);
        // (the run of a tensor whose lists overflowed may be anything: such a tensor is passed over below)
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const uint32_t i = 64u * (uint32_t)u + (uint32_t)lane;
                e[s][u] = make_uint2(0u, 0u);
                if (i < run.cnt[s] && run.at[s] + i < chunks.cand_entries) e[s][u] = cand.get(run.at[s] + i);
            }
        n = desc[ct.x].n; nchunks = desc[ct.x].nchunks; kcap = desc[ct.x].kcap; residual = desc[ct.x].R;
        reinterpret_cast<uint4*>(sh.chunk.bits[wave])[lane] = make_uint4(0u, 0u, 0u, 0u);
        reinterpret_cast<uint4*>(sh.chunk.code[wave])[lane] = make_uint4(0u, 0u, 0u, 0u);
        if (lane == 0) *reinterpret_cast<uint4*>(sh.chunk.code[wave] + kChunkWords) = make_uint4(0u, 0u, 0u, 0u);
    }
    const uint32_t cc = c - ct.y;
    SBC_TS(0, 1);
    if (mine && (wave == 0u || cc == 0u)) {            // a wavefront for all its tensor's in the workgroup
        const unsigned long long* const from = flow.sides + (size_t)ct.x * 2u * kSideWords;
        const bool wanted = lane < (int)(2u * kSideWords) && (uint32_t)lane % kSideWords < kSideUsed;
        unsigned long long v = 0ull;
        for (uint32_t look = 1u;; ++look) {
            if (wanted) v = flow_load(from + lane);
            if (!__any(wanted && !flow_has(v, tag))) break;
            const bool late = look % sizes.looks == 0u && __hip_atomic_load(flow.started, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - flow.sides_before < n_sides;
            if (late || look == kFlowMostLooks) {      // uniform
                v = 0ull;                              // (kept entries: none)
                if (lane == 0) atomicOr(&flags_sh, kFlowStop | (late ? kFlowLeft : kFlowInternal));
                break;
            }
            __builtin_amdgcn_s_sleep(4);
        }
        if (lane < (int)(2u * kSideWords)) side_sh[wave][lane] = (uint32_t)v;
    }
    SBC_TS(0, 2);
    __syncthreads();
    SBC_TS(0, 3);

    // ---- side and codes of the chunk (as k_apply) ----
    ChunkStream cs;
    cs.c = c; cs.gap = 0u; cs.inner = 0u; cs.any = false; cs.raw = false; cs.at = 0ull;
    float mu_signed = 0.f;
    uint32_t nnz = 0u, tau = 0u, itau = 0u, cnt = 0u;
    int chosen = 0;
    CandPtr list = cand;
    bool usable = false;
    // f(entry) for the chunk's kept entries
    auto for_kept = [&](auto f) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u)
            if (64u * (uint32_t)u < cnt)               // uniform
                if (64u * (uint32_t)u + (uint32_t)lane < cnt && cand_kept(e[0][u].x, e[0][u].y, tau, itau)) f(e[0][u]);
#pragma nounroll
        for (uint32_t i0 = 64u * AHEAD; i0 < cnt; i0 += 256u) {
            uint2 x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t i = i0 + 64u * u + (uint32_t)lane;
                x[u] = list.get(i < cnt ? i : 0u);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + 64u * u + (uint32_t)lane < cnt && cand_kept(x[u].x, x[u].y, tau, itau)) f(x[u]);
        }
    };
    uint32_t* const bm = sh.chunk.bits[min(wave, CPW - 1u)];
    uint32_t* const code = sh.chunk.code[min(wave, CPW - 1u)];
    if (mine) {
        const uint32_t* const v = side_sh[cc < wave ? wave - cc : 0u];
        const uint32_t kept_p = uniform(v[kSideKept]), kept_n = uniform(v[kSideWords + kSideKept]);
        const double mean_p = __longlong_as_double((long long)(((unsigned long long)uniform(v[kSideMeanHi]) << 32) | uniform(v[kSideMeanLo])));
        const double mean_n = __longlong_as_double((long long)(((unsigned long long)uniform(v[kSideWords + kSideMeanHi]) << 32) | uniform(v[kSideWords + kSideMeanLo])));
        uint32_t flags = uniform(v[kSideRaise]) | uniform(v[kSideWords + kSideRaise]);
        // Alg. 2 compares the means (sums that differ may still give equal means: the positive side then)
        chosen = mean_p >= mean_n ? 0 : 1;
        const float mu32 = (float)(chosen ? mean_n : mean_p);
        mu_signed = chosen ? -mu32 : mu32;
        tau = uniform(v[(chosen ? kSideWords : 0u) + kSideTau]); itau = uniform(v[(chosen ? kSideWords : 0u) + kSideItau]);
        nnz = chosen ? kept_n : kept_p;
        ChunkPart part;
        part.first = part.end = part.inner = part.tail = 0u;
        part.starts = cc == 0u ? 1u : 0u;
        usable = kept_p != 0u && kept_n != 0u;
        if (!usable) {
            flags |= kFlowStop;                        // the lists cannot be used: the call's second pass takes the tensor
        } else {
            list = cand + run.at[chosen];
            cnt = uniform(run.cnt[chosen]);
            if (chosen) {                              // uniform
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) e[0][u] = e[1][u];
            }
            wave_lds_fence();
            bool bad = false;
            const uint32_t entries = min(n - cc * (uint32_t)kChunk, (uint32_t)kChunk);
            for_kept([&](const uint2& x) {
                const uint32_t at = x.y - cc * (uint32_t)kChunk;
                bad = bad || at >= entries;            // (cannot happen)
                atomicOr(&bm[(at >> 5) % (uint32_t)kChunkWords], 1u << (at & 31u));
            });
            if (__any(bad) || nnz > kcap) {            // (cannot happen)
                if (lane == 0) atomicOr(&result->err, kErrInternal);
                flags |= kFlowStop | kFlowInternal;
                usable = false;
            }
            wave_lds_fence();
            const ChunkDone done = encode_chunk(bm, code, b);
            cs.inner = done.bits; cs.any = done.end != 0u; cs.raw = done.raw;
            part.first = done.first & (uint32_t)(kChunk - 1); part.end = done.end;
            part.inner = cs.inner;
            // (for the second pass, and for sbc_last_mask)
            uint4* const out = reinterpret_cast<uint4*>(chunks.codes + (uint64_t)c * kChunkWords) + lane;
            if (cs.raw) *out = done.words;
            else if ((uint32_t)lane * 128u < cs.inner) *out = reinterpret_cast<const uint4*>(code)[lane];
            if (lane == 0 && cs.raw) chunks.heads[c] = code[0];
            uint32_t from = cs.inner < 32u ? 0u : cs.inner - 32u;      // the last 32 bits of the bit string
            const uint32_t shift = from & 31u;
            from >>= 5;
            if (__builtin_expect(cs.raw, 0)) {
                const RawCodes rc = raw_codes(bm, b);
                wave_lds_fence();
                if (lane < 2) code[lane] = 0u;
                wave_lds_fence();
                write_raw(rc, b, code, from, 2u);
                wave_lds_fence();
                from = 0u;
            }
            const uint32_t last32 = (uint32_t)(((((unsigned long long)uniform(code[from]) << 32) | uniform(code[from + 1u])) << shift) >> 32);
            part.tail = cs.inner >= 32u ? last32 : cs.inner ? last32 >> (32u - cs.inner) : 0u;
        }
        if (lane == 0) {
            part_sh[wave] = part;
            if (flags) atomicOr(&flags_sh, flags);
            chunks.sum[c] = make_summary(cs.inner, part.first, part.end, cs.raw, cc == 0u);
        }
    } else if (wave < CPW && lane == 0) {
        part_sh[wave] = ChunkPart{0u, 0u, 0u, 0u, 0u};
    }
    __syncthreads();
    SBC_TS(0, 4);

    // ---- the workgroup's chunks together: the first wavefront, a lane per chunk (positions + 1, 0: none) ----
    ChunkPart own = {0u, 0u, 0u, 0u, 0u};
    Stretch piece = {0u, 0u, 0u, 0u};
    uint32_t own_gap = 0u, open_lane = 0xFFFFFFFFu, open_first = 0u;
    if (wave == 0u) {
        const uint32_t chunk_at = (uint32_t)lane * (uint32_t)kChunk;
        if (lane < (int)CPW) own = part_sh[lane];
        uint32_t ended = own.end ? chunk_at + own.end + 1u : own.starts ? chunk_at + 1u : 0u;
        ended = max(ended, dpp_fetch<0x111, 0xf>(ended));
        ended = max(ended, dpp_fetch<0x112, 0xf>(ended));
        ended = max(ended, dpp_fetch<0x114, 0xf>(ended));
        ended = max(ended, dpp_fetch<0x118, 0xf>(ended));
        uint32_t before_own = dpp_fetch<0x111, 0xf>(ended);            // (of all lanes)
        if (own.starts) before_own = chunk_at + 1u;
        const bool open = own.end && before_own == 0u; // the kept entry before its first one lies before the workgroup's chunks
        own_gap = chunk_at + own.first + 1u - before_own;              // (open: position + 1 of the first)
        piece.bits = own.inner; piece.tail = own.tail;
        if (own.end && !open) piece = code_stretch(own_gap, b, own.inner, own.tail);
        if (own.starts) piece.words = kStarts;
        piece = join_lanes<true>(piece);
        const unsigned long long open_at = __ballot(open);
        if (open_at) {                                 // uniform
            open_lane = (uint32_t)__ffsll((long long)open_at) - 1u;
            open_first = (uint32_t)__builtin_amdgcn_readlane((int)own_gap, (int)open_lane);
        }
        if (lane == (int)CPW - 1) {
            // (18 bits for positions + 1 in up to 16 chunks, 24 for their bits, 18 for their words)
            const uint32_t words = piece.words & ~kStarts;
            unsigned long long* const to = flow.groups + a;
            flow_store(to, ended | ((unsigned long long)open_first << 18) | ((unsigned long long)(piece.words >> 31) << 36) | ((unsigned long long)(flags_sh & 63u) << 37), tag);
            flow_store(to + kEmitGroups, piece.bits | ((unsigned long long)piece.head << 24), tag);
            flow_store(to + 2u * kEmitGroups, piece.tail | ((unsigned long long)(words & 0x3FFu) << 32), tag);
            flow_store(to + 3u * kEmitGroups, words >> 10, tag);
        }
    }
    SBC_TS(0, 5);

    // ---- what lies before them: a lane per workgroup of lower chunks ----
    Stretch lower = {0u, 0u, 0u, 0u};
    uint32_t lower_end = 0u, lower_open = 0u;          // positions in the call's chunks + 1
    if ((uint32_t)tid < a) {
        const unsigned long long* const from = flow.groups + tid;
        unsigned long long v0, v1, v2, v3;
        bool missing = false;
        for (uint32_t look = 0u;;) {
            v0 = flow_load(from); v1 = flow_load(from + kEmitGroups); v2 = flow_load(from + 2u * kEmitGroups); v3 = flow_load(from + 3u * kEmitGroups);
            if (flow_has(v0, tag) && flow_has(v1, tag) && flow_has(v2, tag) && flow_has(v3, tag)) break;
            if (++look == kFlowMostLooks) { missing = true; break; }   // cannot happen
            __builtin_amdgcn_s_sleep(4);
        }
        const uint32_t at = (uint32_t)tid * CPW * (uint32_t)kChunk;
        lower_end = (uint32_t)v0 & 0x3FFFFu;
        if (lower_end) lower_end += at;
        lower_open = (uint32_t)(v0 >> 18) & 0x3FFFFu;
        if (lower_open) lower_open += at;
        lower.words = ((v0 >> 36) & 1ull ? kStarts : 0u) | ((uint32_t)(v2 >> 32) & 0x3FFu) | (((uint32_t)v3 & 0xFFu) << 10);
        lower.bits = (uint32_t)v1 & 0xFFFFFFu; lower.head = (uint32_t)(v1 >> 24) & 0xFFFFFFu;
        lower.tail = (uint32_t)v2;
        uint32_t flags = (uint32_t)(v0 >> 37) & 63u;
        if (missing) { atomicOr(&result->err, kErrInternal); flags = kFlowStop | kFlowInternal; }
        if (flags) atomicOr(&flags_sh, flags);
    }
    SBC_TS(0, 6);
    // (up to 64 of them are the first wavefront's)
    const uint32_t end_inc = wave_incl_max(lower_end);
    uint32_t end_before = dpp_fetch<0x138, 0xf>(end_inc), end_in = last_lane(end_inc);     // end_in: where the last kept entry before the
    if (a > 64u) {                                     // uniform                          // workgroup's chunks ends, or its tensor starts
        if (lane == 63) ends_sh[wave] = end_inc;
        __syncthreads();
        const uint32_t ends = lane < (int)NW ? ends_sh[lane] : 0u;     // (ascending, but for zeros)
        end_before = max(end_before, last_lane(wave_incl_max(lane < (int)wave ? ends : 0u)));
        end_in = last_lane(wave_incl_max(ends));
    }
    if (lower_open) lower = joined(code_stretch(lower_open - end_before, b, 0u, 0u), lower);
    if ((wave << 6) < max(a, 1u)) lower = join_lanes<false>(lower);    // uniform
    if (a > 64u) {                                     // uniform
        if (lane == 63) wave_sh[wave] = lower;
        __syncthreads();
        lower = Stretch{0u, 0u, 0u, 0u};
        if (lane < (int)NW) lower = wave_sh[lane];
    }
    if (wave == 0u) {
        wave_lds_fence();                              // (flags_sh, which lanes of this wavefront have raised)
        const Stretch all = a > 64u ? stretch_of_lane(join_lanes<true>(lower), NW - 1u) : stretch_of_lane(lower, 63u);
        // (positions + 1 here and there)
        const uint32_t open_gap = open_first + a * CPW * (uint32_t)kChunk - end_in;
        const Stretch lead = (uint32_t)lane > open_lane ? code_stretch(open_gap, b, 0u, 0u) : Stretch{0u, 0u, 0u, 0u};
        Stretch mine_before;
        mine_before.head = dpp_fetch<0x111, 0xf>(piece.head); mine_before.words = dpp_fetch<0x111, 0xf>(piece.words);
        mine_before.bits = dpp_fetch<0x111, 0xf>(piece.bits); mine_before.tail = dpp_fetch<0x111, 0xf>(piece.tail);
        const Stretch start = joined(joined(all, lead), mine_before);
        ChunkPlace p;
        p.word_off = start.words & ~kStarts; p.at = start.bits; p.before = start.tail;
        if (own.starts) { p.word_off += (p.at + 31u) >> 5; p.at = 0u; p.before = 0u; }
        p.gap = (uint32_t)lane == open_lane ? open_gap : own_gap;
        const uint32_t last = n_chunks - 1u - a * CPW; // the call's last chunk, if it is the workgroup's
        if (lane < (int)CPW) {
            place_sh[lane] = p;
            if ((uint32_t)lane == last) {
                const uint32_t bits = p.at + (own.end ? golomb_len(p.gap, b) + own.inner : 0u);
                const unsigned long long payload_words = (unsigned long long)p.word_off + ((bits + 31u) >> 5);
                uint32_t flags = flags_sh | flow_bits(err_in);
                if (32ull + 24ull * (unsigned)T + 4ull * payload_words > msg_capacity) {       // (cannot happen)
                    flags |= kFlowStop | kFlowInternal;
                    atomicOr(&flags_sh, flags);
                    atomicOr(&result->err, kErrInternal);
                }
                if (flags & (kFlowStop | kFlowInternal)) {
                    // tensors have to be redone, or the call fails: the error word has all of it
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    const uint32_t err = __hip_atomic_load(&result->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) | flow_err(flags);
                    publish(host_word, seq, err & kErrStops ? err : err | kErrInternal, 0ull);
                } else {
                    finish_call(msg, T, b, payload_words, err_in | flow_err(flags), next_result, host_word, seq);
                }
            }
        }
    }
    __syncthreads();
    SBC_TS(0, 7);
    if (!mine) return;
    const ChunkPlace place = place_sh[wave];
    const uint32_t at = uniform(place.at), word_off = uniform(place.word_off);
    cs.gap = uniform(place.gap);
    const uint32_t flags = uniform(flags_sh) | flow_bits(err_in);
    const uint32_t bit_end = at + (cs.any ? golomb_len(cs.gap, b) + cs.inner : 0u);
    const bool fits = 32ull + 24ull * (unsigned)T + 4ull * (word_off + ((bit_end + 31ull) >> 5)) <= msg_capacity;    // (always)
    if (!(flags & (kFlowStop | kFlowInternal)) && fits) {
        const bool ends = cc == nchunks - 1u;
        if (ends && lane == 0) finish_tensor(msg, st, counters, ct.x, mu_signed, nnz, bit_end, word_off);
        write_words<W>(cs, at, uniform(place.before), ends, b, code, bm, reinterpret_cast<uint32_t*>(msg + 32 + 24ull * (unsigned)T) + word_off);
    }
    // ---- Alg. 1: R <- dW - dW* (last: scattered stores, which nobody waits for in this kernel) ----
    if (usable) {
        if (cc == 0u && lane == 0) { st[ct.x].side = chosen ? -1 : 1; st[ct.x].mu_signed = mu_signed; st[ct.x].nnz = nnz; }
        const gfloat_ptr R = as_global(residual);
        for_kept([&](const uint2& x) { R[x.y] = __uint_as_float(bits_of_key(chosen ? ~x.x : x.x)) - mu_signed; });
    }
    SBC_TS(0, 8);
}

// Exclusive prefix sum / maximum over a workgroup with one barrier; scratch: 16 words used by this scan alone.
// (the wavefronts' values lie in the first lanes: two or four steps scan them)
template <int NW, bool MAX>
__device__ __forceinline__ uint32_t scan_block(uint32_t v, uint32_t& total, uint32_t* scratch) {
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t inc = MAX ? wave_incl_max(v) : wave_incl_sum(v);
    if (lane == 63) scratch[w] = inc;
    __syncthreads();
    uint32_t waves = lane < NW ? scratch[lane] : 0u;
    auto step = [&](uint32_t o) { waves = MAX ? max(waves, o) : waves + o; };
    step(dpp_fetch<0x111, 0xf>(waves));
    step(dpp_fetch<0x112, 0xf>(waves));
    if constexpr (NW > 4) {
        step(dpp_fetch<0x114, 0xf>(waves));
        step(dpp_fetch<0x118, 0xf>(waves));
    }
    static_assert(NW <= 16, "a row of lanes");
    total = (uint32_t)__builtin_amdgcn_readlane((int)waves, NW - 1);
    const uint32_t before = w ? (uint32_t)__builtin_amdgcn_readlane((int)waves, w - 1) : 0u;
    if constexpr (MAX) return max(before, dpp_fetch<0x138, 0xf>(inc));         // (the lane before; 0 for lane 0)
    else return before + inc - v;
}

// --------------------------------------------------------------------------
// The message behind k_apply, for calls of up to kScanAllChunks chunks that k_emit_all does not take or has left to
// the second pass: a wavefront per chunk.  NT threads, at most kScanAllPer chunks each in the scan, which every workgroup
// repeats: that is cheaper than a launch for it (1.6 us and its own round trips), up to 4096 chunks: 6.4 us
// on the 3243 chunks of the ResNet-50 shape, 4.9 on 512, 4.3 on 41 (11, 9 and 9 us for codes into staging
// words and a copy from there into the message); with 8060 chunks, eight per thread, 22 us, where
// k_tensor_scan and k_emit take 4.8 and 5.9.  Workgroups of 256 threads for few chunks, for the scans over
// sixteen wavefronts cost more than what they scan there.
// --------------------------------------------------------------------------
constexpr int kScanAllPer = 4;
constexpr uint32_t kScanAllChunks = 1024 * kScanAllPer;
static_assert(kEmitAllChunks <= kScanAllChunks, "whatever k_emit_all leaves");
constexpr uint32_t kScanFew = 256 * kScanAllPer;       // calls of up to so many chunks take workgroups of 256 threads
template <int NT>
__global__ __launch_bounds__(NT) void k_emit_scan(
        const uint2* __restrict__ chunk_tensor, const ChunkSummary* __restrict__ sum, const uint32_t* __restrict__ codes,
        const uint32_t* __restrict__ heads, TensorState* __restrict__ st, unsigned long long* __restrict__ counters, int T, int b, uint32_t n_chunks,
        uint8_t* __restrict__ msg, uint64_t msg_capacity, ResultBlock* __restrict__ result, ResultBlock* __restrict__ next_result,
        unsigned long long* __restrict__ host_word, uint32_t seq) {
    constexpr int NW = NT / 64, PER = kScanAllPer;
    __shared__ uint32_t scratch[4][16];
    constexpr uint32_t W = NT <= 256 ? 1024u : 256u;   // (words of a crowded chunk put together at a time)
    __shared__ __attribute__((aligned(16))) uint32_t win_sh[NW][kWindow<W>];
    extern __shared__ uint32_t offs[];                 // every chunk's bit offset in the payload, then the gaps
    uint32_t* const gaps = offs + n_chunks;
    constexpr uint32_t kNone = 0x80000000u, kStarts = 0x40000000u;     // (gaps are below 2^26 here)
    static_assert((uint64_t)kScanAllChunks * kChunk <= 1u << 26, "positions and offsets in 32 bits");
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t c = blockIdx.x * (uint32_t)NW + (uint32_t)wave;
    const uint32_t per = (n_chunks + NT - 1u) / NT, c0 = (uint32_t)tid * per;
    const uint32_t err_in = result->err;
    ChunkSummary s[PER], own = make_uint2(0u, 0u);
    uint2 ct = make_uint2(0u, 0u);
    if (c < n_chunks) { own = sum[c]; ct = chunk_tensor[c]; }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        s[j] = make_uint2(0u, 0u);
        if ((uint32_t)j < per && c0 + (uint32_t)j < n_chunks) s[j] = sum[c0 + (uint32_t)j];
    }
    if (err_in & kErrStops) {                          // uniform: tensors have to be redone, or the call fails
        if (blockIdx.x == 0 && tid == 0) publish(host_word, seq, err_in, 0ull);
        return;
    }
    const uint4 mine = load_codes(codes, c, own);
    const float mu_signed = st[ct.x].mu_signed;
    const uint32_t nnz = st[ct.x].nnz;
    // what precedes the thread's chunks: the end of the last kept entry, or the start of the tensor (positions in
    // the call-wide numbering of chunks)
    uint32_t end = 0u, all;                            // (all: first the scan's unused total, then the bits of all chunks)
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t base = (c0 + (uint32_t)j) * (uint32_t)kChunk;
        if (sum_starts(s[j])) end = base;
        if (sum_any(s[j])) end = base + sum_end(s[j]);
    }
    end = scan_block<NW, true>(end, all, scratch[0]);
    uint32_t gap[PER], len[PER], bits = 0u;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t base = (c0 + (uint32_t)j) * (uint32_t)kChunk;
        if (sum_starts(s[j])) end = base;
        gap[j] = base + sum_first(s[j]) - end;
        len[j] = sum_any(s[j]) ? golomb_len(gap[j], b) + sum_inner(s[j]) : 0u;
        bits += len[j];
        if (sum_any(s[j])) end = base + sum_end(s[j]);
    }
    uint32_t at = scan_block<NW, false>(bits, all, scratch[1]);
    uint32_t payload_words = (all + 31u) >> 5, shift = 0u;     // shift: of the tensor the thread's first chunk belongs to,
                                                               // from the bits of all chunks one after another
    if (T > 1) {                                       // uniform: every tensor starts on a word
        // where, among those bits, the tensor that a chunk belongs to starts
        uint32_t origin = 0u, last_origin, x = at;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (sum_starts(s[j])) origin = x;
            x += len[j];
        }
        origin = scan_block<NW, true>(origin, last_origin, scratch[2]);
        // words of the tensors before that one (a tensor's are counted where the next one starts)
        uint32_t words = 0u, from = origin;
        x = at;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (sum_starts(s[j])) { words += (x - from + 31u) >> 5; from = x; }
            x += len[j];
        }
        const uint32_t before = scan_block<NW, false>(words, payload_words, scratch[3]);
        payload_words += (all - last_origin + 31u) >> 5;
        shift = 32u * before - origin;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t cj = c0 + (uint32_t)j;
        if ((uint32_t)j < per && cj < n_chunks) {
            if (sum_starts(s[j])) shift = ((at + shift + 31u) & ~31u) - at;    // (a word boundary behind the tensor before)
            offs[cj] = at + shift;
            gaps[cj] = (sum_any(s[j]) ? gap[j] : kNone) | (sum_starts(s[j]) ? kStarts : 0u);
            at += len[j];
        }
    }
    uint32_t err = err_in;
    if (32ull + 24ull * (unsigned)T + 4ull * payload_words > msg_capacity) err |= kErrInternal;      // (cannot happen)
    if (blockIdx.x == 0 && tid == 0) {
        if (err & kErrInternal) publish(host_word, seq, err, 0ull);
        else finish_call(msg, T, b, payload_words, err, next_result, host_word, seq);
    }
    if (err & kErrInternal) return;                    // uniform
    stage_codes(win_sh[wave], mine);
    __syncthreads();
    if (c >= n_chunks) return;
    const uint32_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)gaps[c]), o = (uint32_t)__builtin_amdgcn_readfirstlane((int)offs[c]);
    ChunkStream cs;
    cs.c = c; cs.gap = g & (kStarts - 1u); cs.inner = sum_inner(own); cs.any = !(g & kNone); cs.raw = sum_raw(own); cs.at = o;
    if ((tid & 63) == 0 && (c + 1u == n_chunks || (gaps[c + 1u] & kStarts))) {
        const uint32_t tensor = offs[ct.y];
        finish_tensor(msg, st, counters, ct.x, mu_signed, nnz, (unsigned long long)(o - tensor) + (cs.any ? golomb_len(cs.gap, b) + cs.inner : 0u), tensor >> 5);
    }
    write_chunk<W>(cs, b, win_sh[wave], sum, codes, heads, reinterpret_cast<uint32_t*>(msg + 32 + 24ull * (unsigned)T),
                [&](uint32_t f, uint32_t& gap_f, bool& any_f) {
                    if (f >= n_chunks) return false;
                    const uint32_t gf = gaps[f];
                    gap_f = gf & (kStarts - 1u);
                    any_f = !(gf & kNone);
                    return !(gf & kStarts);
                });
}

// --------------------------------------------------------------------------
// The same behind k_tensor_scan, a wavefront per chunk.  DIRECT: into the message; else into the tensor's
// staging words, for k_finish_message.
// --------------------------------------------------------------------------
template <bool DIRECT>
__global__ __launch_bounds__(kEncThreads) void k_emit(
        const TensorDesc* __restrict__ desc, const uint2* __restrict__ chunk_tensor, const ChunkSummary* __restrict__ sum,
        const uint32_t* __restrict__ codes, const uint32_t* __restrict__ heads, const uint32_t* __restrict__ chunk_gap,
        const uint64_t* __restrict__ chunk_bitoff, TensorState* __restrict__ st, unsigned long long* __restrict__ counters,
        int T, int b, int pass, uint32_t n_chunks,
        uint32_t* __restrict__ stage, uint8_t* __restrict__ msg, uint64_t msg_capacity, ResultBlock* __restrict__ result,
        ResultBlock* __restrict__ next_result, unsigned long long* __restrict__ host_word, uint32_t seq) {
    constexpr uint32_t W = 512u;
    __shared__ __attribute__((aligned(16))) uint32_t win_sh[kEncWaves][kWindow<W>];
    const uint32_t lane = threadIdx.x & 63u;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t c = blockIdx.x * (uint32_t)kEncWaves + (uint32_t)wave;
    if (c >= n_chunks) return;
    const uint2 ct = chunk_tensor[c];                  // (tensor, its first chunk)
    const ChunkSummary own = sum[c];
    const uint32_t t = ct.x, gap = chunk_gap[c];
    const unsigned long long at = chunk_bitoff[c];
    const uint4 mine = load_codes(codes, c, own);
    const uint32_t err_in = DIRECT ? result->err : 0u;
    const uint32_t nchunks = desc[t].nchunks;
    const unsigned long long bit_len = st[t].bit_len, n_words = (bit_len + 31ull) >> 5;
    uint32_t* to;
    if constexpr (DIRECT) {
        if (err_in & kErrStops) {                      // uniform: tensors have to be redone, or the call fails
            if (c == 0u && lane == 0u) publish(host_word, seq, err_in, 0ull);
            return;
        }
        // the streams before this tensor's (all of them, for the chunk that writes the header)
        unsigned long long before = 0ull, all = 0ull;
        for (uint32_t i = lane; i < (c == 0u ? (uint32_t)T : t); i += 64u) {
            const unsigned long long w = (st[i].bit_len + 31ull) >> 5;
            all += w;
            if (i < t) before += w;
        }
        before = last_lane(wave_incl_sum(before));
        all = last_lane(wave_incl_sum(all));
        // (a stream beyond its bound cannot happen, k_tensor_scan has looked; nor can all of them together be too
        // long for the message then: the first chunk says so, the others write nothing)
        const unsigned long long most = (msg_capacity - 32ull - 24ull * (unsigned)T) >> 2;
        const bool fits = (c == 0u ? all : before + n_words) <= most;
        if (c == 0u && lane == 0u) {
            if (fits) finish_call(msg, T, b, all, err_in, next_result, host_word, seq);
            else publish(host_word, seq, err_in | kErrInternal, 0ull);
        }
        if (!fits) return;
        if (c - ct.y == nchunks - 1u && lane == 0u) finish_tensor(msg, st, counters, t, st[t].mu_signed, st[t].nnz, bit_len, before);
        to = reinterpret_cast<uint32_t*>(msg + 32 + 24ull * (unsigned)T) + before;
    } else {
        if (!encoded_in_pass(st[t].flags, pass)) return;
        if (n_words > desc[t].bound_words) return;     // would leave the tensor's staging words (cannot happen: k_tensor_scan)
        to = stage + desc[t].stage_off;
    }
    stage_codes(win_sh[wave], mine);
    ChunkStream cs;
    cs.c = c; cs.gap = gap; cs.inner = sum_inner(own); cs.any = sum_any(own); cs.raw = sum_raw(own); cs.at = at;
    const uint32_t last = ct.y + nchunks;
    write_chunk<W>(cs, b, win_sh[wave], sum, codes, heads, to, [&](uint32_t f, uint32_t& gap_f, bool& any_f) {
        if (f >= last) return false;
        gap_f = chunk_gap[f];
        any_f = sum_any(sum[f]);
        return true;
    });
}

}  // namespace sbc
