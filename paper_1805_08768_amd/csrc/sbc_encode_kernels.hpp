// The rest of the client step once the thresholds are known, a wavefront per chunk of 8192 entries:
//   k_apply    : Alg. 2's side decision, Alg. 1's residual line and Alg. 3 within the chunk, from the
//                chunk's run of candidates: the codes of all its kept entries but the first, whose
//                predecessor lies in another chunk, as a bit string of its own, and a summary
//   k_emit_all : the message in one launch: every workgroup scans the summaries of the call's chunks
//                (predecessors, bit offsets, the tensors' places in the payload), then every wavefront
//                puts its chunk's first code and bit string together, shifted to their place
//   k_tile_summary, k_tensor_scan, k_emit : the same in steps for calls of very many chunks (the scan
//                over a tensor's chunks in tiles of 4096), and for calls whose other tensors the streaming
//                kernel has finished (the streams then go to the tensors' staging words and the message
//                is assembled by k_finish_message)
//
// Candidates of one chunk sit next to each other in their tensor's lists (a workgroup of the
// streaming kernel appends them as one run), so the chunk is the unit of work here and no kept
// position is ever sorted: a bitmap, in LDS, puts a chunk's in order, and chunks are in order.
//
// A word of the payload is written once, whole, by the chunk that its first bit belongs to, which adds
// the first bits of the chunks behind it: nothing has to be cleared beforehand, no word is shared
// through atomics and nothing is copied afterwards.
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
// Does a pass of k_apply / k_emit work on a tensor with these state flags?
__device__ __forceinline__ bool encoded_in_pass(uint32_t flags, int pass) {
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
// so that no lane has more than 32 codes of a stretch (8192 kept entries at b = 6, 1800 words: k_emit_all 25 us;
// 60 with 128 codes of a lane in each of seven stretches of 256 words).
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
    if (!encoded_in_pass(flags, pass)) return;
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
    uint32_t inner_bits, first, last_end;
    const ChunkCodes codes_of = chunk_codes(reinterpret_cast<const uint4*>(bm)[lane], b, inner_bits, first, last_end);
    // a chunk crowded with kept entries: the bitmap goes out instead, and of the codes only the first word
    const bool raw = inner_bits > 32u * (uint32_t)kChunkWords;
    if (__builtin_expect(raw, 0)) write_head(codes_of, b, code_sh[wave]);
    else write_codes(codes_of, b, code_sh[wave]);
    wave_lds_fence();
    uint4* const out = reinterpret_cast<uint4*>(codes + (uint64_t)c * kChunkWords) + lane;
    if (raw) *out = codes_of.words;
    else if ((uint32_t)lane * 128u < inner_bits) *out = reinterpret_cast<const uint4*>(code_sh[wave])[lane];
    if (lane == 0) {
        if (raw) heads[c] = code_sh[wave][0];
        sum[c] = make_summary(inner_bits, first, last_end, raw, cc == 0u);
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

// Most chunks of a call whose workgroups scan the summaries of all chunks themselves (8 bytes each), and
// how many of them a thread takes; calls of up to kEmitFew chunks take workgroups of 256 threads.
constexpr int kEmitAllPer = 4;
constexpr uint32_t kEmitAllChunks = 1024 * kEmitAllPer;
constexpr uint32_t kEmitFew = 256 * kEmitAllPer;

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
// The whole message.  NT threads, at most kEmitAllPer chunks each in the scan, which every workgroup
// repeats: that is cheaper than a launch for it (1.6 us and its own round trips), up to 4096 chunks: 6.4 us
// on the 3243 chunks of the ResNet-50 shape, 4.9 on 512, 4.3 on 41 (11, 9 and 9 us for codes into staging
// words and a copy from there into the message); with 8060 chunks, eight per thread, 22 us, where
// k_tensor_scan and k_emit take 4.8 and 5.9.  Workgroups of 256 threads for few chunks, for the scans over
// sixteen wavefronts cost more than what they scan there.
// --------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(NT) void k_emit_all(
        const uint2* __restrict__ chunk_tensor, const ChunkSummary* __restrict__ sum, const uint32_t* __restrict__ codes,
        const uint32_t* __restrict__ heads, TensorState* __restrict__ st, unsigned long long* __restrict__ counters, int T, int b, uint32_t n_chunks,
        uint8_t* __restrict__ msg, uint64_t msg_capacity, ResultBlock* __restrict__ result, ResultBlock* __restrict__ next_result,
        unsigned long long* __restrict__ host_word, uint32_t seq) {
    constexpr int NW = NT / 64, PER = kEmitAllPer;
    __shared__ uint32_t scratch[4][16];
    constexpr uint32_t W = NT <= 256 ? 1024u : 256u;   // (words of a crowded chunk put together at a time)
    __shared__ __attribute__((aligned(16))) uint32_t win_sh[NW][kWindow<W>];
    extern __shared__ uint32_t offs[];                 // every chunk's bit offset in the payload, then the gaps
    uint32_t* const gaps = offs + n_chunks;
    constexpr uint32_t kNone = 0x80000000u, kStarts = 0x40000000u;     // (gaps are below 2^26 here)
    static_assert((uint64_t)kEmitAllChunks * kChunk <= 1u << 26, "positions and offsets in 32 bits");
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
