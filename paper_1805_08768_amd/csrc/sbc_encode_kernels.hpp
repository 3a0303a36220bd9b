// The rest of the client step once the thresholds are known, a wavefront per chunk of 8192 entries:
//   k_apply  : Alg. 2's side decision, Alg. 1's residual line and the kept-position bitmap from the
//              chunk's run of candidates; per chunk, count / first / last kept position and the code
//              bits of every kept entry whose predecessor lies in the same chunk
//   k_tile_summary, k_tensor_scan : tensors of many chunks only: scan over a tensor's chunks in
//              tiles of 4096 (predecessor of each chunk's first kept entry, bit offset of each chunk)
//   k_emit   : Alg. 3: writes q ones, a zero and the b-bit remainder of every kept entry at its bit
//              offset in the tensor's staging words (tensors of few chunks: the wavefront first scans
//              the summaries of the chunks before its own)
// (the message is then assembled by k_finish_message)
//
// Candidates of one chunk sit next to each other in their tensor's lists (a workgroup of the
// streaming kernel appends them as one run), so the chunk is the unit of work here and no kept
// position is ever sorted: the bitmap, in LDS, puts a chunk's in order, and chunks are in order.  A
// wavefront per chunk needs no barrier, and its 256 bitmap words are four per lane.  Both kernels are
// bound by their three dependent round trips to memory: 5.7 and 6.9 us on 25.6e6 entries at p = 0.001
// (3243 chunks), 10.7 and 8.2 us at p = 0.01, 4.9 and 5.4 us on 41 chunks.
#pragma once

#include "sbc_device.hpp"
#include "sbc_threshold_kernels.hpp"

namespace sbc {

constexpr int kEncThreads = 256;
constexpr int kEncWaves = kEncThreads / 64;
static_assert(kChunkWords == 256, "four bitmap words per lane");

__device__ __forceinline__ uint32_t golomb_len(uint32_t gap, int b) { return (gap >> b) + 1u + (uint32_t)b; }

// val (< 2^nb, 1 <= nb <= 32) written MSB-first at bit `pos` of a zero-initialised word array.
__device__ __forceinline__ void put_bits(uint32_t* words, unsigned long long pos, uint32_t val, int nb) {
    const unsigned long long w = pos >> 5;
    const int off = (int)(pos & 31ull);
    const unsigned long long v = (unsigned long long)val << (64 - off - nb);
    const uint32_t hi = (uint32_t)(v >> 32), lo = (uint32_t)v;
    if (hi) atomicOr(&words[w], hi);
    if (lo) atomicOr(&words[w + 1], lo);
}

// q one-bits starting at bit `pos`.
__device__ __forceinline__ void put_ones(uint32_t* words, unsigned long long pos, unsigned long long q) {
    while (q) {
        const unsigned long long w = pos >> 5;
        const uint32_t room = 32u - (uint32_t)(pos & 31ull);
        const uint32_t take = q < room ? (uint32_t)q : room;
        if (take == 32u) words[w] = 0xFFFFFFFFu;        // the whole word belongs to this run
        else atomicOr(&words[w], ((1u << take) - 1u) << (room - take));
        pos += take;
        q -= take;
    }
}

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

// --------------------------------------------------------------------------
// Side, mean, residual update and bitmap.
// --------------------------------------------------------------------------
__global__ __launch_bounds__(kEncThreads) void k_apply(
        const TensorDesc* __restrict__ desc, const uint2* __restrict__ chunk_tensor, const ChunkRun* __restrict__ runs,
        const TensorState* __restrict__ st, TensorState* res, const uint2* __restrict__ cand,
        uint64_t cand_entries, uint32_t* __restrict__ bitmap, ChunkSummary* __restrict__ sum,
        uint32_t* __restrict__ stage, int b, int pass, uint32_t n_chunks, ResultBlock* __restrict__ result) {
    __shared__ __attribute__((aligned(16))) uint32_t bits_sh[kEncWaves][kChunkWords];
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
        if ((uint32_t)lane < run.cnt[s] && run.at[s] < cand_entries - 64u) e0[s] = cand[run.at[s] + (uint32_t)lane];
    }
    reinterpret_cast<uint4*>(bm)[lane] = make_uint4(0u, 0u, 0u, 0u);
    const TensorDesc d = desc[t];
    const uint32_t flags = st[t].flags, kc0 = st[t].kc[0], kc1 = st[t].kc[1];
    const double Sp = st[t].S[0], Sn = st[t].S[1];
    if (!encoded_in_pass(flags, pass)) return;
    // Alg. 2 compares the means (sums that differ may still give equal means: the positive side then)
    const int chosen = (Sp / (double)kc0 >= Sn / (double)kc1) ? 0 : 1;
    const float mu32 = (float)((chosen ? Sn : Sp) / (double)(chosen ? kc1 : kc0));
    const float mu_signed = chosen ? -mu32 : mu32;
    const uint32_t tau = st[t].tau[chosen], itau = st[t].itau[chosen];
    if (cc == 0u && lane == 0) { res[t].side = chosen ? -1 : 1; res[t].mu_signed = mu_signed; }
    // this chunk's share of the tensor's staging words, for k_emit
    {
        const uint32_t per = (d.bound_words + d.nchunks - 1u) / d.nchunks;
        const uint32_t lo = per * cc;
        const uint32_t hi = (lo + per < d.bound_words) ? lo + per : d.bound_words;
        for (uint32_t w = lo + lane; w < hi; w += 64u) stage[d.stage_off + w] = 0u;
    }
    const uint2* __restrict__ list = cand + run.at[chosen];
    const uint32_t cnt = run.cnt[chosen];
    const gfloat_ptr R = as_global(d.R);
    wave_lds_fence();
    bool bad = false;
    auto keep = [&](const uint2& e) {
        if (!cand_kept(e.x, e.y, tau, itau)) return;
        if (e.y >= d.n || e.y / (uint32_t)kChunk != cc) { bad = true; return; }      // (cannot happen)
        const float a = __uint_as_float(bits_of_key(chosen ? ~e.x : e.x));
        R[e.y] = a - mu_signed;                        // Alg. 1: R <- dW - dW*
        atomicOr(&bm[(e.y % (uint32_t)kChunk) >> 5], 1u << (e.y & 31u));
    };
    // (at the very end of the array the first entries were not read ahead)
    const bool ahead = run.at[chosen] < cand_entries - 64u;
    if (ahead && (uint32_t)lane < cnt) keep(chosen ? e0[1] : e0[0]);
    for (uint32_t i0 = ahead ? 64u : 0u; i0 < cnt; i0 += 256u) {
        uint2 e[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t i = i0 + 64u * u + (uint32_t)lane;
            e[u] = list[i < cnt ? i : 0u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + 64u * u + (uint32_t)lane < cnt) keep(e[u]);
    }
    if (bad) atomicOr(&result->err, kErrInternal);
    wave_lds_fence();
    const uint4 words = reinterpret_cast<const uint4*>(bm)[lane];
    reinterpret_cast<uint4*>(bitmap + (uint64_t)c * kChunkWords)[lane] = words;
    const uint32_t p0 = (uint32_t)lane * 128u;
    uint32_t last_end, bits = 0u, first = 0xFFFFFFFFu;
    uint32_t pe = wave_excl_max(last_bit_end(words, p0), &last_end);
    for_bits(words, p0, [&](uint32_t x) {
        if (pe) bits += golomb_len(x - pe, b);
        else first = x;                                // the only entry of the chunk without predecessor
        pe = x + 1u;
    });
    const uint32_t count = (uint32_t)(__popc(words.x) + __popc(words.y) + __popc(words.z) + __popc(words.w));
    const unsigned long long both = wave_incl_sum((unsigned long long)bits | ((unsigned long long)count << 32));
    const unsigned long long has = __ballot(first != 0xFFFFFFFFu);
    first = (uint32_t)__builtin_amdgcn_readlane((int)first, has ? __ffsll((long long)has) - 1 : 0);
    if (lane == 63) {
        ChunkSummary cs;
        cs.cnt = (uint32_t)(both >> 32); cs.first = first; cs.last_end = last_end; cs.inner_bits = (uint32_t)both;
        sum[c] = cs;
    }
}

constexpr int kScanThreads = 1024;
constexpr int kScanPer = 4;              // consecutive chunks per thread
constexpr uint32_t kScanTile = kScanThreads * kScanPer;   // chunks per workgroup of the scan

// What a tile of kScanTile consecutive chunks of a tensor contributes to the scan over all of
// the tensor's chunks.  The code of the tile's first kept entry depends on where the previous
// kept entry lies, which the tile does not know: its bits are left out and its position kept.
struct TileSummary {
    uint32_t cnt;              // kept entries in the tile
    uint32_t end;              // position + 1 of the last one (0: none)
    uint32_t first;            // position of the first one (if cnt != 0)
    uint32_t pad;
    unsigned long long bits;   // code bits of all of them but the first
    unsigned long long pad2;
};

// Tiles of tensor t live at tiles[chunk0 / kScanTile + t ...]: tensors never overlap there
// (floor((a + n) / T) + 1 >= floor(a / T) + ceil(n / T)).
__device__ __forceinline__ uint32_t tile_base(const TensorDesc& d, int t) { return d.chunk0 / kScanTile + (uint32_t)t; }

// One tile's share of the scan, given what precedes the tile: predecessor of each chunk's first
// kept entry, bit offset of each chunk.  WRITE = false only adds up the tile (first pass of a
// tensor of several tiles, carries unknown: pe == 0 marks the tile's first kept entry).
template <bool WRITE>
__device__ __forceinline__ void scan_tile(const TensorDesc& d, uint32_t tile, const ChunkSummary* __restrict__ sum,
                                          uint32_t carry_end, unsigned long long carry_bits, int b,
                                          uint32_t* __restrict__ chunk_prev_end, uint64_t* __restrict__ chunk_bitoff,
                                          uint32_t* scratch32, unsigned long long* scratch64,
                                          uint32_t& tile_end, unsigned long long& tile_bits, uint32_t& tile_cnt,
                                          uint32_t& first_pos, bool& has_first) {
    const int tid = threadIdx.x;
    const uint32_t c0 = tile * kScanTile + (uint32_t)tid * kScanPer;
    ChunkSummary s[kScanPer];
    uint32_t gend[kScanPer], my_end = 0u, my_cnt = 0u;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        s[j].cnt = 0u; s[j].first = 0u; s[j].last_end = 0u; s[j].inner_bits = 0u;
        if (c0 + j < d.nchunks) s[j] = sum[d.chunk0 + c0 + j];
        gend[j] = s[j].cnt ? (c0 + j) * (uint32_t)kChunk + s[j].last_end : 0u;
        if (gend[j] > my_end) my_end = gend[j];
        my_cnt += s[j].cnt;
    }
    uint32_t pe = block_excl_max<uint32_t, kScanThreads>(my_end, &tile_end, scratch32);
    if (carry_end > pe) pe = carry_end;
    // predecessor end and code bits of every chunk's first kept entry
    uint32_t pes[kScanPer];
    unsigned long long bits[kScanPer], my_bits = 0ull;
    has_first = false; first_pos = 0u;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        pes[j] = pe;
        bits[j] = 0ull;
        if (s[j].cnt) {
            const uint32_t pos = (c0 + j) * (uint32_t)kChunk + s[j].first;
            bits[j] = (unsigned long long)s[j].inner_bits;
            if (!WRITE && pe == 0u) { has_first = true; first_pos = pos; }      // (a kept entry's end is at least 1)
            else bits[j] += (unsigned long long)((pos - pe) >> b) + 1ull + (unsigned long long)b;
            pe = gend[j];
        }
        my_bits += bits[j];
    }
    unsigned long long off = carry_bits + block_excl_sum<unsigned long long, kScanThreads>(my_bits, &tile_bits, scratch64);
    (void)block_excl_sum<uint32_t, kScanThreads>(my_cnt, &tile_cnt, scratch32);
    if (WRITE) {
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            if (c0 + j < d.nchunks) {
                chunk_prev_end[d.chunk0 + c0 + j] = pes[j];
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
    uint32_t tile_end, tile_cnt, first_pos;
    unsigned long long tile_bits;
    bool has_first;
    scan_tile<false>(d, blockIdx.y, sum, 0u, 0ull, b, nullptr, nullptr, scratch32, scratch64, tile_end, tile_bits, tile_cnt,
                     first_pos, has_first);
    TileSummary* const out = tiles + tile_base(d, t) + blockIdx.y;
    if (has_first) out->first = first_pos;              // exactly one thread of a tile that holds entries
    if (tid == 0) { out->cnt = tile_cnt; out->end = tile_end; out->bits = tile_bits; }
}

// grid (T, tiles): per tensor, scan over its chunks: every tile folds the summaries of the
// tiles before it, then scans its own chunks.
__global__ __launch_bounds__(kScanThreads) void k_tensor_scan(const TensorDesc* __restrict__ desc,
                                                              const ChunkSummary* __restrict__ sum,
                                                              const TileSummary* __restrict__ tiles,
                                                              uint32_t* __restrict__ chunk_prev_end,
                                                              uint64_t* __restrict__ chunk_bitoff,
                                                              TensorState* __restrict__ st, int b, int pass) {
    __shared__ uint32_t scratch32[kScanThreads / 64];
    __shared__ unsigned long long scratch64[kScanThreads / 64];
    const int t = blockIdx.x, tid = threadIdx.x;
    const TensorDesc d = desc[t];
    if (!encoded_in_pass(st[t].flags, pass)) return;
    const uint32_t n_tiles = (d.nchunks + kScanTile - 1u) / kScanTile;
    if (blockIdx.y >= n_tiles) return;
    uint32_t carry_end = 0u, carry_cnt = 0u;            // position+1 of the last kept entry so far (0: none)
    unsigned long long carry_bits = 0ull;
    const TileSummary* __restrict__ ts = tiles + tile_base(d, t);
    for (uint32_t j = 0; j < blockIdx.y; ++j) {         // (every thread: the same few loads)
        const TileSummary s = ts[j];
        if (s.cnt) {
            carry_bits += s.bits + (unsigned long long)((s.first - carry_end) >> b) + 1ull + (unsigned long long)b;
            carry_end = s.end;                           // positions grow from tile to tile
            carry_cnt += s.cnt;
        }
    }
    uint32_t tile_end, tile_cnt, first_pos;
    unsigned long long tile_bits;
    bool has_first;
    scan_tile<true>(d, blockIdx.y, sum, carry_end, carry_bits, b, chunk_prev_end, chunk_bitoff, scratch32, scratch64,
                    tile_end, tile_bits, tile_cnt, first_pos, has_first);
    if (tid == 0 && blockIdx.y == n_tiles - 1u) { st[t].bit_len = carry_bits + tile_bits; st[t].nnz = carry_cnt + tile_cnt; }
}

// Most chunks a tensor may have for the wavefronts of k_emit to do the scan's work themselves (each
// reads the summaries of all chunks before its own: up to eight per lane).
constexpr int kSelfScanPer = 8;
constexpr uint32_t kSelfScanChunks = 64 * kSelfScanPer;
constexpr uint32_t kEmitWords = 384;     // stream words of a chunk put together in LDS (a chunk's usual share even at p = 0.4)

// What precedes chunk cc of a tensor, from the summaries of its chunks 0 .. cc-1: position + 1 of
// the last kept entry before the chunk (0: none), the code bits and the kept entries before it.
__device__ __forceinline__ void scan_before_chunk(uint32_t chunk0, uint32_t cc, const ChunkSummary* __restrict__ sum,
                                                  int b, uint32_t& prev_end, unsigned long long& bit_off, uint32_t& cnt_before) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t per = (cc + 63u) / 64u;              // consecutive chunks of a lane
    ChunkSummary s[kSelfScanPer];
    uint32_t gend[kSelfScanPer], my_end = 0u;
    unsigned long long my_cnt = 0ull;
#pragma unroll
    for (int j = 0; j < kSelfScanPer; ++j) {
        s[j].cnt = 0u; s[j].first = 0u; s[j].last_end = 0u; s[j].inner_bits = 0u;
        if ((uint32_t)j < per) {                        // uniform
            const uint32_t i = lane * per + (uint32_t)j;
            if (i < cc) s[j] = sum[chunk0 + i];
        }
    }
#pragma unroll
    for (int j = 0; j < kSelfScanPer; ++j) {
        gend[j] = s[j].cnt ? (lane * per + (uint32_t)j) * (uint32_t)kChunk + s[j].last_end : 0u;
        my_end = gend[j] > my_end ? gend[j] : my_end;
        my_cnt += s[j].cnt;
    }
    uint32_t pe = wave_excl_max(my_end, &prev_end);
    unsigned long long my_bits = 0ull;
#pragma unroll
    for (int j = 0; j < kSelfScanPer; ++j) {
        if (s[j].cnt) {
            const uint32_t pos = (lane * per + (uint32_t)j) * (uint32_t)kChunk + s[j].first;
            my_bits += (unsigned long long)s[j].inner_bits + (unsigned long long)golomb_len(pos - pe, b);
            pe = gend[j];
        }
    }
    bit_off = last_lane(wave_incl_sum(my_bits));
    cnt_before = (uint32_t)last_lane(wave_incl_sum(my_cnt));
}

template <bool SELF>
__global__ __launch_bounds__(kEncThreads) void k_emit(
        const TensorDesc* __restrict__ desc, const uint2* __restrict__ chunk_tensor,
        const uint32_t* __restrict__ bitmap, const ChunkSummary* __restrict__ sum,
        const uint32_t* __restrict__ chunk_prev_end, const uint64_t* __restrict__ chunk_bitoff,
        const TensorState* __restrict__ st, TensorState* res, int b, int pass,
        uint32_t* __restrict__ stage, uint32_t n_chunks, ResultBlock* __restrict__ result) {
    __shared__ uint32_t words_sh[kEncWaves][kEmitWords + 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t c = blockIdx.x * (uint32_t)kEncWaves + (uint32_t)wave;
    if (c >= n_chunks) return;
    // (everything the chunk may need is asked for at once, before the descriptor says whether it is)
    const uint2 ct = chunk_tensor[c];                  // (tensor, its first chunk)
    const uint32_t t = ct.x, cc = c - ct.y;
    const uint4 words = reinterpret_cast<const uint4*>(bitmap + (uint64_t)c * kChunkWords)[lane];
    const uint32_t cnt = sum[c].cnt;
    uint32_t prev_end = SELF ? 0u : chunk_prev_end[c], cnt_before = 0u;
    unsigned long long bit_off = SELF ? 0ull : chunk_bitoff[c];
    const TensorDesc d = desc[t];
    const uint32_t flags = st[t].flags;
    // (garbage if an earlier kernel has left the tensor alone, and then not used)
    if (SELF && cc) scan_before_chunk(ct.y, cc, sum, b, prev_end, bit_off, cnt_before);
    if (!encoded_in_pass(flags, pass)) return;
    const bool last_chunk = SELF && cc == d.nchunks - 1u;
    if (cnt == 0u && !last_chunk) return;
    if (cnt == 0u) {
        if (lane == 0) { res[t].bit_len = bit_off; res[t].nnz = cnt_before; }
        return;
    }
    const uint32_t e0 = cc * (uint32_t)kChunk, p0 = e0 + (uint32_t)lane * 128u;
    uint32_t last_end;
    uint32_t pe = wave_excl_max(last_bit_end(words, p0), &last_end);
    if (pe == 0u) pe = prev_end;
    unsigned long long bits = 0ull;
    {
        uint32_t p = pe;
        for_bits(words, p0, [&](uint32_t x) {
            bits += (unsigned long long)((x - p) >> b) + 1ull + (unsigned long long)b;
            p = x + 1u;
        });
    }
    const unsigned long long inc = wave_incl_sum(bits), chunk_bits = last_lane(inc);
    if (last_chunk && lane == 0) { res[t].bit_len = bit_off + chunk_bits; res[t].nnz = cnt_before + cnt; }
    if (((bit_off + chunk_bits + 31ull) >> 5) > d.bound_words) {      // would leave the tensor's staging words
        if (lane == 0) atomicOr(&result->err, kErrInternal);
        return;
    }
    uint32_t* __restrict__ out = stage + d.stage_off;
    const unsigned long long w0 = bit_off >> 5;
    const unsigned long long n_words = ((bit_off + chunk_bits + 31ull) >> 5) - w0;
    auto write_codes = [&](uint32_t* dst, unsigned long long pos) {
        for_bits(words, p0, [&](uint32_t x) {
            const uint32_t gap = x - pe;
            const uint32_t q = gap >> b;
            put_ones(dst, pos, q);
            pos += q;
            put_bits(dst, pos, gap & ((1u << b) - 1u), b + 1);        // the zero and the remainder
            pos += (unsigned)b + 1u;
            pe = x + 1u;
        });
    };
    if (n_words <= (unsigned long long)kEmitWords) {
        // the chunk's words in LDS; only the first and the last may hold other chunks' bits as well
        uint32_t* const lds = words_sh[wave];
        const uint32_t nw = (uint32_t)n_words;
        for (uint32_t w = lane; w < nw + 1u; w += 64u) lds[w] = 0u;
        wave_lds_fence();
        write_codes(lds, (bit_off & 31ull) + (inc - bits));
        wave_lds_fence();
        for (uint32_t w = lane; w < nw; w += 64u) {
            const uint32_t v = lds[w];
            if (w != 0u && w + 1u != nw) out[w0 + w] = v;
            else if (v) atomicOr(&out[w0 + w], v);
        }
    } else {
        write_codes(out, bit_off + (inc - bits));      // (a long run of ones, or a chunk of many ties)
    }
}

}  // namespace sbc
