// Server step for all messages of a round at once (Alg. 1: dW <- 1/|I_t| sum of the clients' sparse
// updates): instead of one pass of scattered additions per message,
//   k_average_decode   decodes every stream of every message at the same time, into ascending lists of
//                      positions, and notes where each block of 2048 entries starts in them
//   k_average_apply    a wavefront per block of 2048 entries adds the messages' entries up in LDS, in
//                      message order (so that the sums are those of one message after another, bit for
//                      bit), and stores the block once
// The dense result is written once, in full lines, and never cleared or read beforehand.
// ResNet-50 shape (25.6e6 entries): 32 messages at p = 0.001 took 303 us one after another (a clear and
// 32 launches of 8.4 us that leave most of the chip idle), now 50 us for the two kernels and the status
// (47 us per call among others, for the call returns when the status is known); four at p = 0.01 took 109 us, now 72 us.
#pragma once

#include "sbc_decode_kernels.hpp"
#include "sbc_encode_kernels.hpp"

namespace sbc {

constexpr int kAvgMaxMsgs = 64;               // messages per pass (a lane each)
constexpr uint32_t kAvgBlock = 2048;          // entries per wavefront of k_average_apply
constexpr uint32_t kAvgPerChunk = kChunk / kAvgBlock;
// ... of which it holds a part at a time: half for few messages, whole blocks for many (see k_average_apply)
constexpr int kAvgWholeFrom = 48;
constexpr uint32_t kAvgTags = 256;            // places of k_average_apply where entries of equal positions meet
constexpr uint32_t kAvgNone = 0xFFFFFFFFu;    // no stream
constexpr uint32_t kAvgWhole = 0xFFFFFFFEu;   // in a workgroup's second place: all wavefronts take the first stream
constexpr uint32_t kAvgWaveSegs = 128;        // streams of up to this many segments are decoded by one wavefront
constexpr uint32_t kAvgMaxTiles = 16;         // ... and of up to this many tiles by one workgroup; longer ones are left
                                              // to the tile kernels, a message at a time

struct AvgTensor {
    float* out;
    uint32_t n;
    uint32_t kcap;        // positions there is room for per message
    uint32_t pos_off;     // first of them in a message's list
    uint32_t mark_off;    // first of the tensor's (blocks + 1) marks
};
struct AvgMsgs {                              // (a kernel argument)
    const uint8_t* msg[kAvgMaxMsgs];
    unsigned long long bytes[kAvgMaxMsgs];
};

constexpr int kAvgMinB = 2;                   // remainders of fewer bits (p above a fifth) are left to the general way, too

// Codes that can begin in a wavefront's 64 segments: 4096 bits, b + 1 of them each at the least.
template <int D>
constexpr uint32_t kAvgStage = D == 2 ? 1408u : 512u;

// Bound by the latency of a tile's steps (about 8 us: header, words, functions, sums, positions) times
// the tiles in turn and the workgroups' turns on a compute unit: 24 us for 32 messages at p = 0.001 of the
// ResNet-50 shape (28.5 with a limit of 64 segments for one wavefront instead of 128, 28.0 with 256).
// Positions go through LDS, for a compute unit sustains one scattered store per 3 ns (65 us for four
// messages at p = 0.01 with a store per lane and code, 46 with whole lines, 35 with the tiles of a
// stream shared).
// The streams that take whole workgroups come first, for all messages, the workgroups of short streams last: they are
// done soonest, and a few of them begin a second turn (message after message: 26 us).
// Workgroup by workgroup of the table, for all M messages.  ids: eight places per workgroup: a stream for each wavefront, or one
// for all of them, kAvgWhole, and which share of its tiles out of how many.
template <int D>
__global__ __launch_bounds__(kDecThreads) void k_average_decode(
        const AvgMsgs msgs, uint32_t M, const uint32_t* __restrict__ ids, const AvgTensor* __restrict__ tensors, int T, int b, float scale,
        uint32_t pos_stride, uint32_t* __restrict__ positions, uint32_t* __restrict__ marks, float* __restrict__ addends,
        ResultBlock* __restrict__ result, ResultBlock* __restrict__ next_result) {
    __shared__ __attribute__((aligned(16))) DecShared<D> sh;
    __shared__ uint32_t stage_sh[kDecWaves][kAvgStage<D>];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t which = blockIdx.x / M, m = blockIdx.x - which * M;
    SBC_TS(2, 0);
    if (which == 0u && m == 0u && tid == 0) next_result->err = 0u;
    const uint32_t second = ids[which * kDecWaves + 1];
    const bool whole = second == kAvgWhole;
    const uint32_t t = ids[which * kDecWaves + (whole ? 0 : wave)];
    if (tid < 256) build_table<D>(sh.fn, (uint32_t)tid, b);
    __syncthreads();
    if (t == kAvgNone) return;                             // (a wavefront of a workgroup that meets no barrier below)
    SBC_TS(2, 1);
    const AvgTensor a = tensors[t];
    const StreamInfo si = stream_info(msgs.msg[m], msgs.bytes[m], a.n, T, b, (int)t);
    if (!si.ok || si.nnz > a.kcap) {
        // (more positions than a sender with this p keeps: such a message is decoded on its own)
        if (lane == 0) atomicOr(&result->err, si.ok ? kErrDeferred : kErrCorrupt);
        return;
    }
    // The tiles of a long stream are shared among workgroups: each decodes those before its own, too, but
    // puts down only its own, and the last one what there is behind its tile.
    const uint32_t share = whole ? ids[which * kDecWaves + 2] : 0u;
    const bool last = !whole || share + 1u == ids[which * kDecWaves + 3];
    const unsigned long long seg_end = last ? si.n_seg : min(si.n_seg, (unsigned long long)(share + 1u) * kDecThreads);
    if (share && si.n_seg <= (unsigned long long)share * kDecThreads) return;
    if ((whole ? tid : lane) == 0 && share == 0u) addends[(size_t)t * M + m] = scale * si.mu;
    uint32_t* const pos = positions + (size_t)m * pos_stride + a.pos_off;
    uint32_t* const mk = marks + (size_t)a.mark_off * M + m;
    const uint32_t n_blocks = (a.n + kAvgBlock - 1u) / kAvgBlock;
    uint32_t* const stage = stage_sh[wave];
    // Marks: a block's is the number of positions before its start.  Blocks that start in (from, to]:
    auto mark = [&](unsigned long long from, unsigned long long to, uint32_t value, uint32_t first, uint32_t step) {
        const uint32_t last = (uint32_t)min(to / kAvgBlock, (unsigned long long)n_blocks);
        for (uint32_t blk = (uint32_t)min(from / kAvgBlock, (unsigned long long)n_blocks) + 1u + first; blk <= last; blk += step) mk[(size_t)blk * M] = value;
    };
    bool bad = false;
    auto put = [&](CodeWalk& w, bool active, uint32_t count) {
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)w.codes);
        const unsigned long long start = (w.ones << b) + w.rem + w.codes;
        if (active)
            while (w.x < 64) {
                const uint32_t at = w.next(), i = (uint32_t)w.codes - 1u - first;
                if (at != 0xFFFFFFFFu && i < kAvgStage<D>) stage[i] = at;
            }
        wave_lds_fence();
        // a lane per code: its position goes out, and the marks of the blocks between it and the code before it
        const uint32_t staged = min(count, kAvgStage<D>);
        uint32_t from = (uint32_t)min(start, 0xFFFFFFFFull);
        from = (uint32_t)__builtin_amdgcn_readfirstlane((int)from);
        for (uint32_t i = (uint32_t)lane; i < staged; i += 64u) {
            const uint32_t at = stage[i], before = i ? stage[i - 1u] : from;
            if (first + i < si.nnz) pos[first + i] = at;
            if (at / kAvgBlock != before / kAvgBlock) mark(before, at, first + i, 0u, 1u);
        }
        if (staged) from = stage[staged - 1u];
        const unsigned long long end = (w.ones << b) + w.rem + w.codes;    // of the last lane: the wavefront's
        const uint32_t to = last_lane((uint32_t)min(end, 0xFFFFFFFFull));
        if (to / kAvgBlock != from / kAvgBlock) mark(from, to, first + staged, (uint32_t)lane, 64u);
        wave_lds_fence();
    };
    const unsigned long long reached =
        whole ? decode_codes<D, kDecWaves>(sh, si, a.n, b, seg_end, [&](uint32_t tile) { return tile == share || (last && tile > share); }, bad, put)
              : decode_codes<D, 1>(sh, si, a.n, b, si.n_seg, [](uint32_t) { return true; }, bad, put);
    if (bad) atomicOr(&result->err, kErrCorrupt);          // (and nothing is applied)
    SBC_TS(2, 6);
    if (seg_end < si.n_seg) return;
    // the start of the list, and the blocks behind its end
    const uint32_t id = whole ? (uint32_t)tid : (uint32_t)lane, ids_n = whole ? kDecThreads : 64u;
    if (id == 0u) mk[0] = 0u;
    mark(reached, (unsigned long long)n_blocks * kAvgBlock, si.nnz, id, ids_n);
}

// Clears the tensors, a workgroup per chunk, and (if given) a result block.
__global__ __launch_bounds__(256) void k_average_clear(const uint2* __restrict__ chunk_tensor, const AvgTensor* __restrict__ tensors,
                                                       ResultBlock* __restrict__ block) {
    if (block && blockIdx.x == 0 && threadIdx.x == 0) block->err = 0u;
    const uint2 ct = chunk_tensor[blockIdx.x];             // (tensor, its first chunk)
    const AvgTensor a = tensors[ct.x];
    const uint32_t e0 = (blockIdx.x - ct.y) * (uint32_t)kChunk, cnt = min((uint32_t)kChunk, a.n - e0);
    const gfloat_ptr out = as_global(a.out + e0);
    const f32x4_any zero = 0.f;
#pragma unroll
    for (uint32_t i = 0; i < kChunk / 1024u; ++i) {
        const uint32_t at = (i * 256u + threadIdx.x) * 4u;
        if (at + 4u <= cnt) *(gf32x4_any_ptr)(out + at) = zero;
        else for (uint32_t j = 0; j < 4u; ++j) if (at + j < cnt) out[at + j] = 0.f;
    }
}

// A workgroup per chunk of 8192 entries, a wavefront per block of 2048: enough entries of all messages
// together (about 64 for 32 messages at p = 0.001) to give each lane one.  Bound by the store of the
// result, which starts four round trips after the kernel: 102 MB in 20.3 us (a plain fill: 16 us); 55.9 us with
// the messages one after another in each wavefront, two lanes busy at a time (issue bound).
// PART: entries of a block in LDS at a time.  Half a block leaves room for seven workgroups on a compute unit
// instead of four, but goes through the entries twice, with a search among the messages for each: ResNet-50
// shape, half / whole, 4 messages at p = 0.01 19.2 / 21.4 us, 8 24.2 / 25.8, 16 36.1 / 36.0, 32 59.1 / 56.3, 64
// 105.0 / 97.6; at p = 0.001 32 messages 20.2 / 20.3 (with other data in the caches in between 22.4 / 24.1), 64 26.2 / 24.6.
// ADD: out already holds the sum of the messages before these.
template <bool ADD, uint32_t PART>
__global__ __launch_bounds__(kEncThreads) void k_average_apply(
        const uint2* __restrict__ chunk_tensor, const AvgTensor* __restrict__ tensors, uint32_t M, uint32_t pos_stride,
        const uint32_t* __restrict__ positions, const uint32_t* __restrict__ marks, const float* __restrict__ addends,
        const ResultBlock* __restrict__ result) {
    static_assert(kAvgPerChunk == (uint32_t)kEncWaves, "a wavefront per block");
    __shared__ __attribute__((aligned(16))) float acc_sh[kEncWaves][PART];
    __shared__ __attribute__((aligned(16))) uint32_t tag_sh[kEncWaves][kAvgTags];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint2 ct = chunk_tensor[blockIdx.x];             // (tensor, its first chunk)
    const AvgTensor a = tensors[ct.x];
    const uint32_t blk = (blockIdx.x - ct.y) * kAvgPerChunk + wave, e0 = blk * kAvgBlock;
    if (e0 >= a.n || result->err) return;
    const uint32_t cnt = min(kAvgBlock, a.n - e0);
    float* const acc = acc_sh[wave];
    uint32_t* const tag = tag_sh[wave];
    const gfloat_ptr out = as_global(a.out + e0);
    // lane m: the entries of message m, s, s + 1, ... of its list
    uint32_t s = 0u, k = 0u;
    float addend = 0.f;
    if (lane < M) {
        const uint32_t* __restrict__ mk = marks + ((size_t)a.mark_off + blk) * M + lane;
        s = mk[0];
        k = mk[M] - s;
        addend = addends[(size_t)ct.x * M + lane];
    }
    const uint32_t end = (uint32_t)wave_incl_sum((unsigned long long)k), total = last_lane(end);
    const uint32_t shift = s - (end - k);
    // Entry e of the block, message after message: its message, position and addend.
    struct Entry { uint32_t m, at; float x; };
    auto entry = [&](uint32_t e) -> Entry {
        uint32_t m = 0u;                               // messages that end at or before e
#pragma unroll
        for (uint32_t step = 32u; step; step >>= 1) if ((uint32_t)__shfl((int)end, (int)(m + step - 1u), 64) <= e) m += step;
        const uint32_t i = e + (uint32_t)__shfl((int)shift, (int)m, 64);
        Entry r = {m, kAvgNone, __shfl(addend, (int)m, 64)};
        if (e < total) r.at = positions[(size_t)m * pos_stride + a.pos_off + i] - e0;
        return r;
    };
    const Entry first = entry(lane);                   // (of most blocks, all there are)
    uint32_t turn = 0u;
#pragma unroll
    for (uint32_t i = 0; i < kAvgTags / 256u; ++i) reinterpret_cast<uint4*>(tag)[i * 64u + lane] = make_uint4(0u, 0u, 0u, 0u);
#pragma nounroll
    for (uint32_t h0 = 0u; h0 < cnt; h0 += PART) {
#pragma unroll
        for (uint32_t i = 0; i < PART / 256u; ++i) {
            const uint32_t at = h0 + (i * 64u + lane) * 4u;
            f32x4 v = 0.f;
            if (ADD) {
                if (at + 4u <= cnt) v = *(const gf32x4_any_ptr)(out + at);
                else for (uint32_t j = 0; j < 4u; ++j) if (at + j < cnt) v[j] = out[at + j];
            }
            reinterpret_cast<f32x4*>(acc)[i * 64u + lane] = v;
        }
        wave_lds_fence();
        // A lane per entry, in message order.  Entries of one position are added in that order: where lanes meet at a
        // tag (a hash of the position), the first of them goes first, the others take another turn.  A message's
        // positions are distinct, so a batch of one message has nothing to sort out.
        Entry next = first;
        if (h0 && total > 64u) next = entry(lane);
        for (uint32_t base = 0u; base < total; base += 64u) {
            const Entry now = next;
            if (base + 64u < total) next = entry(base + 64u + lane);
            const uint32_t at = now.at - h0;
            bool todo = at < PART;                 // (kAvgNone, or of the other half: not)
            const bool single = (uint32_t)__builtin_amdgcn_readfirstlane((int)now.m) ==
                                (uint32_t)__builtin_amdgcn_readlane((int)now.m, (int)min(63u, total - base - 1u));
            if (single) {
                if (todo) acc[at] += now.x;
            } else {
                while (__any(todo)) {
                    turn += 64u;                       // (tags only grow: none is ever cleared)
                    const uint32_t mine = turn + 63u - lane;
                    uint32_t* const place = tag + (at & (kAvgTags - 1u));
                    if (todo) __hip_atomic_fetch_max(place, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    wave_lds_fence();
                    if (todo && *place == mine) {
                        acc[at] += now.x;
                        todo = false;
                    }
                    wave_lds_fence();
                }
            }
            wave_lds_fence();
        }
#pragma unroll
        for (uint32_t i = 0; i < PART / 256u; ++i) {
            const uint32_t at = h0 + (i * 64u + lane) * 4u;
            const f32x4 v = reinterpret_cast<const f32x4*>(acc)[i * 64u + lane];
            if (at + 4u <= cnt) *(gf32x4_any_ptr)(out + at) = v;
            else for (uint32_t j = 0; j < 4u; ++j) if (at + j < cnt) out[at + j] = v[j];
        }
        wave_lds_fence();
    }
}

}  // namespace sbc
