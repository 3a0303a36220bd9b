// Alg. 2's selection: per tensor and sign side, the exact threshold (key of the k-th most extreme
// entry and, among entries equal to it, the highest index kept), and S, the sum of the kept values.
//
//   k_threshold      one workgroup per (tensor, side).  The two sides of a tensor are independent
//                    until their means are compared, so they run on two compute units at once and
//                    whoever needs the side compares the two results (k_apply, k_finish_message).
//   k_wide_count,    for tensors that keep very many entries: the window histogram of a side's list,
//   k_wide_collect   then the entries of the k-th entry's bin copied out and the entries beyond that
//                    bin summed, both as sweeps by many workgroups; k_threshold then selects among
//                    the copied entries alone.
//
// A side is selected in two passes over its list: the first counts the leading 20 key bits in a window of
// two octaves above the filter key, which gives the k-th entry's bin; the second adds up the entries beyond
// that bin and collects the few in it, whose ranks among one another give the threshold (more than 256 of
// them: their other 12 bits are counted, too).  That is exact whatever the ties.  Sums are exact integers
// rounded once to fp64 (or one integer per fp32 exponent where the values spread too far).
#pragma once

#include "sbc_device.hpp"

namespace sbc {

constexpr int kThThreads = 1024;
constexpr int kThShift = 12;                              // low key bits: the second pass's bins
constexpr int kThBins = 1 << kThShift;                    // bins of either pass; 2048 of the first per octave
constexpr uint32_t kThRanked = 256;                       // most entries of the k-th entry's bin that are ranked one against the others

constexpr int kWideThreads = 1024;       // sweeps over the lists of tensors that keep very many entries
constexpr int kMaxWide = 64;             // such tensors per call
// The call's wide tensors, passed to the kernels by value: a workgroup learns its tensor from the
// kernel arguments instead of from a load that everything else would have to wait for.
struct WideIds { uint32_t id[kMaxWide]; };

// What k_wide_collect leaves for k_threshold, per (wide tensor, side).
struct WideState {
    uint32_t ok;          // 0: the steps did not apply, k_threshold works on the whole list
    uint32_t prefix;      // leading key bits of the k-th entry
    uint32_t need;        // its rank among the entries with those bits
    uint32_t count;       // entries copied out
    uint32_t next_rank_bin; // window bin a following call's filter key sits at (0xFFFFFFFF: not in the window)
    uint32_t pad[3];
};

// The first side key that an fp64 sum of up to kc values at or beyond `from` may not contain if it is to
// be exact: below it all of them are multiples of from's last place and add up to less than 2^53 of
// those (24 bits, one per binade beyond from's, those of kc).  0: no such sum (values of both signs).
__device__ __forceinline__ uint32_t exact_limit(uint32_t from, uint32_t kc) {
    const uint32_t bits_k = 32u - (uint32_t)__clz((int)kc);
    if (from <= 0x80000000u || bits_k > 29u) return 0u;
    return 0x80000000u | (min(((from >> 23) & 0xFFu) + 29u - bits_k + 1u, 0xFFu) << 23);
}

// Room for the copied entries of a side: the tensor's own bitmap words, which nothing uses before
// the positions are written (k_apply).
__device__ __forceinline__ uint32_t wide_room(const TensorDesc& d) { return d.nchunks * (uint32_t)(kChunkWords / 4); }
__device__ __forceinline__ CandPtr wide_list(const TensorDesc& d, uint32_t* bitmap, int s) {
    return {bitmap + (uint64_t)d.chunk0 * kChunkWords + (s ? 2u * wide_room(d) : 0u), wide_room(d)};
}

__device__ __forceinline__ bool cand_kept(uint32_t key, uint32_t idx, uint32_t tau, uint32_t itau) {
    return key > tau || (key == tau && idx <= itau);
}

// Mantissa (signed the way the side sums it) and exponent slot of the value a side key stands for.
__device__ __forceinline__ long long signed_mantissa(uint32_t key, int s, uint32_t& ex) {
    const uint32_t u = bits_of_key(s ? ~key : key);
    ex = (u >> 23) & 0xFFu;
    long long m = (long long)(ex ? ((u & 0x7FFFFFu) | 0x800000u) : (u & 0x7FFFFFu));
    if (ex == 0u) ex = 1u;
    if (((u >> 31) != 0u) != (s != 0)) m = -m;         // the negative side sums -A
    return m;
}

// A tensor's candidates per side, and where those of each segment of side s start in the list as one piece.
struct ListCounts {
    uint32_t p, n;
    uint32_t segs;
    uint32_t over;        // some segment has more than it holds (nothing was stored beyond its end)
    uint32_t crowded;     // some segment holds more than twice its part of the list
    uint32_t cnt[kSegs], before[kSegs];
    __device__ __forceinline__ uint32_t of(int side) const { return side ? n : p; }
    // as it was left in LDS, without the segments' figures
    __device__ __forceinline__ static ListCounts totals(const ListCounts& l) {
        ListCounts c;
        c.p = uniform(l.p); c.n = uniform(l.n); c.segs = uniform(l.segs); c.over = uniform(l.over); c.crowded = uniform(l.crowded);
        return c;
    }
    // Entries [lo, hi) of the list as one piece that lie in segment g, counted from its start.
    __device__ __forceinline__ uint2 part_of(uint32_t g, uint32_t lo, uint32_t hi) const {
        const uint32_t b = uniform(before[g]), e = b + uniform(cnt[g]);
        lo = max(lo, b); hi = min(hi, e);
        return lo < hi ? make_uint2(lo - b, hi - b) : make_uint2(0u, 0u);
    }
    // Of `parts` wavefronts (more than there are segments) that share a crowded list of `all` entries, number me's:
    // a segment, its place in it, and how many have that segment.  Every segment that holds anything has one, the
    // others go by the entries, what is left over to the largest.
    __device__ __forceinline__ uint3 share_of(uint32_t me, uint32_t parts, uint32_t all) const {
        const uint32_t per = all / (parts - kSegs) + 1u;
        uint32_t left = parts, largest = 0u, most = 0u;
#pragma nounroll
        for (uint32_t g = 0; g < kSegs; ++g) {
            const uint32_t c = uniform(cnt[g]);
            left -= c ? 1u + c / per : 0u;
            if (c > most) { most = c; largest = g; }
        }
        uint3 share = make_uint3(largest, 0u, 1u);
        uint32_t at = 0u;
#pragma nounroll
        for (uint32_t g = 0; g < kSegs; ++g) {
            const uint32_t c = uniform(cnt[g]), has = (c ? 1u + c / per : 0u) + (g == largest ? left : 0u);
            if (me - at < has) share = make_uint3(g, me - at, has);
            at += has;
        }
        return share;
    }
};
// Entries of a segment that are not worth cutting (k_threshold: what two wavefronts hold in registers).
constexpr uint32_t kSegWhole = 2048;
// Added up from the segments' counters by the first wavefront of a workgroup, for all of them: `to` lies in
// LDS and holds once the next barrier has been passed.  (Every wavefront by itself: 0.6 us more.)
__device__ __forceinline__ void count_list(ListCounts& to, const TensorDesc& d, const TensorState* __restrict__ st,
                                           const unsigned long long* __restrict__ counters, int t, int s, uint32_t flags) {
    if (threadIdx.x >= 64u) return;
    const uint32_t lane = threadIdx.x;
    unsigned long long own = counters[((size_t)t * kSegs + lane % kSegs) * kCounterStride];
    const uint32_t segs = (flags & kStExact) ? 1u : d.segs;            // (the histogram route's lists are in one piece)
    if (segs == 1u) own = lane ? 0ull : (unsigned long long)st[t].cand_cnt[0] | ((unsigned long long)st[t].cand_cnt[1] << 32);
    bool over = false;
    if (d.cand_cap < d.n) {                            // (uniform; else there is room for every entry)
        const uint32_t room = seg_before(d, segs, min(lane + 1u, segs)) - seg_before(d, segs, min(lane, segs));
        over = lane < segs && ((uint32_t)own > room || (uint32_t)(own >> 32) > room);
    }
    over = __any(over);
    static_assert(kSegs == 8, "three steps");
    unsigned long long upto = own;
    upto += dpp_fetch<0x111, 0xf>(upto);
    upto += dpp_fetch<0x112, 0xf>(upto);
    upto += dpp_fetch<0x114, 0xf>(upto);
    const int half = s ? 32 : 0;
    const uint32_t mine = (uint32_t)(own >> half), all = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(upto >> half), (int)kSegs - 1);
    const bool crowded = segs > 1u && __any(lane < kSegs && mine > kSegWhole && mine > all / (kSegs / 2u));
    if (lane < kSegs) {
        to.cnt[lane] = mine;
        to.before[lane] = (uint32_t)(upto >> half) - mine;
    }
    if (lane == kSegs - 1u) {
        to.p = (uint32_t)upto; to.n = (uint32_t)(upto >> 32); to.segs = segs; to.over = over ? 1u : 0u; to.crowded = crowded ? 1u : 0u;
    }
}

// What a tensor's candidate counts rule out before any selection: true if the tensor cannot be
// selected from its lists (the thread with `lead` set has then flagged it, for the histogram route
// or as an error).
__device__ __forceinline__ bool lists_unusable(const TensorDesc& d, TensorState* __restrict__ st, int t, const ListCounts& counts,
                                               int pass, bool lead, ResultBlock* __restrict__ result) {
    const uint32_t cnt_p = counts.p, cnt_n = counts.n;
    const bool sampled = (d.flags & kDescSampled) != 0u;
    if (cnt_p > d.n || cnt_n > d.n || (sampled && (cnt_p == 0u || cnt_n == 0u))) {
        // (a sampled threshold is the key of an entry of the tensor, so that entry is a candidate)
        if (lead) { st[t].flags = kStFailed; atomicOr(&result->err, kErrInternal); }
        return true;
    }
    if (counts.over) {
        // compact context: more candidates than a list (or a segment of it) holds (nothing was stored beyond its end).  The
        // histogram route extracts a tighter set; if that does not fit either, the call fails.
        if (lead) {
            st[t].flags = kStFailed;
            st[t].bit_len = 0ull; st[t].nnz = 0u;
            atomicOr(&result->err, pass == 0 && !sampled ? kErrPrefilter : kErrOverflow);
        }
        return true;
    }
    if (!sampled && (cnt_p < d.k || cnt_n < d.k)) {
        // the filter kept too few entries on a side: the histogram path redoes this tensor
        if (lead) {
            st[t].flags = kStFailed;
            st[t].bit_len = 0ull; st[t].nnz = 0u;
            atomicOr(&result->err, pass == 0 ? kErrPrefilter : kErrInternal);
        }
        return true;
    }
    return false;
}

// Entries a side keeps: k; in the subsampled variant every candidate (all entries at or beyond the
// sampled threshold), up to the cap.
__device__ __forceinline__ uint32_t kept_of_side(const TensorDesc& d, uint32_t cnt) {
    return (d.flags & kDescSampled) ? min(cnt, d.kcap) : d.k;
}

// Bin of a side key in the window above the side's filter key; the top bin takes everything beyond.
__device__ __forceinline__ uint32_t window_bin(uint32_t key, uint32_t base) {
    // (no candidate lies below its filter key)
    return min(max(key >> kThShift, base) - base, (uint32_t)(kThBins - 1));
}

// Walking the kThBins counts of hist (LDS) from the top bin down: the bin at which the running
// count reaches need (res[0]; 0xFFFFFFFF if it never does), the count before it (res[1]), the bin's
// own count (res[3]), and the bin at which the running count reaches rank2 (res[2], or 0xFFFFFFFF;
// rank2 = 0 looks for none).  res[0] and res[2] must hold 0xFFFFFFFF when the first barrier is
// reached.  The counts are zero again afterwards.  Two barriers.  (All 1024 threads, four bins each: one
// 16-byte piece of LDS per thread, without bank conflicts; by 256 threads with sixteen bins 1.6 us instead of 0.7.)
// Returns the thread's counts, of the bins from piece_bin() on.
__device__ __forceinline__ uint32_t piece_bin() { return (uint32_t)(kThBins - 4) - 4u * threadIdx.x; }
__device__ __forceinline__ uint4 pick_bin(uint32_t* hist, uint32_t need, uint32_t rank2, uint32_t* scratch, uint32_t* res) {
    static_assert(kThBins == 4 * kThThreads && kThThreads / 64 == 16, "16-byte pieces; one row of lanes holds the wavefronts' sums");
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    uint4* const h4 = reinterpret_cast<uint4*>(hist);
    const uint32_t piece = piece_bin() / 4u;
    const uint4 v = h4[piece];
    h4[piece] = make_uint4(0u, 0u, 0u, 0u);
    const uint32_t sum = v.x + v.y + v.z + v.w;
    const uint32_t inc = wave_incl_sum(sum);
    if (lane == 63) scratch[w] = inc;
    __syncthreads();
    // the wavefronts before this one: a lane each, added up in the first row of 16
    uint32_t cum = lane < w ? scratch[lane] : 0u;
    cum += dpp_fetch<0x111, 0xf>(cum);
    cum += dpp_fetch<0x112, 0xf>(cum);
    cum += dpp_fetch<0x114, 0xf>(cum);
    cum += dpp_fetch<0x118, 0xf>(cum);
    cum = (uint32_t)__builtin_amdgcn_readlane((int)cum, 15) + inc - sum;
    if ((cum < need && need <= cum + sum) || (cum < rank2 && rank2 <= cum + sum)) {
        const uint32_t c[4] = {v.w, v.z, v.y, v.x};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t bin = 4u * piece + 3u - (uint32_t)j;
            if (cum < need && need <= cum + c[j]) { res[0] = bin; res[1] = cum; res[3] = c[j]; }
            if (cum < rank2 && rank2 <= cum + c[j]) res[2] = bin;
            cum += c[j];
        }
    }
    __syncthreads();
    return v;
}

struct ThresholdShared {
    union {
        uint32_t hist[kThBins];
        long long acc[256];                            // per-exponent integer sums
    };
    uint32_t found[kThRanked];                         // the entries of the k-th entry's bin
    uint32_t ranks[kThRanked];
    uint32_t n_found;
    uint32_t scratch[kThThreads / 64];
    uint32_t res[2][4];
    uint32_t rank[3];                                  // the threshold, entries of the bin beyond it, and at or beyond it
    double dsum[kThThreads / 64];
    long long isum[kThThreads / 64];
    ListCounts counts;
    uint32_t spread;                                   // some kept entry is too far beyond the threshold for the fp64 sum
};

// Sum over the wavefronts' values v[0 .. kThThreads/64): every lane of the calling wavefront gets it.
__device__ __forceinline__ long long sum_of_waves(const long long* v) {
    const int lane = threadIdx.x & 63;
    return (long long)last_lane(wave_incl_sum((unsigned long long)(lane < kThThreads / 64 ? v[lane] : 0ll)));
}

// fp64 sum of exact per-exponent integers in a fixed order: lane l adds exponents 4l..4l+3 ascending,
// then a fixed tree; every lane of the calling wavefront gets it.
template <typename F>
__device__ __forceinline__ double sum_of_exponents(F at) {
    double v = 0.0;
#pragma nounroll
    for (int j = 0; j < 4; ++j) {
        const int ex = 4 * (int)(threadIdx.x & 63) + j;
        v += ldexp((double)at(ex), ex - 150);
    }
    return last_lane(wave_sum_f64(v));
}

// --------------------------------------------------------------------------
// One workgroup of 1024 threads per (tensor, side); `order` lists the tensors by decreasing size
// (null: as they come).  pass 0: every tensor no earlier kernel has finished or flagged; pass 1:
// tensors handed over (histogram route, or left by the streaming kernel).  sweeps: k_wide_count and
// k_wide_collect have run in this pass.  PAIRS: in the second pass of a call with the fused step, where lists
// that the streaming kernel has left are in pairs (pairs_of).
// Every workgroup runs its code once, and for most it is a chain of short dependent steps: 1.2 us to the
// counts, 1.3 to the list and its histogram, 0.8 to the bin, 0.5 for the second pass, 0.6 for the ranks, 0.7 to
// the end, whatever the list.  Long lists are bound by the LDS histogram (14 cycles per 64 keys) and by the
// fp64 sums: 10.2 us on 12,500 entries, 12.3 on 27,000, 18.6 on 60,000 (with the sweeps of k_wide_count and
// k_wide_collect before a workgroup that staged keys in LDS: 19 us in all on 27,000, 37 on 61,000).  Keys stay in
// registers between the passes where a list has up to sixteen per thread; longer ones are read again.  (Tried:
// 32 per thread, the next loads on their way during a batch, two copies of the histogram: no difference.)
// For k_emit_all: one thread calls running() on the way (behind the list's loads, which would wait for what it
// does) and done() when the state has been written.
// --------------------------------------------------------------------------
struct SideResult {
    bool ok;                                           // false: the lists cannot be used, or an invariant is violated
    uint32_t tau, itau, kc, raise;
    double mean;
};
template <bool PAIRS, typename Running, typename Done>
__device__ __forceinline__ void select_side(ThresholdShared& sh, const uint32_t item,
        const TensorDesc* __restrict__ desc, const uint32_t* __restrict__ order, TensorState* __restrict__ st,
        const unsigned long long* __restrict__ counters, const CandPtr cand, uint32_t* __restrict__ bitmap, const WideState* __restrict__ ws,
        uint32_t* __restrict__ whist, const long long* __restrict__ wacc, int pass, int sweeps, int carry, ResultBlock* __restrict__ result,
        Running running, Done done) {
    SBC_TS(1, 0);
    const int s = (int)(item & 1u), tid = threadIdx.x;
    const int t = order ? (int)order[item >> 1] : (int)(item >> 1);
    const TensorDesc d = desc[t];
    const uint32_t flags = st[t].flags;
    const uint32_t lo_key = st[t].lo_key[s], expect = st[t].expect[s];
    const int prev_side = st[t].side;
    {
        uint4* const z = reinterpret_cast<uint4*>(sh.hist);
        static_assert(kThBins == 4 * kThThreads, "four bins per thread");
        z[tid] = make_uint4(0u, 0u, 0u, 0u);
        if (tid < (int)kThRanked) { sh.found[tid] = 0u; sh.ranks[tid] = 0u; }
        if (tid < 8) (&sh.res[0][0])[tid] = 0xFFFFFFFFu;
        if (tid == 8) sh.spread = 0u;
        if (tid == 9) sh.n_found = 0u;
    }
    if (pass == 0 ? (flags & (kStInlineDone | kStDeferred | kStFailed)) != 0u : (flags & (kStExact | kStDeferred)) == 0u) {
        if (tid == 0) { running(); done(t, s, SideResult{false, 0u, 0u, 0u, 0u, 0.0}); }       // (not in k_emit_all)
        return;
    }
    count_list(sh.counts, d, st, counters, t, s, flags);
    __syncthreads();                                   // (and the histogram's counts are zero)
    SBC_TS(1, 1);
    const ListCounts counts = ListCounts::totals(sh.counts);
    if (lists_unusable(d, st, t, counts, pass, s == 0 && tid == 0, result)) {
        if (tid == 0) { running(); done(t, s, SideResult{false, 0u, 0u, 0u, 0u, 0.0}); }
        return;
    }
    const uint32_t full_cnt = counts.of(s);
    const uint32_t kc = kept_of_side(d, full_cnt);
    const bool pick = kc < full_cnt || !(d.flags & kDescSampled);      // else every candidate is kept

    // a wide tensor: the entries of the k-th entry's bin have been copied out, the others summed
    const uint32_t w2 = 2u * d.wide + (uint32_t)s;
    WideState wst;
    wst.ok = 0u;
    const bool swept = sweeps && (d.flags & kDescWide);
    if (swept) {
        wst = ws[w2];
        // (every workgroup of k_wide_collect has read the window's counts: they end the call clean)
        reinterpret_cast<uint4*>(whist + (size_t)w2 * kThBins)[tid] = make_uint4(0u, 0u, 0u, 0u);
    }
    const bool wide = wst.ok != 0u;
    // The list: this thread takes every step-th four of the `mine_cnt` entries from `list` on, starting with its own
    // (a list in segments: two wavefronts each, unless one of them is crowded: 21,000 kept entries all in one
    // segment 37.6 us with two wavefronts, 14.5 so; spread evenly 15).
    const uint32_t segs = wide ? 1u : counts.segs;
    CandPtr list = wide ? wide_list(d, bitmap, s) : cand + d.cand_off + (s ? d.cand_cap : 0u);
    uint32_t mine_cnt = wide ? wst.count : full_cnt, step_by = kThThreads, first = (uint32_t)tid;
    if (segs > 1u) {                                   // uniform
        uint3 share = make_uint3(uniform((uint32_t)tid >> 6) / 2u, uniform((uint32_t)tid >> 6) % 2u, 2u);
        if (__builtin_expect(counts.crowded != 0u, 0)) share = sh.counts.share_of(uniform((uint32_t)tid >> 6), kThThreads / 64u, full_cnt);
        mine_cnt = uniform(sh.counts.cnt[share.x]);
        list = list + seg_before(d, segs, share.x);
        step_by = share.z * 64u;
        first = share.y * 64u + (uint32_t)(tid & 63);
    }
    const uint32_t base = lo_key >> kThShift;
    // Sixteen keys of a thread at a time, in four loads that are in flight together; 0, which is the key of no
    // number, where there is none.  (The last four may read up to three keys beyond the list: the arrays have
    // room for them.)
    constexpr int kVecs = 4;
    const u32x4_any* __restrict__ vecs = reinterpret_cast<const u32x4_any*>(list.key);
    const u32x4_any* __restrict__ index_vecs = reinterpret_cast<const u32x4_any*>(list.key + list.to_idx);
    const bool pairs = PAIRS && (flags & kStDeferred);
    const uint2* const pair = pairs_of(cand, d.cand_off, s);
    const auto pair_at = [&](uint32_t i) { return pair[min(i, mine_cnt - 1u)]; };
    auto keys_at = [&](uint32_t p) -> u32x4_any {
        if constexpr (PAIRS)
            if (pairs) return u32x4_any{pair_at(4u * p).x, pair_at(4u * p + 1u).x, pair_at(4u * p + 2u).x, pair_at(4u * p + 3u).x};
        return vecs[p];
    };
    auto indexes_at = [&](uint32_t p) -> u32x4_any {
        if constexpr (PAIRS)
            if (pairs) return u32x4_any{pair_at(4u * p).y, pair_at(4u * p + 1u).y, pair_at(4u * p + 2u).y, pair_at(4u * p + 3u).y};
        return index_vecs[p];
    };
    const uint32_t fours = mine_cnt / 4u + (mine_cnt % 4u ? 1u : 0u);          // (so that no place passes 2^32)
    const uint32_t wave_first = uniform(first);        // (the wavefront's first lane's)
    u32x4_any held[kVecs];
    auto load = [&](uint32_t p0) {
#pragma unroll
        for (int j = 0; j < kVecs; ++j) {
            const uint32_t p = p0 + (uint32_t)j * step_by;
            held[j] = 0u;
            if (p < fours) held[j] = keys_at(p);
        }
#pragma unroll
        for (int j = 0; j < kVecs; ++j) {
            const uint32_t p = p0 + (uint32_t)j * step_by, left = mine_cnt - 4u * p;
            if (p < fours && left < 4u) {            // (one lane of a list)
                held[j].w = 0u;
                if (left <= 2u) held[j].z = 0u;
                if (left <= 1u) held[j].y = 0u;
            }
        }
    };
    const bool once = mine_cnt <= 4u * (uint32_t)kVecs * step_by;      // the keys stay in `held`
    auto for_fours = [&](bool again, auto f) {         // f(four keys, entries from the first lane's on) for the thread's share
        for (uint32_t w0 = wave_first, p0 = first; w0 < fours; w0 += (uint32_t)kVecs * step_by, p0 += (uint32_t)kVecs * step_by) {
            if (!again || !once) load(p0);
#pragma unroll
            for (int j = 0; j < kVecs; ++j) {
                const uint32_t w = w0 + (uint32_t)j * step_by;
                if (w < fours) f(held[j], mine_cnt - 4u * w);        // uniform
            }
        }
    };
    // The same from memory, entry by entry, for what is rare: f(key, index), of which the index is only there
    // for keys that need_index(key) names.  (Both arrays have room for the last four's.)  Short lists take the short
    // way: most are, and code that is fetched for the first time costs more than what it does (2.4 us on 64 entries).
    auto again = [&](auto need_index, auto f) {
        if (__builtin_expect(mine_cnt <= step_by, 1)) {                // uniform
            if (first < mine_cnt) {
                if constexpr (PAIRS)
                    if (pairs) { const uint2 e = pair[first]; f(e.x, e.y); return; }
                const uint32_t k = list.key[first];
                f(k, need_index(k) ? list.key[first + list.to_idx] : 0u);
            }
            return;
        }
#pragma nounroll
        for (uint32_t p0 = first; p0 < fours; p0 += 2u * step_by) {
            u32x4_any k[2], x[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) { const uint32_t p = p0 + (uint32_t)j * step_by; k[j] = keys_at(p < fours ? p : p0); }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t p = p0 + (uint32_t)j * step_by;
                x[j] = 0u;
                if (need_index(k[j].x) || need_index(k[j].y) || need_index(k[j].z) || need_index(k[j].w))
                    x[j] = indexes_at(p < fours ? p : p0);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint32_t p = p0 + (uint32_t)j * step_by, left = p < fours ? mine_cnt - 4u * p : 0u;
#pragma unroll
                for (uint32_t e = 0; e < 4u; ++e) if (e < left) f(k[j][e], x[j][e]);
            }
        }
    };
    auto no_index = [](uint32_t) { return false; };

    uint32_t tau = lo_key, itau = 0xFFFFFFFFu, keep = 0u, ties = 0u;
    // Filter key a following call may start from instead of sampling.  With the residual carried
    // over, the k-th entry sits at the edge of a cliff (everything above it has just been cut down
    // to about mu), so a margin in value below it lets a flood of entries pass, while a margin in
    // rank does not: the key is the lower edge of the window bin of this call's r-th most extreme
    // entry (carried_rank).  A call that started from a carried key sees how many entries its update
    // moved across it: `expect` were known to lie beyond it, less those the call before then sent.
    uint32_t next_bin = wide ? wst.next_rank_bin : 0xFFFFFFFFu;
    const bool net_known = pass == 0 && carry && expect != 0u && !swept;
    const uint32_t sent_before = prev_side == (s ? -1 : 1) ? d.k : 0u;
    const uint32_t rank2 = net_known ? carried_rank(d.k, (long long)full_cnt - ((long long)expect - (long long)sent_before))
                                     : carried_rank(d.k);
    // S, the sum of the kept values (negated on the negative side), is an fp64 sum that is exact in any
    // order, as long as no kept value reaches `limit` (else it is added up again from integers)
    double mine = 0.0;
    uint32_t limit = 0u, most = 0u;
    auto add = [&](uint32_t k, bool counts_in) {
        uint32_t x = counts_in ? k : 0u;
        asm("" : "+v"(x));                             // (chosen as 32 bits, not as the 64 that it is converted to)
        mine += (double)fabsf(__uint_as_float(x));
        most = max(most, k);                           // (what is not kept lies below the limit)
    };
    bool ok = true, placed = true;
    uint32_t need = kc, prefix = 0u, in_bin = 0u;
    if (wide) {
        need = wst.need; prefix = wst.prefix;
    } else if (pick) {
        // (the places without an entry are counted, too, in whatever bin the key 0 has, and taken out again)
        uint32_t empty = 0u;
        for_fours(false, [&](const u32x4_any& k, uint32_t left) {
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicAdd(&sh.hist[min((k[e] >> kThShift) - base, (uint32_t)(kThBins - 1))], 1u);
            empty += 256u - min(left, 256u);
        });
        if (empty && (tid & 63) == 0) atomicSub(&sh.hist[min(0u - base, (uint32_t)(kThBins - 1))], empty);
        __syncthreads();
        SBC_TS(1, 2);
        pick_bin(sh.hist, need, carry ? rank2 : 0u, sh.scratch, sh.res[0]);
        const uint32_t digit = uniform(sh.res[0][0]);
        next_bin = uniform(sh.res[0][2]);
        in_bin = uniform(sh.res[0][3]);
        prefix = base + digit;
        placed = digit < (uint32_t)(kThBins - 1);      // else beyond the window (uniform)
        if (placed) need -= uniform(sh.res[0][1]);
        SBC_TS(1, 3);
    }
    if (tid == 0) running();
    if (placed) {
        // the entries beyond the bin (if all are kept: every one, and there is no bin), and those in it
        const uint32_t from = pick ? prefix << kThShift : 0xFFFFF000u, beyond = pick ? from + (uint32_t)(kThBins - 1) : 0u;
        const bool few = !wide && in_bin <= kThRanked; // uniform
        limit = exact_limit(pick ? from : tau, kc);
        for_fours(pick && !wide, [&](const u32x4_any& k, uint32_t) {
            // (one test for four entries: those of the bin are few)
            if (min(min(k.x - from, k.y - from), min(k.z - from, k.w - from)) < (uint32_t)kThBins) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (k[e] - from < (uint32_t)kThBins) {
                        if (few) sh.found[atomicAdd(&sh.n_found, 1u)] = k[e];
                        else atomicAdd(&sh.hist[k[e] - from], 1u);
                    }
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) add(k[e], k[e] > beyond);
        });
        __syncthreads();
        SBC_TS(1, 4);
        if (few) {
            // (exactly in_bin of them.)  How many of the others each one has above it, and at least at it.
            auto both_of = [&](uint32_t me, uint32_t from_j, uint32_t to_j) {         // above in the low half, at least in the high half
                uint32_t both = 0u;
                for (uint32_t j = from_j; j < to_j; j += 4u) {         // (zeros behind the last one)
                    const uint4 o = *reinterpret_cast<const uint4*>(sh.found + j);
                    both += (o.x > me ? 1u : 0u) + (o.y > me ? 1u : 0u) + (o.z > me ? 1u : 0u) + (o.w > me ? 1u : 0u);
                    both += (o.x >= me ? 65536u : 0u) + (o.y >= me ? 65536u : 0u) + (o.z >= me ? 65536u : 0u) + (o.w >= me ? 65536u : 0u);
                }
                return both;
            };
            const bool shared = in_bin > 16u;          // uniform
            if (shared) {
                // groups of one, two or four wavefronts, which hold all of them, take a share of the others each
                const uint32_t lg = in_bin <= 64u ? 0u : in_bin <= 128u ? 1u : 2u, wv = uniform((uint32_t)tid >> 6), g = wv >> lg;
                const uint32_t i = ((wv & ((1u << lg) - 1u)) << 6) + (uint32_t)(tid & 63);
                const uint32_t share = ((in_bin >> (4u - lg)) + 4u) & ~3u;            // (times the number of groups: in_bin at the least)
                if (i < in_bin) {
                    const uint32_t both = both_of(sh.found[i], g * share, min(in_bin, (g + 1u) * share));
                    if (both) atomicAdd(&sh.ranks[i], both);
                }
                __syncthreads();
            }
            if ((uint32_t)tid < in_bin) {
                const uint32_t me = sh.found[tid], both = shared ? sh.ranks[tid] : both_of(me, 0u, in_bin);
                const uint32_t above = both & 0xFFFFu, at_least = both >> 16;
                if (above < need && need <= at_least) { sh.rank[0] = me; sh.rank[1] = above; sh.rank[2] = at_least; }   // (equal entries write the same)
                if (at_least < need) mine += (double)__uint_as_float(me & 0x7FFFFFFFu);
            }
        } else if (pick) {
            const uint4 in_piece = pick_bin(sh.hist, need, 0u, sh.scratch, sh.res[1]);
            const uint32_t digit = uniform(sh.res[1][0]);
            ok = digit != 0xFFFFFFFFu;
            tau = from | (digit & (uint32_t)(kThBins - 1));
            ties = uniform(sh.res[1][3]);
            need -= uniform(sh.res[1][1]);
            // the bin's entries beyond tau, from their counts
            const uint32_t counted[4] = {in_piece.x, in_piece.y, in_piece.z, in_piece.w};
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j) {
                const uint32_t k = from + piece_bin() + j;
                if (counted[j] != 0u && k > tau) mine += (double)counted[j] * (double)__uint_as_float(k & 0x7FFFFFFFu);
            }
        }
        if (limit == 0u || most >= limit) sh.spread = 1u;
        mine = wave_sum_f64(mine);
        if ((tid & 63) == 63) sh.dsum[tid >> 6] = mine;
        __syncthreads();
        if (few && pick) { tau = uniform(sh.rank[0]); need -= uniform(sh.rank[1]); ties = uniform(sh.rank[2]) - uniform(sh.rank[1]); }
        SBC_TS(1, 5);
    }
    if (pick) {
        keep = need;
        if (__builtin_expect(!placed || (ok && keep < ties), 0)) {     // uniform
            // tau from the top, for what the window cannot place (rare); then, if fewer than all entries equal
            // to tau are kept, the highest index kept among them: the keep-th largest complemented index.
            // 12 + 12 + 8 bits at a time.
#pragma nounroll
            for (int mode = placed ? 1 : 0; mode < 2 && ok; ++mode) {
                uint32_t r = mode ? keep : kc, found = 0u, same = 0u;
                if (mode && keep >= ties) break;
#pragma nounroll
                for (int level = 0; level < 3 && ok; ++level) {
                    const int shift = level == 0 ? 20 : level == 1 ? 8 : 0, bits = level == 2 ? 8 : 12;
                    __syncthreads();                   // the results of the step before have been read
                    if (tid < 4) sh.res[0][tid] = 0xFFFFFFFFu;
                    again([&](uint32_t k) { return mode && k == tau; }, [&](uint32_t k, uint32_t idx) {
                        if (mode && k != tau) return;
                        const uint32_t v = mode ? ~idx : k;
                        if (level == 0 || (v >> (shift + bits)) == found) atomicAdd(&sh.hist[(v >> shift) & ((1u << bits) - 1u)], 1u);
                    });
                    __syncthreads();
                    pick_bin(sh.hist, r, 0u, sh.scratch, sh.res[0]);
                    const uint32_t digit = uniform(sh.res[0][0]);
                    if (digit == 0xFFFFFFFFu) { ok = false; break; }   // uniform
                    r -= uniform(sh.res[0][1]);
                    same = uniform(sh.res[0][3]);
                    found = (found << bits) | digit;
                }
                if (mode) itau = ~found;
                else { tau = found; keep = r; ties = same; }
            }
        }
        if (!ok) {                                     // uniform; cannot happen
            if (tid == 0) {
                atomicOr(&result->err, kErrInternal);
                done(t, s, SideResult{false, 0u, 0u, 0u, 0u, 0.0});
            }
            return;
        }
    }
    if (!placed) {                                     // uniform: added up here, with the threshold that was found at last
        limit = exact_limit(tau, kc);
        again(no_index, [&](uint32_t k, uint32_t) { add(k, k > tau); });
        if (limit == 0u || most >= limit) sh.spread = 1u;
        mine = wave_sum_f64(mine);
        if ((tid & 63) == 63) sh.dsum[tid >> 6] = mine;
        __syncthreads();
    }
    const uint32_t e_tau = max((tau >> 23) & 0xFFu, 1u);               // (tau's fp32 exponent, if it is positive)
    double S = last_lane(wave_sum_f64((tid & 63) < kThThreads / 64 ? sh.dsum[tid & 63] : 0.0)) +
               (double)keep * (double)__uint_as_float(tau & 0x7FFFFFFFu);
    if (__builtin_expect(uniform(sh.spread) != 0u, 0)) {        // uniform
        // Values of both signs, or too far apart: integers, each at the scale of tau's exponent while it fits
        // 64 bits, else one integer per exponent (all read from memory once more).
        const bool common = kc <= 32768u && tau > 0x80000000u, all = !pick;
        __syncthreads();
        if (tid < 256) sh.acc[tid] = 0ll;
        __syncthreads();
        long long scaled = 0ll;
        again([&](uint32_t k) { return k == tau; }, [&](uint32_t k, uint32_t idx) {
            if (!all && !cand_kept(k, idx, tau, itau)) return;
            uint32_t ex;
            const long long m = signed_mantissa(k, s, ex);
            if (common && ex - e_tau <= 24u) scaled += m << (ex - e_tau);
            else if (m != 0ll) atomicAdd(reinterpret_cast<unsigned long long*>(&sh.acc[ex]), (unsigned long long)m);
        });
        const unsigned long long wave_sum = wave_incl_sum((unsigned long long)scaled);
        if ((tid & 63) == 63) sh.isum[tid >> 6] = (long long)wave_sum;
        __syncthreads();
        S = sum_of_exponents([&](int ex) { return sh.acc[ex]; }) + ldexp((double)sum_of_waves(sh.isum), (int)e_tau - 150);
    }
    if (wide) {
        // what k_wide_collect has added up: slot 255 at the scale of the bin's exponent (tau's), which holds
        // all but the entries too far beyond the bin; those are in their exponents' slots
        const long long* __restrict__ g = wacc + (size_t)w2 * 256;
        S += sum_of_exponents([&](int ex) { return ex < 255 ? g[ex] : 0ll; }) + ldexp((double)g[255], (int)e_tau - 150);
    }
    SBC_TS(1, 6);                                      // sum done
    if (tid != 0) return;
    const double mean = S / (double)kc;
    st[t].cand_seen[s] = full_cnt;                     // (inspection only)
    st[t].tau[s] = tau;
    st[t].itau[s] = itau;
    st[t].kc[s] = kc;
    st[t].S[s] = S;
    st[t].mean[s] = mean;
    uint32_t raise = 0u;
    if (carry && pick) {
        const bool ranked = next_bin != 0xFFFFFFFFu;
        uint32_t next = (base + next_bin) << kThShift;
        if (__builtin_expect(!ranked, 0)) {
            // The list does not reach that rank.  A guess at what lies below it may be far off, and for a tensor
            // that keeps many entries a flood costs most (data of two scales: half the tensor, a call of 2.4 ms):
            // at most a tenth below the key of this call, then.  (That alone: lists of 118,000 now and then
            // where they have 74,000 with the guess.)
            const uint32_t tenth = lowered_key(lo_key, 0.1f);
            next = swept ? tenth : extrapolated_key(tau, lo_key, d.k, rank2, d.n, full_cnt);
            if (d.flags & kDescWide) next = max(next, tenth);
        }
        st[t].lo_key[s] = next;
        st[t].expect[s] = ranked ? rank2 : 0u;
    }
    // many times more candidates than needed: the next call should estimate its keys afresh
    if (full_cnt > loose_limit(d.k, d.n)) raise |= kErrLoose;
    if (wide) raise |= kErrWide;
    if ((d.flags & kDescWide) && full_cnt > long_list(d.k)) raise |= kErrLong;
    if (raise) atomicOr(&result->err, raise);
    done(t, s, SideResult{true, tau, itau, kc, raise, mean});
    SBC_TS(1, 7);
}

template <bool PAIRS>
__global__ __launch_bounds__(kThThreads, 8) void k_threshold(
        const TensorDesc* __restrict__ desc, const uint32_t* __restrict__ order, TensorState* __restrict__ st,
        const unsigned long long* __restrict__ counters, const CandPtr cand, uint32_t* __restrict__ bitmap, const WideState* __restrict__ ws,
        uint32_t* __restrict__ whist, const long long* __restrict__ wacc, int pass, int sweeps, int carry, ResultBlock* __restrict__ result) {
    __shared__ __attribute__((aligned(16))) ThresholdShared sh;
    select_side<PAIRS>(sh, blockIdx.x, desc, order, st, counters, cand, bitmap, ws, whist, wacc, pass, sweeps, carry, result,
                       []() {}, [](int, int, const SideResult&) {});
}

// --------------------------------------------------------------------------
// Tensors that keep very many entries (lists too long for one workgroup).  grid
// (workgroups, 2 x wide tensors); a list gets only as many of the workgroups as it has use for: a
// workgroup adds its counts to the shared histogram bin by bin, and those atomics cost more than
// the reading when every workgroup has few entries per bin.
// --------------------------------------------------------------------------
// Entries that keep a workgroup of a sweep busy.  Eight workgroups take a list of up to 147455 entries, each
// a segment, sixteen one of up to 278527 and so on: what a sweep over short lists costs is above all the workgroups'
// additions to the shared histogram (20 lists by 32 workgroups with 1536 bins each: 8.5 us, by 8: 2.7 us).  3.9e6
// entries a side (1.5e9-entry tensor): 15 + 31 us (25 + 34 with a load of a thread in flight at a time instead of
// eight or four; 69 + 62 with workgroups of 256 threads and 4096 entries).
constexpr uint32_t kWidePerWorkgroup = 16384, kWideFew = 8;
constexpr uint32_t kWideFound = 512;                   // entries of the k-th entry's bin that a workgroup collects in LDS

__device__ __forceinline__ uint32_t wide_workgroups(uint32_t cnt) {
    static_assert(kWideFew % kSegs == 0, "the same number for every segment");
    const uint32_t want = max((cnt / kWidePerWorkgroup + kWideFew - 1u) / kWideFew * kWideFew, kWideFew);
    return min(want, gridDim.x);                       // (gridDim.x: a multiple of kWideFew)
}

// The lists can be selected from, and the subsampled variant does not keep all of this one.
__device__ __forceinline__ bool wide_applies(const TensorDesc& d, const ListCounts& c) {
    if (c.over) return false;
    return (d.flags & kDescSampled) ? c.p >= 1u && c.n >= 1u : c.p >= d.k && c.n >= d.k;
}

// f(key, place in the list) for a thread's share of a side's list, which nb of the workgroups take: nb / segs of
// each segment, or, where a segment is crowded, each its part of the list as a whole (42,000 kept entries all in
// one segment: both sweeps 63 us the first way, 21 the second).
template <int UNROLL, typename F>
__device__ __forceinline__ void sweep_list(const TensorDesc& d, const ListCounts& c, uint32_t segs, int s, uint32_t nb, const CandPtr cand, F f) {
    const CandPtr whole = cand + d.cand_off + (s ? d.cand_cap : 0u);
    uint32_t g = blockIdx.x % segs, last = g + 1u, lo = 0u, hi = 0u;
    const bool crowded = uniform(c.crowded) != 0u;
    if (crowded) {
        const uint32_t all = uniform(c.of(s)), per = all / nb + 1u;
        g = 0u; last = segs;
        lo = (uint32_t)min((uint64_t)blockIdx.x * per, (uint64_t)all);
        hi = (uint32_t)min((uint64_t)lo + per, (uint64_t)all);
    }
#pragma nounroll
    for (; g < last; ++g) {
        uint64_t from = (uint64_t)(blockIdx.x / segs) * kWideThreads, stride = (uint64_t)(nb / segs) * kWideThreads, to = uniform(c.cnt[g]);
        if (crowded) {
            const uint2 part = c.part_of(g, lo, hi);
            from = part.x; to = part.y; stride = kWideThreads;
        }
        const CandPtr list = whole + seg_before(d, segs, g);
#pragma nounroll
        for (uint64_t i0 = from + threadIdx.x; i0 < to; i0 += UNROLL * stride) {
            uint32_t key[UNROLL];                      // (loads in flight together)
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) { const uint64_t i = i0 + u * stride; key[u] = list.key[i < to ? i : i0]; }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) { const uint64_t i = i0 + u * stride; if (i < to) f(key[u], list + i); }
        }
    }
}

// k_wide_count: window histogram of a side's list.  (Counting where the streaming kernel stores the
// candidates would save this sweep, but every count would be an atomic on memory that all
// compute-unit groups share, and those on one bin queue up for about half a microsecond each: four
// times the streaming kernel's time on Gaussian data.)
__global__ __launch_bounds__(kWideThreads) void k_wide_count(
        const TensorDesc* __restrict__ desc, const WideIds wide_ids, const TensorState* __restrict__ st,
        const unsigned long long* __restrict__ counters, const CandPtr cand, uint32_t* __restrict__ whist, long long* __restrict__ wacc,
        WideState* __restrict__ ws) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kThBins];
    __shared__ ListCounts counts_sh;
    const int w = blockIdx.y >> 1, s = blockIdx.y & 1, tid = threadIdx.x;
    const int t = (int)wide_ids.id[w];
    const TensorDesc d = desc[t];
    count_list(counts_sh, d, st, counters, t, s, 0u);
    const uint32_t base = st[t].lo_key[s] >> kThShift;
    uint4* const h4 = reinterpret_cast<uint4*>(hist);
#pragma unroll
    for (int i = 0; i < kThBins / 4 / kWideThreads; ++i) h4[i * kWideThreads + tid] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const ListCounts counts = ListCounts::totals(counts_sh);
    const uint32_t cnt = counts.of(s);
    if (blockIdx.x == 0) {                             // the call before this one has read its sums
        if (tid < 256) wacc[(size_t)blockIdx.y * 256 + tid] = 0ll;
        if (tid == 0) {
            WideState z;
            z.ok = 0u; z.prefix = 0u; z.need = 0u; z.count = 0u; z.next_rank_bin = 0xFFFFFFFFu;
            z.pad[0] = z.pad[1] = z.pad[2] = 0u;
            ws[blockIdx.y] = z;
        }
    }
    if (!wide_applies(d, counts) || kept_of_side(d, cnt) == cnt) return;      // uniform
    const uint32_t nb = wide_workgroups(cnt);
    if (blockIdx.x >= nb) return;
    sweep_list<8>(d, counts_sh, counts.segs, s, nb, cand, [&](uint32_t key, const CandPtr) { atomicAdd(&hist[window_bin(key, base)], 1u); });
    __syncthreads();
    uint32_t* __restrict__ g = whist + (size_t)blockIdx.y * kThBins;
    for (int i = tid; i < kThBins; i += kWideThreads) {
        const uint32_t v = hist[i];
        if (v) atomicAdd(&g[i], v);
    }
}

// k_wide_collect: every workgroup finds the bin of the side's k-th entry from the window's counts (all
// of them at once from the same counts, instead of a launch of one workgroup in between); then the
// entries of that bin are copied out and those beyond it are added up.
__global__ __launch_bounds__(kWideThreads) void k_wide_collect(
        const TensorDesc* __restrict__ desc, const WideIds wide_ids, const TensorState* __restrict__ st,
        const unsigned long long* __restrict__ counters, const CandPtr cand, uint32_t* __restrict__ bitmap, const uint32_t* __restrict__ whist,
        long long* __restrict__ wacc, WideState* __restrict__ ws) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kThBins];
    __shared__ long long acc[256];
    __shared__ uint2 found[kWideFound];
    __shared__ uint32_t scratch[kWideThreads / 64], res[4], n_found, found_at;
    __shared__ ListCounts counts_sh;
    const int w = blockIdx.y >> 1, s = blockIdx.y & 1, tid = threadIdx.x;
    const int t = (int)wide_ids.id[w];
    // (the window's counts are asked for together with the descriptor and the state, before those say
    // whether they are needed: one round trip to memory less)
    uint4 mine[kThBins / 4 / kWideThreads];
    {
        const uint4* __restrict__ g4 = reinterpret_cast<const uint4*>(whist + (size_t)blockIdx.y * kThBins);
#pragma unroll
        for (int i = 0; i < kThBins / 4 / kWideThreads; ++i) mine[i] = g4[i * kWideThreads + tid];
    }
    const TensorDesc d = desc[t];
    count_list(counts_sh, d, st, counters, t, s, 0u);
    const uint32_t base = st[t].lo_key[s] >> kThShift;
#pragma unroll
    for (int i = 0; i < kThBins / 4 / kWideThreads; ++i) reinterpret_cast<uint4*>(hist)[i * kWideThreads + tid] = mine[i];
    if (tid < 256) acc[tid] = 0ll;
    if (tid < 4) res[tid] = 0xFFFFFFFFu;
    if (tid == 4) n_found = 0u;
    __syncthreads();
    const ListCounts counts = ListCounts::totals(counts_sh);
    if (!wide_applies(d, counts)) return;              // k_threshold flags the tensor
    const uint32_t cnt = counts.of(s), nb = wide_workgroups(cnt);
    if (blockIdx.x >= nb) return;
    const uint32_t kc = kept_of_side(d, cnt);
    const bool all = (d.flags & kDescSampled) && kc == cnt;
    uint32_t prefix = 0u;
    if (!all) {
        pick_bin(hist, kc, carried_rank(kc), scratch, res);
        const uint32_t digit = uniform(res[0]);
        // beyond the window, or more entries in the bin than there is room for (equal values): k_threshold
        // then works on the whole list
        if (digit >= (uint32_t)(kThBins - 1) || res[3] > wide_room(d)) {       // uniform
            if (blockIdx.x == 0 && tid == 0) ws[blockIdx.y].next_rank_bin = res[2];
            return;
        }
        prefix = base + digit;
        if (blockIdx.x == 0 && tid == 0) {             // (count: raised by atomics below, not read here)
            ws[blockIdx.y].prefix = prefix;
            ws[blockIdx.y].need = kc - res[1];
            ws[blockIdx.y].next_rank_bin = res[2];
        }
    }
    if (blockIdx.x == 0 && tid == 0) ws[blockIdx.y].ok = 1u;
    const CandPtr out = wide_list(d, bitmap, s);
    const uint32_t room = wide_room(d);
    const uint32_t from = all ? st[t].lo_key[s] : prefix << kThShift, limit = exact_limit(from, kc);
    double near = 0.0;
    sweep_list<4>(d, counts_sh, counts.segs, s, nb, cand, [&](uint32_t key, const CandPtr entry) {
        const uint32_t v = key >> kThShift;
        if (all || v > prefix) {
            if (key < limit) {
                near += (double)__uint_as_float(key & 0x7FFFFFFFu);
            } else {
                uint32_t ex;
                const long long m = signed_mantissa(key, s, ex);
                if (m != 0ll && ex < 255u) atomicAdd(reinterpret_cast<unsigned long long*>(&acc[ex]), (unsigned long long)m);
            }
        } else if (v == prefix) {
            // (a workgroup's few go out together: one atomic on the shared counter instead of one each,
            // which queue up there for about 60 ns apiece)
            const uint32_t q = atomicAdd(&n_found, 1u);
            const uint2 e = entry.get(0);
            if (q < kWideFound) found[q] = e;
            else {
                const uint32_t at = atomicAdd(&ws[blockIdx.y].count, 1u);
                if (at < room) out.put(at, e.x, e.y);
            }
        }
    });
    near = wave_sum_f64(near);
    if ((tid & 63) == 63 && near != 0.0) {
        // (an integer at the scale of from's exponent, below 2^53)
        const int e = (int)max((from >> 23) & 0xFFu, 1u);
        atomicAdd(reinterpret_cast<unsigned long long*>(&acc[255]), (unsigned long long)(long long)ldexp(near, 150 - e));
    }
    __syncthreads();
    const uint32_t mine_found = min(n_found, kWideFound);
    if (mine_found) {                                  // uniform
        if (tid == 0) found_at = atomicAdd(&ws[blockIdx.y].count, mine_found);
        __syncthreads();
        for (uint32_t i = tid; i < mine_found; i += kWideThreads)
            if (found_at + i < room) out.put(found_at + i, found[i].x, found[i].y);
    }
    const long long v = tid < 256 ? acc[tid] : 0ll;
    if (v != 0ll) atomicAdd(reinterpret_cast<unsigned long long*>(&wacc[(size_t)blockIdx.y * 256 + tid]), (unsigned long long)v);
}

}  // namespace sbc
