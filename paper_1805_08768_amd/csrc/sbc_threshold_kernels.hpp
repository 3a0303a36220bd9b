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
// A side is selected in two counting passes over its list: the leading 20 key bits in a window of
// two octaves above the filter key, then the other 12 bits of the entries in the k-th entry's bin.
// That is exact whatever the ties (equal values are one bin of the second pass).  Sums are exact
// integers rounded once to fp64 (or one integer per fp32 exponent where the values spread too far).
#pragma once

#include "sbc_device.hpp"

namespace sbc {

constexpr int kThThreads = 1024;
constexpr int kThShift = 12;                              // low key bits: the second pass's bins
constexpr int kThBins = 1 << kThShift;                    // bins of either pass; 2048 of the first per octave
constexpr uint32_t kThMaxStaged = 24576;                  // most keys of a list that LDS holds; longer lists are read from
                                                          // memory in every pass

// Keys of a list that k_threshold stages for a call whose tensors keep at most kmax entries per side
// (those with sweeps of their own aside: of theirs, one bin's entries): lists are about 3 k, up to 4 k,
// on carried keys.  Calls of many tensors want two workgroups on a compute unit.
__host__ inline uint32_t threshold_staged(uint32_t kmax, bool any_wide) {
    const uint64_t want = (4ull * kmax + 512ull + 255ull) / 256ull * 256ull, least = any_wide ? 8192ull : 2048ull;
    return (uint32_t)(want < least ? least : want > kThMaxStaged ? kThMaxStaged : want);
}

constexpr int kWideThreads = 256;        // sweeps over the lists of tensors that keep very many entries
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
__device__ __forceinline__ uint2* wide_list(const TensorDesc& d, uint32_t* bitmap, int s) {
    return reinterpret_cast<uint2*>(bitmap + (uint64_t)d.chunk0 * kChunkWords) + (s ? wide_room(d) : 0u);
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

// What a tensor's candidate counts rule out before any selection: true if the tensor cannot be
// selected from its lists (the thread with `lead` set has then flagged it, for the histogram route
// or as an error).
__device__ __forceinline__ bool lists_unusable(const TensorDesc& d, TensorState* __restrict__ st, int t, uint32_t cnt_p,
                                               uint32_t cnt_n, int pass, bool lead, ResultBlock* __restrict__ result) {
    const bool sampled = (d.flags & kDescSampled) != 0u;
    if (cnt_p > d.n || cnt_n > d.n || (sampled && (cnt_p == 0u || cnt_n == 0u))) {
        // (a sampled threshold is the key of an entry of the tensor, so that entry is a candidate)
        if (lead) { st[t].flags = kStFailed; atomicOr(&result->err, kErrInternal); }
        return true;
    }
    if (cnt_p > d.cand_cap || cnt_n > d.cand_cap) {
        // compact context: more candidates than a list holds (nothing was stored beyond its end).  The
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
    const uint32_t v = key >> kThShift;
    const uint32_t o = v >= base ? v - base : 0u;      // (no candidate lies below its filter key)
    return o < (uint32_t)(kThBins - 1) ? o : (uint32_t)(kThBins - 1);
}

// Walking the kThBins counts of hist (LDS) from the top bin down: the bin at which the running
// count reaches need (res[0]; 0xFFFFFFFF if it never does), the count before it (res[1]), the bin's
// own count (res[3]), and the bin at which the running count reaches rank2 (res[2], or 0xFFFFFFFF;
// rank2 = 0 looks for none).  res[0] and res[2] must hold 0xFFFFFFFF when the first barrier is
// reached.  The counts are zero again afterwards.  c: the calling thread's counts, of the bins
// kThBins-1 - (threadIdx * size), downwards.  Two barriers.
template <int NT>
__device__ __forceinline__ void pick_bin(uint32_t* hist, uint32_t need, uint32_t rank2, uint32_t* scratch, uint32_t* res,
                                         uint32_t (&c)[kThBins / NT]) {
    constexpr int PER = kThBins / NT;
    static_assert(PER % 4 == 0 && NT / 64 <= 16, "16-byte pieces; one row of lanes holds the wavefronts' sums");
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    uint4* const h4 = reinterpret_cast<uint4*>(hist);
    uint32_t sum = 0u;
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {
        const int at = kThBins / 4 - 1 - (tid * (PER / 4) + q);
        const uint4 v = h4[at];
        h4[at] = make_uint4(0u, 0u, 0u, 0u);
        c[4 * q] = v.w; c[4 * q + 1] = v.z; c[4 * q + 2] = v.y; c[4 * q + 3] = v.x;
        sum += v.x + v.y + v.z + v.w;
    }
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
        const uint32_t top = (uint32_t)(kThBins - 1 - tid * PER);
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (cum < need && need <= cum + c[j]) { res[0] = top - (uint32_t)j; res[1] = cum; res[3] = c[j]; }
            if (cum < rank2 && rank2 <= cum + c[j]) res[2] = top - (uint32_t)j;
            cum += c[j];
        }
    }
    __syncthreads();
}

struct ThresholdShared {
    union {
        uint32_t hist[kThBins];
        long long acc[256];                            // per-exponent integer sums
    };
    uint32_t scratch[kThThreads / 64];
    uint32_t res[2][4];
    double dsum[kThThreads / 64];
    long long isum[kThThreads / 64];
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
// tensors handed over (histogram route, or left by the streaming kernel).
// The keys of a list of up to `staged` candidates are copied to LDS (the index is only read, from
// memory, for entries equal to the threshold if some of them are dropped).  The kernel is a chain of
// short dependent steps and every workgroup runs its code once, from a cold instruction cache: a
// tensor with 64 entries takes as long as one with 10,000 candidates, and what helps is less code.
// So both counting passes share theirs, loops stay rolled, and what is rare stands at the end (34 KB of
// unrolled code with the keys in registers: 18 us on 161 tensors of 25.6e6 entries at p = 0.001, 12.9
// us on one of 4.2e6; this form, 14 KB: 10.6 and 9.4 us; 8192-candidate lists take 8.4 us, 64 entries 5.5).
// Two workgroups fit a compute unit (64 KiB of LDS each at p = 0.001, at most 64 registers).
// --------------------------------------------------------------------------
__global__ __launch_bounds__(kThThreads, 8) void k_threshold(
        const TensorDesc* __restrict__ desc, const uint32_t* __restrict__ order, TensorState* __restrict__ st,
        const uint2* __restrict__ cand, uint32_t* __restrict__ bitmap, const WideState* __restrict__ ws,
        uint32_t* __restrict__ whist, const long long* __restrict__ wacc, int pass, int carry, uint32_t staged, ResultBlock* __restrict__ result) {
    __shared__ __attribute__((aligned(16))) ThresholdShared sh;
    extern __shared__ uint32_t keys[];                 // `staged` of them
    SBC_TS(1, 0);
    const int s = (int)(blockIdx.x & 1u), tid = threadIdx.x;
    const int t = order ? (int)order[blockIdx.x >> 1] : (int)(blockIdx.x >> 1);
    const TensorDesc d = desc[t];
    const uint32_t flags = st[t].flags;
    const uint32_t cnt_p = st[t].cand_cnt[0], cnt_n = st[t].cand_cnt[1];
    const uint32_t lo_key = st[t].lo_key[s], expect = st[t].expect[s];
    const int prev_side = st[t].side;
    {
        uint4* const z = reinterpret_cast<uint4*>(sh.hist);
        static_assert(kThBins == 4 * kThThreads, "four bins per thread");
        z[tid] = make_uint4(0u, 0u, 0u, 0u);
        if (tid < 8) (&sh.res[0][0])[tid] = 0xFFFFFFFFu;
        if (tid == 8) sh.spread = 0u;
    }
    if (pass == 0 ? (flags & (kStInlineDone | kStDeferred | kStFailed)) != 0u : (flags & (kStExact | kStDeferred)) == 0u) return;
    if (lists_unusable(d, st, t, cnt_p, cnt_n, pass, s == 0 && tid == 0, result)) return;
    const uint32_t full_cnt = s ? cnt_n : cnt_p;
    const uint32_t kc = kept_of_side(d, full_cnt);
    const bool pick = kc < full_cnt || !(d.flags & kDescSampled);      // else every candidate is kept

    // a wide tensor: the entries of the k-th entry's bin have been copied out, the others summed
    const uint32_t w2 = 2u * d.wide + (uint32_t)s;
    WideState wst;
    wst.ok = 0u;
    if (pass == 0 && (d.flags & kDescWide)) {
        wst = ws[w2];
        // (every workgroup of k_wide_collect has read the window's counts: they end the call clean)
        reinterpret_cast<uint4*>(whist + (size_t)w2 * kThBins)[tid] = make_uint4(0u, 0u, 0u, 0u);
    }
    const bool wide = wst.ok != 0u;
    const uint2* __restrict__ list = wide ? wide_list(d, bitmap, s) : cand + d.cand_off + (s ? d.cand_cap : 0u);
    const uint32_t cnt = wide ? wst.count : full_cnt;
    const uint32_t base = lo_key >> kThShift;
    const bool in_lds = cnt <= staged;
    __syncthreads();                                   // the counts are zero
    if (in_lds) {
        // eight loads of a thread in flight at a time; the window's counts in the same sweep
        const uint32_t below = pick && !wide ? (uint32_t)kThBins : 0u;
        for (uint32_t i0 = tid; i0 < cnt; i0 += 8u * kThThreads) {
            uint32_t x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) { const uint32_t i = i0 + (uint32_t)j * kThThreads; x[j] = list[i < cnt ? i : 0u].x; }
#pragma unroll
            for (int j = 0; j < 8; ++j) { 
                const uint32_t i = i0 + (uint32_t)j * kThThreads;
                if (i < cnt) {
                    keys[i] = x[j];
                    const uint32_t o = window_bin(x[j], base);
                    if (o < below) atomicAdd(&sh.hist[o], 1u);
                }
            }
        }
    }
    auto stream = [&](auto f) {                        // f(entry) for this thread's share of the list in memory
#pragma unroll 4
        for (uint32_t i = tid; i < cnt; i += kThThreads) f(list[i]);
    };
    auto for_keys = [&](auto f) {                      // f(key): a thread sees the keys it has staged itself
        if (in_lds) {
#pragma unroll 4
            for (uint32_t i = tid; i < cnt; i += kThThreads) f(keys[i]);
        } else {
            stream([&](const uint2& e) { f(e.x); });
        }
    };
    SBC_TS(1, 1);                                      // list read

    uint32_t tau = lo_key, itau = 0xFFFFFFFFu, keep = 0u, ties = 0u;
    // Filter key a following call may start from instead of sampling.  With the residual carried
    // over, the k-th entry sits at the edge of a cliff (everything above it has just been cut down
    // to about mu), so a margin in value below it lets a flood of entries pass, while a margin in
    // rank does not: the key is the lower edge of the window bin of this call's r-th most extreme
    // entry (carried_rank).  A call that started from a carried key sees how many entries its update
    // moved across it: `expect` were known to lie beyond it, less those the call before then sent.
    uint32_t next_bin = wide ? wst.next_rank_bin : 0xFFFFFFFFu;
    const bool net_known = pass == 0 && carry && expect != 0u && !(d.flags & kDescWide);
    const uint32_t sent_before = prev_side == (s ? -1 : 1) ? d.k : 0u;
    const uint32_t rank2 = net_known ? carried_rank(d.k, (long long)full_cnt - ((long long)expect - (long long)sent_before))
                                     : carried_rank(d.k);
    // S, the sum of the kept values (negated on the negative side), is an fp64 sum that is exact in any
    // order, as long as no kept value reaches `limit` (else it is added up again from integers)
    double mine = 0.0;
    uint32_t limit = 0u;
    auto add = [&](uint32_t k) {
        mine += (double)__uint_as_float(k & 0x7FFFFFFFu);
        if (k >= limit) sh.spread = 1u;
    };
    bool ok = true, placed = true;
    if (pick) {
        uint32_t need = kc, prefix = 0u, c[kThBins / kThThreads];
        if (wide) { need = wst.need; prefix = wst.prefix; }
#pragma nounroll
        for (int step = wide ? 1 : 0; step < 2; ++step) {
            // step 0: leading bits, in the window; step 1: the other bits of the entries in the bin `prefix`,
            // and the sum of the entries beyond it
            const uint32_t from = step ? prefix << kThShift : base, cap = step ? 0xFFFFFFFFu : (uint32_t)(kThBins - 1);
            const uint32_t beyond = step ? from + (uint32_t)(kThBins - 1) : 0xFFFFFFFFu;
            const int shift = step ? 0 : kThShift;
            limit = exact_limit(from, kc);
            if (step || !in_lds) for_keys([&](uint32_t k) {            // (lists in LDS: counted when they were read)
                const uint32_t o = min((k >> shift) - from, cap);
                if (o < (uint32_t)kThBins) atomicAdd(&sh.hist[o], 1u);
                else if (k > beyond) add(k);
            });
            __syncthreads();
            SBC_TS(1, 2 + 2 * step);
            uint32_t* const r = sh.res[step];
            pick_bin<kThThreads>(sh.hist, need, carry && !step ? rank2 : 0u, sh.scratch, r, c);
            const uint32_t digit = r[0];
            if (step == 0) {
                next_bin = r[2];
                if (digit >= (uint32_t)(kThBins - 1)) { placed = false; break; }   // beyond the window (uniform)
                prefix = base + digit;
            } else {
                ok = digit != 0xFFFFFFFFu;
                tau = (prefix << kThShift) | (digit & (uint32_t)(kThBins - 1));
                ties = r[3];
                // the bin's entries beyond tau, from their counts
#pragma unroll
                for (int j = 0; j < kThBins / kThThreads; ++j) {
                    const uint32_t k = from + (uint32_t)(kThBins - 1 - tid * (kThBins / kThThreads) - j);
                    if (c[j] != 0u && k > tau) mine += (double)c[j] * (double)__uint_as_float(k & 0x7FFFFFFFu);
                }
            }
            need -= r[1];
            SBC_TS(1, 3 + 2 * step);
        }
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
                    stream([&](const uint2& e) {
                        const uint32_t v = mode ? ~e.y : e.x;
                        if ((mode == 0 || e.x == tau) && (level == 0 || (v >> (shift + bits)) == found))
                            atomicAdd(&sh.hist[(v >> shift) & ((1u << bits) - 1u)], 1u);
                    });
                    __syncthreads();
                    pick_bin<kThThreads>(sh.hist, r, 0u, sh.scratch, sh.res[0], c);
                    const uint32_t digit = sh.res[0][0];
                    if (digit == 0xFFFFFFFFu) { ok = false; break; }   // uniform
                    r -= sh.res[0][1];
                    same = sh.res[0][3];
                    found = (found << bits) | digit;
                }
                if (mode) itau = ~found;
                else { tau = found; keep = r; ties = same; }
            }
        }
        if (!ok) {                                     // uniform; cannot happen
            if (tid == 0) atomicOr(&result->err, kErrInternal);
            return;
        }
    }
    if (!pick || !placed) {                            // uniform: added up here, with the final threshold
        const bool all = !pick;
        limit = exact_limit(tau, kc);
        if (!wide) for_keys([&](uint32_t k) { if (k > tau || all) add(k); });
    }
    if (tid == 0 && limit == 0u) sh.spread = 1u;
    mine = wave_sum_f64(mine);
    if ((tid & 63) == 63) sh.dsum[tid >> 6] = mine;
    __syncthreads();
    const uint32_t e_tau = max((tau >> 23) & 0xFFu, 1u);               // (tau's fp32 exponent, if it is positive)
    double S = last_lane(wave_sum_f64((tid & 63) < kThThreads / 64 ? sh.dsum[tid & 63] : 0.0)) +
               (double)keep * (double)__uint_as_float(tau & 0x7FFFFFFFu);
    if (__builtin_expect(sh.spread != 0u, 0)) {        // uniform
        // Values of both signs, or too far apart: integers, each at the scale of tau's exponent while it fits
        // 64 bits, else one integer per exponent (all read from memory once more).
        const bool common = kc <= 32768u && tau > 0x80000000u, all = !pick;
        __syncthreads();
        if (tid < 256) sh.acc[tid] = 0ll;
        __syncthreads();
        long long scaled = 0ll;
        stream([&](const uint2& e) {
            if (!all && !cand_kept(e.x, e.y, tau, itau)) return;
            uint32_t ex;
            const long long m = signed_mantissa(e.x, s, ex);
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
    st[t].cand_seen[s] = full_cnt;                     // (inspection only)
    st[t].tau[s] = tau;
    st[t].itau[s] = itau;
    st[t].kc[s] = kc;
    st[t].S[s] = S;
    st[t].mean[s] = S / (double)kc;
    uint32_t raise = 0u;
    if (carry && pick) {
        const bool ranked = next_bin != 0xFFFFFFFFu;
        uint32_t next = (base + next_bin) << kThShift;
        if (__builtin_expect(!ranked, 0))
            next = (d.flags & kDescWide) ? lowered_key(lo_key, 0.1f) : extrapolated_key(tau, lo_key, d.k, rank2, d.n, full_cnt);
        st[t].lo_key[s] = next;
        st[t].expect[s] = ranked && !(d.flags & kDescWide) ? rank2 : 0u;
    }
    // many times more candidates than needed: the next call should estimate its keys afresh
    if (full_cnt > loose_limit(d.k, d.n)) raise |= kErrLoose;
    if (wide) raise |= kErrWide;
    if (raise) atomicOr(&result->err, raise);
    SBC_TS(1, 7);
}

// --------------------------------------------------------------------------
// Tensors that keep very many entries (lists too long for one workgroup's registers).  grid
// (workgroups, 2 x wide tensors); a list gets only as many of the workgroups as it has use for: a
// workgroup adds its counts to the shared histogram bin by bin, and those atomics cost more than
// the reading when every workgroup has few entries per bin.
// --------------------------------------------------------------------------
// Entries that keep a workgroup of a sweep busy (short lists: 1024 each, up to 32 workgroups).  Both
// sweeps together: 12 us on lists of 30,000 entries (2^20-entry tensor, p = 0.01), 23 us on ten tensors
// with up to 70,000 each, 146 us on 3e6 (1.5e9 entries, p = 0.001; 160 us with 2048 each).
constexpr uint32_t kWidePerWorkgroup = 4096;
constexpr uint32_t kWideFound = 512;                   // entries of the k-th entry's bin that a workgroup collects in LDS

__device__ __forceinline__ uint32_t wide_workgroups(uint32_t cnt) {
    const uint32_t few = min((cnt + 1023u) / 1024u, 32u), many = (cnt + kWidePerWorkgroup - 1u) / kWidePerWorkgroup;
    const uint32_t want = few > many ? few : many;
    return want < gridDim.x ? (want ? want : 1u) : gridDim.x;
}

// The lists can be selected from, and the subsampled variant does not keep all of this one.
__device__ __forceinline__ bool wide_applies(const TensorDesc& d, uint32_t cnt_p, uint32_t cnt_n) {
    if (cnt_p > d.cand_cap || cnt_n > d.cand_cap) return false;
    return (d.flags & kDescSampled) ? cnt_p >= 1u && cnt_n >= 1u : cnt_p >= d.k && cnt_n >= d.k;
}

// k_wide_count: window histogram of a side's list.  (Counting where the streaming kernel stores the
// candidates would save this sweep, but every count would be an atomic on memory that all
// compute-unit groups share, and those on one bin queue up for about half a microsecond each: four
// times the streaming kernel's time on Gaussian data.)
__global__ __launch_bounds__(kWideThreads) void k_wide_count(
        const TensorDesc* __restrict__ desc, const WideIds wide_ids, const TensorState* __restrict__ st,
        const uint2* __restrict__ cand, uint32_t* __restrict__ whist, long long* __restrict__ wacc,
        WideState* __restrict__ ws) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kThBins];
    const int w = blockIdx.y >> 1, s = blockIdx.y & 1, tid = threadIdx.x;
    const int t = (int)wide_ids.id[w];
    const TensorDesc d = desc[t];
    const uint32_t cnt_p = st[t].cand_cnt[0], cnt_n = st[t].cand_cnt[1];
    const uint32_t cnt = s ? cnt_n : cnt_p;
    const uint32_t base = st[t].lo_key[s] >> kThShift;
    if (blockIdx.x == 0) {                             // the call before this one has read its sums
        wacc[(size_t)blockIdx.y * 256 + tid] = 0ll;
        if (tid == 0) {
            WideState z;
            z.ok = 0u; z.prefix = 0u; z.need = 0u; z.count = 0u; z.next_rank_bin = 0xFFFFFFFFu;
            z.pad[0] = z.pad[1] = z.pad[2] = 0u;
            ws[blockIdx.y] = z;
        }
    }
    if (!wide_applies(d, cnt_p, cnt_n) || kept_of_side(d, cnt) == cnt) return;      // uniform
    const uint32_t nb = wide_workgroups(cnt);
    if (blockIdx.x >= nb) return;
    const uint2* __restrict__ list = cand + d.cand_off + (s ? d.cand_cap : 0u);
    uint4* const h4 = reinterpret_cast<uint4*>(hist);
#pragma unroll
    for (int i = 0; i < kThBins / 4 / kWideThreads; ++i) h4[i * kWideThreads + tid] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const uint64_t stride = (uint64_t)nb * kWideThreads;
#pragma unroll 8
    for (uint64_t i = (uint64_t)blockIdx.x * kWideThreads + tid; i < cnt; i += stride)
        atomicAdd(&hist[window_bin(list[i].x, base)], 1u);
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
        const uint2* __restrict__ cand, uint32_t* __restrict__ bitmap, const uint32_t* __restrict__ whist,
        long long* __restrict__ wacc, WideState* __restrict__ ws) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kThBins];
    __shared__ long long acc[256];
    __shared__ uint2 found[kWideFound];
    __shared__ uint32_t scratch[kWideThreads / 64], res[4], n_found, found_at;
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
    const uint32_t cnt_p = st[t].cand_cnt[0], cnt_n = st[t].cand_cnt[1];
    const uint32_t cnt = s ? cnt_n : cnt_p;
    const uint32_t base = st[t].lo_key[s] >> kThShift;
    if (!wide_applies(d, cnt_p, cnt_n)) return;        // k_threshold flags the tensor
    const uint32_t nb = wide_workgroups(cnt);
    if (blockIdx.x >= nb) return;
    const uint32_t kc = kept_of_side(d, cnt);
    const bool all = (d.flags & kDescSampled) && kc == cnt;
#pragma unroll
    for (int i = 0; i < kThBins / 4 / kWideThreads; ++i) reinterpret_cast<uint4*>(hist)[i * kWideThreads + tid] = mine[i];
    acc[tid] = 0ll;
    if (tid < 4) res[tid] = 0xFFFFFFFFu;
    if (tid == 4) n_found = 0u;
    __syncthreads();
    uint32_t prefix = 0u;
    if (!all) {
        uint32_t c[kThBins / kWideThreads];
        pick_bin<kWideThreads>(hist, kc, carried_rank(kc), scratch, res, c);
        const uint32_t digit = res[0];
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
    uint2* __restrict__ out = wide_list(d, bitmap, s);
    const uint32_t room = wide_room(d);
    const uint2* __restrict__ list = cand + d.cand_off + (s ? d.cand_cap : 0u);
    const uint64_t stride = (uint64_t)nb * kWideThreads;
    const uint32_t from = all ? st[t].lo_key[s] : prefix << kThShift, limit = exact_limit(from, kc);
    double near = 0.0;
#pragma unroll 4
    for (uint64_t i = (uint64_t)blockIdx.x * kWideThreads + tid; i < cnt; i += stride) {
        const uint2 e = list[i];
        const uint32_t v = e.x >> kThShift;
        if (all || v > prefix) {
            if (e.x < limit) {
                near += (double)__uint_as_float(e.x & 0x7FFFFFFFu);
            } else {
                uint32_t ex;
                const long long m = signed_mantissa(e.x, s, ex);
                if (m != 0ll && ex < 255u) atomicAdd(reinterpret_cast<unsigned long long*>(&acc[ex]), (unsigned long long)m);
            }
        } else if (v == prefix) {
            // (a workgroup's few go out together: one atomic on the shared counter instead of one each,
            // which queue up there for about 60 ns apiece)
            const uint32_t q = atomicAdd(&n_found, 1u);
            if (q < kWideFound) found[q] = e;
            else {
                const uint32_t at = atomicAdd(&ws[blockIdx.y].count, 1u);
                if (at < room) out[at] = e;
            }
        }
    }
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
            if (found_at + i < room) out[found_at + i] = found[i];
    }
    const long long v = acc[tid];
    if (v != 0ll) atomicAdd(reinterpret_cast<unsigned long long*>(&wacc[(size_t)blockIdx.y * 256 + tid]), (unsigned long long)v);
}

}  // namespace sbc
