// Stage 1 of the client step and the candidate search around it.
//
// Fast path (two launches):
//   k_sample_thresholds  per tensor: a stratified sample of A = R + dW gives, for each sign
//                        side, a key that is with overwhelming probability at or below the
//                        k-th most extreme entry of the whole tensor (conservative: only a
//                        filter, never the answer)
//   k_accumulate_filter  per chunk: A = R + dW written over R (Alg. 1, client line
//                        dW_i <- R_i + local update); every entry at or beyond a side's
//                        filter key is appended to that side's candidate list
// If a side ends up with fewer than k candidates the filter was too tight for that tensor;
// the histogram path below then finds its candidates exactly from a second read of A:
//   k_hist_flagged, k_pick_bins, k_extract
// Either way k_threshold receives, per tensor and side, a list that contains the k most
// extreme entries, and the result is exact.
#pragma once

#include "sbc_device.hpp"

namespace sbc {

// --------------------------------------------------------------------------
// Plain streaming copy of 16-byte units: the yardstick the streaming kernels are measured
// against (same workgroup shape and loads in flight as the accumulation kernel).
// --------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_copy_baseline(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                       uint64_t n16) {
    const uint64_t base = (uint64_t)blockIdx.x * 2048ull + threadIdx.x;
    if (base - threadIdx.x + 2048ull <= n16) {
        uint4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = src[base + 256ull * i];
#pragma unroll
        for (int i = 0; i < 8; ++i) dst[base + 256ull * i] = v[i];
    } else {
        for (uint64_t j = base; j < n16; j += 256ull) dst[j] = src[j];
    }
}

__global__ __launch_bounds__(256) void k_zero_words(uint32_t* __restrict__ p, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0u;
}

// The status of a server call, sent to pinned host memory by a dispatch of its own behind the decode
// kernels (the runtime's own device-to-host copy and its wait for the stream take longer).
__global__ void k_publish(unsigned long long* __restrict__ host_word, const ResultBlock* __restrict__ src, uint32_t seq) {
    if (threadIdx.x == 0) publish(host_word, seq, src->err, 0ull);
}

__device__ __forceinline__ uint32_t mix32(uint32_t x) {
    x ^= x >> 16; x *= 0x7FEB352Du; x ^= x >> 15; x *= 0x846CA68Bu; x ^= x >> 16;
    return x;
}

// --------------------------------------------------------------------------
// Prefilter thresholds from a sample.  One workgroup (1024 threads) per tensor.  Tensors of up to
// kSampleMax entries are read completely (the threshold is then the exact k-th key to 16
// bits); larger ones contribute 256 runs of 64 consecutive entries, one run at a pseudo-random
// place in each of 256 equal strata.  With m sampled entries out of n, lambda = k*m/n of them
// are expected among the tensor's k most extreme; the filter key is the lower edge of the
// 16-bit key bucket holding the sample's r-th most extreme entry, r = lambda + 4*sqrt(lambda)
// + 3, so that the chance of cutting into the true top k is negligible (and harmless: the
// histogram path then redoes the tensor).  Both sides are selected together, the negative side
// on complemented keys.  The kernel also clears the per-tensor state, and
// it tells whether the keys the previous call left for this one (they are still in the state when
// the kernel starts) would have held: if the sample says that far more entries than a selection
// wants lie at or above them, kErrStaleKeys is raised, and the host goes on sampling.
// For tensors flagged kDescSampled ("Sparse Binarization": the threshold is estimated from a
// random subsample, which makes the amount of sparsity noisy) the key is instead the full 32-bit
// key of the sample's r-th most extreme entry, r = max(1, floor(p*m)): the threshold itself.
// Bound by its chain of dependent steps, of which the counting passes over a thread's share of the sample grow
// with that share: 13.6 us on 9 tensors with 1024 threads (15.8 with 512, and the counts cleared before the
// loads went out).  No more than 512 keys are ranked: beyond that the byte passes are the shorter way.
// --------------------------------------------------------------------------
__global__ __launch_bounds__(kSampleThreads) void k_sample_thresholds(
        const TensorDesc* __restrict__ desc, TensorState* __restrict__ st,
        ResultBlock* __restrict__ result, int force_exact, double sampled_p) {
    constexpr int RUNS = kSampleMax / 64;             // 256
    constexpr int COPIES = 16;
    constexpr uint32_t RANKED = 512u;                 // most keys of a bucket that are ranked one against the others
    __shared__ uint32_t skey[kSampleMax];             // the sample, as keys (loops stay rolled: small code)
    __shared__ uint32_t hist0[2][256][COPIES];        // first byte: lane-private copies, one bank each
    __shared__ uint32_t hist[4][2][256];
    __shared__ uint32_t whist[2][kSampleWindow];      // leading 16 key bits, counted down from the extreme
    __shared__ uint32_t wave_ext[2][kSampleThreads / 64];
    __shared__ uint32_t wave_above[kSampleThreads / 64];
    __shared__ uint32_t blist[2][RANKED];     // subsampled variant: the sampled keys of the threshold's bucket
    __shared__ uint32_t bcnt[2], btau[2];
    __shared__ uint32_t res[4][8];
    __shared__ unsigned long long scratch[kSampleThreads / 64];
    SBC_TS(0, 0);
    const int t = blockIdx.x, tid = threadIdx.x;
    const TensorDesc d = desc[t];
    const uint32_t old_p = st[t].lo_key[0], old_n = st[t].lo_key[1];      // what the previous call left
    __syncthreads();                                  // (every thread has them before the state is cleared)
    if (tid == 0) {
        // (the call's result block is clean already: the previous call's last kernel, or the host
        // after an error, cleared it.  A plain store to it here would sit in this compute-unit group's
        // L2 until the kernel ends and then overwrite the bits other groups' workgroups raise below.)
        TensorState z;
        z.lo_key[0] = z.lo_key[1] = force_exact ? 0xFFFFFFFFu : 0u;
        z.cand_cnt[0] = z.cand_cnt[1] = 0u;
        z.bin[0] = z.bin[1] = 0u;
        z.tau[0] = z.tau[1] = 0u;
        z.itau[0] = z.itau[1] = 0u;
        z.kc[0] = z.kc[1] = 0u;
        z.S[0] = z.S[1] = 0.0; z.mean[0] = z.mean[1] = 0.0;
        z.side = 0; z.mu_signed = 0.f; z.nnz = 0u; z.flags = 0u; z.bit_len = 0ull;
        z.done = 0u; z.sorted_kept = 0u; z.cand_seen[0] = z.cand_seen[1] = 0u; z.expect[0] = z.expect[1] = 0u;
        st[t] = z;
    }
    if (force_exact) return;
    // a one-chunk tensor that the streaming kernel finishes by itself needs no filter key
    if ((d.flags & kDescInline) && d.nchunks == 1u && d.n <= 6144u) return;       // (kSmallMaxN of the streaming kernel)

    const uint32_t n = d.n;
    const uint32_t m = n < (uint32_t)kSampleMax ? n : (uint32_t)kSampleMax;
    const bool sampled = (d.flags & kDescSampled) != 0u;
    uint32_t rs = d.k;
    if (sampled) {
        // "Sparse Binarization", subsampled variant: the r-th most extreme sampled value itself is
        // the threshold, r = max(1, floor(p * m))
        const double r = floor(sampled_p * (double)m);
        rs = r < 1.0 ? 1u : (uint32_t)r;
    } else if (n > (uint32_t)kSampleMax) {
        rs = sample_rank(d.k, m, n);
    }
    if (rs >= m) return;                              // keep the all-pass keys (0, 0)
    const int passes = sampled ? 4 : 2;               // all 32 key bits, or the leading 16

    uint32_t need[2] = {rs, rs};
    const bool active[2] = {true, true};
    uint32_t prefix[2] = {0u, 0u};
    int first_pass = 0;
    // The sample: all of a thread's loads are issued before the first key is formed, so that the
    // kernel pays the memory latency once.
    const gcfloat_ptr R = as_global(d.R);
    const gcfloat_ptr dW = as_global(d.dW);
    {
        constexpr int PER = kSampleMax / kSampleThreads;      // 16
        float a[PER], w[PER];
        if (n <= (uint32_t)kSampleMax) {
#pragma unroll
            for (int s = 0; s < PER; ++s) {
                const uint32_t i = s * kSampleThreads + tid;
                const uint32_t j = i < m ? i : 0u;
                a[s] = R[j]; w[s] = dW[j];
            }
        } else {
            const unsigned long long slots = n / 64u;     // >= RUNS
            const uint32_t lane = tid & 63u;
#pragma unroll
            for (int s = 0; s < PER; ++s) {
                const uint32_t run = s * (kSampleThreads / 64) + (tid >> 6);             // 0..RUNS-1
                const uint32_t h = mix32(run * 0x9E3779B9u + (uint32_t)t * 0x85EBCA6Bu + 1u);
                const uint32_t s_lo = (uint32_t)(run * slots / RUNS), s_hi = (uint32_t)((run + 1u) * slots / RUNS);
                const uint32_t i = (s_lo + __umulhi(h, s_hi - s_lo)) * 64u + lane;       // a slot of the run's stratum
                a[s] = R[i]; w[s] = dW[i];
            }
        }
        // (the counts are cleared while the loads are on their way; the barrier below precedes their first use)
        for (int i = tid; i < 3 * 2 * 256; i += kSampleThreads) (&hist[1][0][0])[i] = 0u;
        for (int i = tid; i < 2 * kSampleWindow; i += kSampleThreads) (&whist[0][0])[i] = 0u;
        // Keys, and the most extreme key of each side (this thread's, then the workgroup's).
        uint32_t key[PER], ext_p = 0u, ext_n = 0u, above = 0u;       // above: sampled entries at or beyond the old keys, 16 bits per side
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            key[s] = key_of_bits(__float_as_uint(a[s] + w[s]));
            skey[s * kSampleThreads + tid] = key[s];
            if ((uint32_t)(s * kSampleThreads + tid) < m) {
                ext_p = key[s] > ext_p ? key[s] : ext_p;
                ext_n = ~key[s] > ext_n ? ~key[s] : ext_n;
                above += (key[s] >= old_p ? 1u : 0u) + (~key[s] >= old_n ? 0x10000u : 0u);
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const uint32_t op = __shfl_xor(ext_p, off, 64), on = __shfl_xor(ext_n, off, 64);
            ext_p = op > ext_p ? op : ext_p;
            ext_n = on > ext_n ? on : ext_n;
            above += __shfl_xor(above, off, 64);      // (at most 1024 per side and wavefront)
        }
        if ((tid & 63) == 0) { wave_ext[0][tid >> 6] = ext_p; wave_ext[1][tid >> 6] = ext_n; wave_above[tid >> 6] = above; }
        __syncthreads();
        SBC_TS(0, 1);                                 // sample loaded
        if (tid == 0) {
            uint32_t ap = 0u, an = 0u;
            for (int wv = 0; wv < kSampleThreads / 64; ++wv) { ap += wave_above[wv] & 0xFFFFu; an += wave_above[wv] >> 16; }
            // scaled to the tensor; the limit is the one beyond which k_threshold calls a list loose
            const double scale = (double)n / (double)m, many = (double)loose_limit(d.k, n);
            if ((double)ap * scale > many || (double)an * scale > many) atomicOr(&result->err, kErrStaleKeys);
        }
#pragma unroll
        for (int wv = 0; wv < kSampleThreads / 64; ++wv) {
            ext_p = wave_ext[0][wv] > ext_p ? wave_ext[0][wv] : ext_p;
            ext_n = wave_ext[1][wv] > ext_n ? wave_ext[1][wv] : ext_n;
        }
        // The r-th most extreme key lies within a few octaves of the most extreme one: the leading
        // 16 key bits are counted in a window of kSampleWindow values (16 octaves) below it, straight
        // from the registers; the bulk of the sample spreads over hundreds of bins there, where the
        // leading byte alone takes a handful of values.  Keys below the window are not counted.
        const uint32_t top[2] = {ext_p >> 16, ext_n >> 16};
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            if ((uint32_t)(s * kSampleThreads + tid) < m) {
                const uint32_t dp = top[0] - (key[s] >> 16), dn = top[1] - (~key[s] >> 16);
                if (dp < (uint32_t)(kSampleWindow - 1)) atomicAdd(&whist[0][(uint32_t)(kSampleWindow - 1) - dp], 1u);
                if (dn < (uint32_t)(kSampleWindow - 1)) atomicAdd(&whist[1][(uint32_t)(kSampleWindow - 1) - dn], 1u);
            }
        }
        __syncthreads();
        SBC_TS(0, 2);                                 // window histogram done
        uint32_t digit[2];
        bool found[2];
        pick_wide_both<kSampleWindow, kSampleThreads>(whist, need, active, res[0], scratch, digit, found);
        SBC_TS(0, 3);
        if (found[0] && found[1]) {                   // uniform
            prefix[0] = top[0] - ((uint32_t)(kSampleWindow - 1) - digit[0]);
            prefix[1] = top[1] - ((uint32_t)(kSampleWindow - 1) - digit[1]);
            first_pass = 2;
        } else {
            need[0] = need[1] = rs;                   // (a found side's need was lowered)
        }
        if (sampled && first_pass == 2) {
            // All 32 bits of the r-th key are wanted: the sampled keys of its bucket (a handful) are
            // collected and each is ranked against the others; the one that need[s] - 1 others
            // exceed is the key.  A crowded bucket is left to the byte passes below.
            if (tid < 2) bcnt[tid] = 0u;
            __syncthreads();
#pragma unroll
            for (int s = 0; s < PER; ++s) {
                if ((uint32_t)(s * kSampleThreads + tid) < m) {
                    if ((key[s] >> 16) == prefix[0]) {
                        const uint32_t q = atomicAdd(&bcnt[0], 1u);
                        if (q < RANKED) blist[0][q] = key[s];
                    }
                    if ((~key[s] >> 16) == prefix[1]) {
                        const uint32_t q = atomicAdd(&bcnt[1], 1u);
                        if (q < RANKED) blist[1][q] = ~key[s];
                    }
                }
            }
            __syncthreads();
            const uint32_t c0 = bcnt[0], c1 = bcnt[1];
            if (c0 <= RANKED && c1 <= RANKED) {      // uniform
#pragma unroll
                for (int sd = 0; sd < 2; ++sd) {
                    const uint32_t cn = sd ? c1 : c0;
                    if ((uint32_t)tid < cn) {
                        const uint32_t me = blist[sd][tid];
                        uint32_t above = 0u, at_least = 0u;
                        for (uint32_t j = 0; j < cn; ++j) {
                            const uint32_t o = blist[sd][j];
                            above += o > me ? 1u : 0u;
                            at_least += o >= me ? 1u : 0u;
                        }
                        if (above < need[sd] && need[sd] <= at_least) btau[sd] = me;   // equal keys write the same value
                    }
                }
                __syncthreads();
                prefix[0] = btau[0]; prefix[1] = btau[1];
                first_pass = 4;
            }
        }
    }
    __syncthreads();
    if (first_pass == 0) {
        // The r-th entry lies below the window (mostly-zero tensors): byte by byte from the top.
        // First byte: floating-point keys take only a handful of values here, so every lane group
        // counts into its own copy and the copies are added up afterwards.
        for (int i = tid; i < 2 * 256 * COPIES; i += kSampleThreads) (&hist0[0][0][0])[i] = 0u;
        __syncthreads();
        const int copy = ((tid >> 6) & 1) * 8 + (tid & 7);
#pragma unroll 8
        for (uint32_t i = tid; i < m; i += kSampleThreads) {
            const uint32_t kp = skey[i];
            atomicAdd(&hist0[0][kp >> 24][copy], 1u);
            atomicAdd(&hist0[1][(~kp) >> 24][copy], 1u);
        }
        __syncthreads();
        if (tid < 2 * 256) {
            uint32_t sum = 0u;
#pragma unroll
            for (int c = 0; c < COPIES; ++c) sum += (&hist0[0][0][0])[tid * COPIES + c];   // tid = side*256 + byte
            (&hist[0][0][0])[tid] = sum;
        }
        __syncthreads();
    }
    SBC_TS(0, 2);                                     // first-byte histogram done
    // the remaining bytes of the r-th largest key (positive side) and of the r-th largest
    // complemented key (negative side), one byte per pass
#pragma nounroll
    for (int pass = first_pass; pass < passes; ++pass) {
        if (pass > 0) {
            const int shift = 24 - 8 * pass;
#pragma unroll 8
            for (uint32_t i = tid; i < m; i += kSampleThreads) {
                const uint32_t kp = skey[i], kn = ~kp;
                if ((kp >> (shift + 8)) == prefix[0]) atomicAdd(&hist[pass][0][(kp >> shift) & 255u], 1u);
                if ((kn >> (shift + 8)) == prefix[1]) atomicAdd(&hist[pass][1][(kn >> shift) & 255u], 1u);
            }
            __syncthreads();
        }
        SBC_TS(0, 3 + 2 * pass);
        const BytePick pk = pick_byte_both<kSampleThreads>(hist[pass], need, active, res[pass], scratch);
        SBC_TS(0, 4 + 2 * pass);
        if (!pk.found[0] || !pk.found[1]) return;     // uniform; cannot happen; all-pass keys stay
        prefix[0] = (prefix[0] << 8) | pk.byte[0];
        prefix[1] = (prefix[1] << 8) | pk.byte[1];
    }
    SBC_TS(0, 11);
    if (tid == 0) {
        const int left = 32 - 8 * passes;             // 16: lower edge of the 16-bit bucket; 0: the key itself
        st[t].lo_key[0] = prefix[0] << left;
        st[t].lo_key[1] = prefix[1] << left;          // same, in the complemented key space
    }
}

// --------------------------------------------------------------------------
// Appends flagged entries of one chunk to the two candidate lists of its tensor with a block
// scan (histogram path).  key[s] is the plain key of the thread's s-th entry (entry s*NT + tid of the
// chunk); bit s of mp / mn flags it for the positive / negative list; the negative list stores
// complemented keys.  Contains barriers; every thread of the workgroup must call it.
// --------------------------------------------------------------------------
template <int PER>
__device__ __forceinline__ void append_candidates(const uint32_t (&key)[PER], uint32_t mp, uint32_t mn,
                                                  uint32_t e_first, const TensorDesc& d, TensorState* __restrict__ st_t,
                                                  const CandPtr cand, ChunkRun* __restrict__ run,
                                                  uint32_t* scratch, uint32_t* base) {
    const int tid = threadIdx.x;
    const uint32_t packed = __popc(mp) | (__popc(mn) << 16);
    uint32_t total;
    const uint32_t ex = block_excl_sum<uint32_t, kStreamThreads>(packed, &total, scratch);
    if (total == 0u) {                                // uniform
        if (tid == 0) *run = chunk_run(d, 0u, 0u, 0u, 0u);
        return;
    }
    if (tid == 0) {
        const uint32_t tp = total & 0xFFFFu, tn = total >> 16;
        const unsigned long long old = atomicAdd(reinterpret_cast<unsigned long long*>(&st_t->cand_cnt[0]),
                                                 (unsigned long long)tp | ((unsigned long long)tn << 32));
        base[0] = (uint32_t)old;
        base[1] = (uint32_t)(old >> 32);
        *run = chunk_run(d, (uint32_t)old, (uint32_t)(old >> 32), tp, tn);
    }
    __syncthreads();
    uint32_t op = base[0] + (ex & 0xFFFFu);
    uint32_t on = base[1] + (ex >> 16);
    __syncthreads();                                  // base may be rewritten by the next call
    // (beyond a list's capacity nothing is stored: the counters then show that the tensor's lists
    // are not usable, see lists_unusable; a list of a full context holds every entry)
    if (op + __popc(mp) > d.cand_cap || on + __popc(mn) > d.cand_cap) return;
    const CandPtr cp = cand + d.cand_off, cn = cp + d.cand_cap;
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        const uint32_t idx = e_first + s * kStreamThreads + tid;
        if (mp & (1u << s)) cp.put(op++, key[s], idx);
        if (mn & (1u << s)) cn.put(on++, ~key[s], idx);
    }
}

// --------------------------------------------------------------------------
// Residual accumulation fused with the prefilter.  One workgroup per chunk of 8192 entries: 8 x 16-byte loads of
// each operand in flight per thread, A stored over R and kept in LDS.  Every thread gathers two bit masks of its 32 entries, those at
// or beyond each side's filter key (the keys' order is that of the values, so this is one comparison
// of floats per side); one scan of the counts and one 64-bit atomic for both sides then give every
// candidate its place, and each thread copies its few from LDS.  However many there are, the path is
// the same.  (One tensor's workgroups queue up on its counter: 512 of them 15.6 us; with eight counters, and
// the lists in as many segments, 11.5.)  Where a chunk's candidates went is recorded (ChunkRun).  Bound by HBM on large calls (54 us
// on 25.6e6 entries, a plain R += dW takes 54.5 us there).  Small ones are bound by latency: with a test, an LDS
// counter and a queue per entry, 18 KB of code, 128 chunks took 11.8 us and 41 took 10.3; now 7.4 and
// 5.6.  Operands that are only 4-byte aligned take the same loads (24 ragged tensors of 12e6 entries in
// one buffer: 27.4 us, 35 with scalar ones).
// --------------------------------------------------------------------------
// Which workgroup takes which chunk, and how many run at a time, is what memory rate hangs on beyond the last-level
// cache.  Workgroups go to the eight compute-unit groups in turn; each takes runs of kRun consecutive chunks, so
// that it has whole pieces of 128 KB of each array.  In large calls two of them share a compute unit instead of the four that
// its registers hold (the launch asks for LDS that nobody uses, kStreamRoom, see kPairsFrom): 32 streams of
// 4 KB requests from every one of 256 compute units keep more of memory's pages open than it has.  Whole steps in us, one
// tensor: 1.5e9 entries 3505, two at a time 3255, with runs of four as well 3050 (6.4 TB/s in this kernel; runs of two
// 3214, of eight 3093, of sixteen 3140, a contiguous eighth per compute-unit group 3112, one at a time 3758; four
// at a time with runs of eight 3320), 400e6 941 / 848, 100e6 258 / 246, LSTM shape 162 / 156; smaller ones beside kPairsFrom.
constexpr uint32_t kRun = 4, kComputeUnitGroups = 8;
constexpr size_t kStreamRoom = 23552;                     // 55 KB in all: two to a compute unit, and room for another kernel's
__device__ __forceinline__ uint32_t chunk_of_workgroup() {
    constexpr uint32_t G = kRun * kComputeUnitGroups;
    const uint32_t i = blockIdx.x % G, g0 = blockIdx.x - i;
    return g0 + G <= gridDim.x ? g0 + i % kComputeUnitGroups * kRun + i / kComputeUnitGroups : blockIdx.x;
}

struct FilterShared {
    f32x4 a[kChunk / 4];
    uint32_t base[2];
    uint32_t scratch[kStreamThreads / 64];
};

// The value whose comparison stands for that of the side key: an entry a has a side key at or above
// `key` if and only if a >= value_of_key<0>(key) on the positive side, -a >= value_of_key<1>(key) on the
// negative side, for every finite a.  (A zero's key is above the middle on the positive side and,
// complemented, below it on the negative one.)
template <int S>
__device__ __forceinline__ float value_of_key(uint32_t key) {
    if (S && key == 0x80000000u) return __uint_as_float(1u);
    return key < 0x00800000u ? -__builtin_inff() : __uint_as_float(bits_of_key(key));     // (below -inf's: all; above +inf's: NaN, none)
}

// What goes past the last-level cache, with the nontemporal hint (the rule is in accumulate_past_cache):
constexpr int kPastNothing = 0, kPastUpdate = 1, kPastAll = 2;     // (kPastAll: update loaded, residual loaded and stored)
template <int PAST>
__global__ __launch_bounds__(kStreamThreads, 4) void k_accumulate_filter(
        const TensorDesc* __restrict__ desc, const uint2* __restrict__ chunk_tensor,
        TensorState* __restrict__ st, unsigned long long* __restrict__ counters, const CandPtr cand,
        ChunkRun* __restrict__ runs, ResultBlock* __restrict__ result) {
    __shared__ FilterShared sh;
    const int tid = threadIdx.x;
    const uint32_t c = chunk_of_workgroup();
    const uint2 ct = chunk_tensor[c];                     // (tensor, its first chunk)
    const int t = (int)ct.x;
    const TensorDesc d = desc[t];
    const float lo_p = value_of_key<0>(st[t].lo_key[0]), lo_n = -value_of_key<1>(st[t].lo_key[1]);
    constexpr int IT = kChunk / 4 / kStreamThreads;       // 8 vectors of four entries per thread
    static_assert(IT * 4 == 32, "a bit per entry");
    const uint32_t e0 = (c - ct.y) * (uint32_t)kChunk;
    const uint32_t cnt = min((uint32_t)kChunk, d.n - e0);
    const gcfloat_ptr dw = as_global(d.dW + e0);
    const gfloat_ptr r = as_global(d.R + e0);
    const gcf32x4_any_ptr dw4 = (gcf32x4_any_ptr)dw;
    const gf32x4_any_ptr r4 = (gf32x4_any_ptr)r;
    const bool whole = cnt == (uint32_t)kChunk;           // uniform
    f32x4 dv[IT], rv[IT];
    uint32_t valid = 0xFFFFFFFFu;                         // entry 4 i + j of the thread is bit 31 - (4 i + j)
    if (whole) {
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            dv[i] = PAST >= kPastUpdate ? __builtin_nontemporal_load(&dw4[i * kStreamThreads + tid]) : dw4[i * kStreamThreads + tid];
            rv[i] = PAST == kPastAll ? __builtin_nontemporal_load(&r4[i * kStreamThreads + tid]) : r4[i * kStreamThreads + tid];
        }
    } else {
        valid = 0u;
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const uint32_t at = (uint32_t)(i * kStreamThreads + tid) * 4u;
            dv[i] = 0.f; rv[i] = 0.f;
            valid <<= 4;
            if (at + 4u <= cnt) {
                dv[i] = dw4[i * kStreamThreads + tid]; rv[i] = r4[i * kStreamThreads + tid];
                valid |= 15u;
            } else if (at < cnt) {                    // the one vector that the tensor ends in
                dv[i].x = dw[at]; rv[i].x = r[at];
                if (at + 1u < cnt) { dv[i].y = dw[at + 1u]; rv[i].y = r[at + 1u]; }
                if (at + 2u < cnt) { dv[i].z = dw[at + 2u]; rv[i].z = r[at + 2u]; }
                valid |= at + 2u < cnt ? 14u : at + 1u < cnt ? 12u : 8u;
            }
        }
    }
    uint32_t mp = 0u, mn = 0u;
    float nonfinite = 0.f;                                // a NaN as soon as some entry is a NaN or an infinity
    auto test = [&](float x) {
        // mask = 2 mask + (comparison): two instructions a side (the compiler makes four and holds every
        // bit in a register of its own)
        asm("v_cmp_ge_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(mp) : "v"(x), "v"(lo_p) : "vcc");
        asm("v_cmp_le_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(mn) : "v"(x), "v"(lo_n) : "vcc");
        nonfinite = __builtin_fmaf(x, 0.f, nonfinite);
    };
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        f32x4 a;
        a.x = rv[i].x + dv[i].x;
        a.y = rv[i].y + dv[i].y;
        a.z = rv[i].z + dv[i].z;
        a.w = rv[i].w + dv[i].w;
        sh.a[i * kStreamThreads + tid] = a;
        if (whole) {                                  // uniform
            if (PAST == kPastAll) __builtin_nontemporal_store((f32x4_any)a, &r4[i * kStreamThreads + tid]);
            else r4[i * kStreamThreads + tid] = a;
        }
        test(a.x); test(a.y); test(a.z); test(a.w);
    }
    if (!whole) {                                     // uniform: the stores of a tensor's last chunk
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const uint32_t at = (uint32_t)(i * kStreamThreads + tid) * 4u;
            if (at + 4u <= cnt) r4[i * kStreamThreads + tid] = sh.a[i * kStreamThreads + tid];
            else if (at < cnt) {
                const f32x4 a = sh.a[i * kStreamThreads + tid];
                r[at] = a.x;
                if (at + 1u < cnt) r[at + 1u] = a.y;
                if (at + 2u < cnt) r[at + 2u] = a.z;
            }
        }
        mp &= valid; mn &= valid;
    }
    if (nonfinite != 0.f) atomicOr(&result->err, kErrNonFinite);    // (true for a NaN)
    uint32_t total;
    const uint32_t ex = block_excl_sum<uint32_t, kStreamThreads>(__popc(mp) | (__popc(mn) << 16), &total, sh.scratch);
    const uint32_t qp = total & 0xFFFFu, qn = total >> 16;
    const uint32_t seg = d.segs == 1u ? 0u : (c - ct.y) % kSegs;
    const uint32_t seg0 = seg_before(d, d.segs, seg), seg1 = seg_before(d, d.segs, seg + 1u);
    if (tid == 0) {
        // both sides' counters advance in one 64-bit atomic: the workgroups of one segment queue up on this
        // address, and the wait grows with the number of atomics
        unsigned long long old = 0ull;
        unsigned long long* const counter = d.segs == 1u ? reinterpret_cast<unsigned long long*>(&st[t].cand_cnt[0])
                                                         : counters + ((size_t)t * kSegs + seg) * kCounterStride;
        if (total) old = atomicAdd(counter, (unsigned long long)qp | ((unsigned long long)qn << 32));
        sh.base[0] = (uint32_t)old;
        sh.base[1] = (uint32_t)(old >> 32);
        runs[c] = chunk_run(d, seg0 + (uint32_t)old, seg0 + (uint32_t)(old >> 32), qp, qn);
    }
    if (total == 0u) return;                              // uniform
    __syncthreads();
    const uint32_t base_p = sh.base[0], base_n = sh.base[1];
    // (beyond a list's capacity nothing is stored: the counters then show that the tensor's lists are not
    // usable, see lists_unusable; a list of a full context holds every entry)
    if ((uint64_t)base_p + qp > seg1 - seg0 || (uint64_t)base_n + qn > seg1 - seg0) return;  // uniform
    const float* const flat = reinterpret_cast<const float*>(sh.a);
    auto copy_out = [&](uint32_t m, const CandPtr to, uint32_t flip) {
        uint32_t i = 0u;
        while (m) {
            const uint32_t s = (uint32_t)__clz((int)m);
            m &= ~(0x80000000u >> s);
            const uint32_t at = ((s >> 2) * (uint32_t)kStreamThreads + (uint32_t)tid) * 4u + (s & 3u);
            to.put(i++, key_of_bits(__float_as_uint(flat[at])) ^ flip, e0 + at);
        }
    };
    copy_out(mp, cand + d.cand_off + seg0 + base_p + (ex & 0xFFFFu), 0u);
    copy_out(mn, cand + d.cand_off + d.cand_cap + seg0 + base_n + (ex >> 16), 0xFFFFFFFFu);
}

// --------------------------------------------------------------------------
// Histogram path, used only for tensors whose prefilter failed (kStFailed).
// k_hist_flagged: per chunk, first-digit histogram of A (already stored in R).
// --------------------------------------------------------------------------
__global__ __launch_bounds__(kStreamThreads) void k_hist_flagged(
        const TensorDesc* __restrict__ desc, const uint2* __restrict__ chunk_tensor,
        const TensorState* __restrict__ st, uint32_t* __restrict__ hist) {
    __shared__ uint32_t lh[kL1Bins];
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x;
    const int t = (int)chunk_tensor[c].x;
    if (!(st[t].flags & kStFailed)) return;
    const TensorDesc d = desc[t];
    const uint32_t e0 = (c - d.chunk0) * (uint32_t)kChunk;
    const uint32_t cnt = min((uint32_t)kChunk, d.n - e0);
    for (int i = tid; i < kL1Bins; i += kStreamThreads) lh[i] = 0u;
    __syncthreads();
    const gcfloat_ptr a = as_global(d.R + e0);
    uint32_t zeros = 0u;
    for (uint32_t i = tid; i < cnt; i += kStreamThreads) {
        const uint32_t u = __float_as_uint(a[i]);
        if ((u << 1) == 0u) ++zeros;
        else atomicAdd(&lh[key_of_bits(u) >> kL1Shift], 1u);
    }
    if (zeros) atomicAdd(&lh[0x80000000u >> kL1Shift], zeros);
    __syncthreads();
    uint32_t* __restrict__ gh = hist + (size_t)t * kL1Bins;
    for (int i = tid; i < kL1Bins; i += kStreamThreads) {
        const uint32_t v = lh[i];
        if (v) atomicAdd(&gh[i], v);
    }
}

// k_pick_bins: per flagged tensor, the bins that hold the k-th largest and k-th smallest
// entry; the tensor's candidate lists restart empty and it is handed to the exact pass.
__global__ __launch_bounds__(256) void k_pick_bins(const TensorDesc* __restrict__ desc,
                                                   const uint32_t* __restrict__ hist,
                                                   TensorState* __restrict__ st,
                                                   ResultBlock* __restrict__ result) {
    __shared__ uint32_t h[kL1Bins];
    __shared__ uint32_t res[2];
    __shared__ uint32_t scratch[4];
    const int t = blockIdx.x, tid = threadIdx.x;
    if (!(st[t].flags & kStFailed)) return;
    const uint32_t k = desc[t].k;
    for (int i = tid; i < kL1Bins; i += 256) h[i] = hist[(size_t)t * kL1Bins + i];
    __syncthreads();
    find_from_top<kL1Bins, 256, false>(h, k, res, scratch);
    const uint32_t bp = res[0];
    __syncthreads();
    find_from_top<kL1Bins, 256, true>(h, k, res, scratch);
    const uint32_t bn = res[0];
    if (tid == 0) {
        if (bp == 0xFFFFFFFFu || bn == 0xFFFFFFFFu) atomicOr(&result->err, kErrInternal);
        st[t].bin[0] = bp;
        st[t].bin[1] = bn;                            // complemented-key numbering
        st[t].lo_key[0] = bp << kL1Shift;             // every candidate's side key is at or above these
        st[t].lo_key[1] = bn << kL1Shift;
        st[t].cand_cnt[0] = 0u; st[t].cand_cnt[1] = 0u;
        st[t].flags = kStExact;
    }
}

// k_extract: per chunk of a tensor in the exact pass, every entry whose first digit lies in or
// beyond a side's threshold bin becomes a candidate of that side.
__global__ __launch_bounds__(kStreamThreads) void k_extract(
        const TensorDesc* __restrict__ desc, const uint2* __restrict__ chunk_tensor,
        TensorState* __restrict__ st, const CandPtr cand, ChunkRun* __restrict__ runs) {
    constexpr int PER = kChunk / kStreamThreads;
    __shared__ uint32_t scratch[kStreamThreads / 64];
    __shared__ uint32_t base[2];
    const int tid = threadIdx.x;
    const uint32_t c = blockIdx.x;
    const int t = (int)chunk_tensor[c].x;
    if (!(st[t].flags & kStExact)) return;
    const TensorDesc d = desc[t];
    const uint32_t e0 = (c - d.chunk0) * (uint32_t)kChunk;
    const uint32_t cnt = min((uint32_t)kChunk, d.n - e0);
    const uint32_t bin_p = st[t].bin[0];
    const uint32_t bin_n = (uint32_t)(kL1Bins - 1) - st[t].bin[1];  // in the plain key space
    const gcfloat_ptr a = as_global(d.R + e0);
    uint32_t key[PER];
    uint32_t mp = 0u, mn = 0u;
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        const uint32_t i = s * kStreamThreads + tid;
        const bool in = i < cnt;
        key[s] = key_of_bits(__float_as_uint(a[in ? i : 0u]));
        const uint32_t bin = key[s] >> kL1Shift;
        if (in && bin >= bin_p) mp |= 1u << s;
        if (in && bin <= bin_n) mn |= 1u << s;
    }
    append_candidates<PER>(key, mp, mn, e0, d, &st[t], cand, &runs[c], scratch, base);
}

}  // namespace sbc
