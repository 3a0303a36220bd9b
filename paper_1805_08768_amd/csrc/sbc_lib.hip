// libsbc: host side of the C ABI declared in include/sbc.h.  Validates arguments, lays the
// call's tensors out as a table of chunks, and enqueues the kernels on the caller's stream.
// No device memory is allocated outside sbc_create().
#include "../../include/sbc.h"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <new>
#include <numeric>
#include <vector>

#include "sbc_accumulate_kernels.hpp"
#include "sbc_threshold_kernels.hpp"
#include "sbc_encode_kernels.hpp"
#include "sbc_decode_kernels.hpp"
#include "sbc_step_kernels.hpp"
#include "sbc_average_kernels.hpp"

using namespace sbc;

namespace {
// kernels of sbc_compress in launch order (the histogram path repeats some of them)
enum Stage { kStSample = 0, kStAccumulate, kStWide, kStThreshold, kStApply, kStTensorScan, kStEmit,
             kStGather, kNumStages };
const char* const kStageNames[kNumStages] = {
    "k_sample_thresholds", "k_client_step", "k_wide_* (sweeps over long lists)", "k_threshold",
    "k_apply", "k_tensor_scan", "k_emit", "k_finish_message"};
}  // namespace

constexpr int kComputeUnits = 256;
constexpr int kDescSlots = 4;             // device copies of the tensor table, keyed by the pointer lists
constexpr uint32_t kAvgAloneChunks = 1024;  // (8.4e6 entries) beyond these, one message alone is added to the cleared result
constexpr uint32_t kMaxDecExtra = 512;    // additional decode workgroups that share a stream's scatter
constexpr uint32_t kDecSharePer = 256;    // kept entries per sharing workgroup
constexpr uint32_t kDecShareMax = kDecWaves;    // (a wavefront's updates each)
constexpr uint32_t kWideMinKept = 8192;   // kept entries from which a stream is decoded by many workgroups
// Sweeps by many workgroups narrow the lists of tensors of kWideMinKept kept entries or more down before
// k_threshold in calls whose longest list is expected beyond kLongList: a tensor of kSweepMinKept kept entries
// has lists of three times that in most calls; a sampled call's lists follow from its sample's rank; otherwise
// the call before has seen a long one (kErrLong).  (Ten tensors with 8,000 to 24,000 in the ResNet-50 shape: 25
// us for k_threshold, 31 with the sweeps.  Expecting lists of six times the kept entries in the second call of
// a run, where a residual that starts from nothing lets them grow to five to eight times: no difference.)
constexpr uint32_t kSweepMinKept = 32768;

struct DescSlot {
    bool valid = false;
    uint64_t stamp = 0;
    std::vector<const float*> dW;
    std::vector<float*> R;
};

struct sbc_ctx {
    int device = 0;
    int64_t max_elems = 0;
    int max_tensors = 0;
    uint64_t max_chunks = 0;
    uint64_t kept_cap = 0;
    uint64_t stage_cap = 0;

    // ---- device scratch of sbc_compress ----
    TensorDesc* d_desc = nullptr;         // kDescSlots tables of max_tensors entries
    uint2* d_chunk_tensor = nullptr;      // chunk -> (tensor, the tensor's first chunk)
    uint2* d_sched = nullptr;             // workgroup of k_client_step -> (chunk, tensor)
    GroupState* d_group = nullptr;        // per group of chunks: candidate and completion counters
    uint64_t max_groups = 0;
    bool compact = false;                 // candidate lists of a few times k entries instead of n
    uint64_t cand_entries = 0;            // entries d_cand holds
    uint32_t* d_order = nullptr;
    uint32_t* d_hist = nullptr;
    TensorState* d_state = nullptr;
    unsigned long long* d_counters = nullptr;   // kSegs per tensor: candidates in each segment of its lists (zero between calls)
    uint32_t* d_cand = nullptr;           // the lists' keys, then their indexes
    CandPtr cand() const { return {d_cand, (cand_entries + 5u) & ~1ull}; }      // (a few more: k_threshold reads four at a time)
    ChunkRun* d_runs = nullptr;           // per chunk: where its candidates lie
    uint32_t* d_bitmap = nullptr;
    uint32_t* d_stage = nullptr;
    uint32_t* d_kept = nullptr;
    ChunkSummary* d_sum = nullptr;
    uint32_t* d_head = nullptr;           // per chunk whose codes do not fit its words: the first word of them
    uint32_t* d_gap = nullptr;            // per chunk: gap before its first kept entry (calls of very many chunks)
    uint64_t* d_bitoff = nullptr;
    TileSummary* d_tile = nullptr;        // per tile of kScanTile chunks of a tensor
    unsigned long long* d_flow = nullptr; // what the workgroups of k_emit_all leave for one another (see flow())
    uint32_t flow_tag = 0;                // number of its latest launch, 1 to 0xFFFF
    uint32_t flow_sides = 0, flow_taken = 0;      // workgroups of its launches that select sides / take chunks
    size_t flow_words() const { return kGroupWords * (size_t)kEmitGroups + 2u * kSideWords * (size_t)std::min<int64_t>(max_tensors, kEmitAllTensors) + 1u; }
    StepFlow flow() const {
        const size_t T = (size_t)std::min<int64_t>(max_tensors, kEmitAllTensors);
        StepFlow f;
        f.groups = d_flow;
        f.sides = f.groups + kGroupWords * (size_t)kEmitGroups;
        f.started = reinterpret_cast<uint32_t*>(f.sides + 2u * kSideWords * T);
        f.sides_before = flow_sides; f.taken = flow_taken;
        f.tag = flow_tag;
        return f;
    }
    ResultBlock* d_result = nullptr;      // two for compress, two for decode, used in turn; [4] collects the
                                          // errors of decode calls whose status is deferred, [5] is a spare
    // sweeps over long lists
    WideState* d_wide_state = nullptr;
    uint32_t* d_wide_hist = nullptr;
    long long* d_wide_acc = nullptr;

    // ---- device scratch of sbc_decompress_accumulate ----
    DecBlock* d_dec_blocks = nullptr;     // what each workgroup of the decode kernel works on
    unsigned long long* d_seg_pack = nullptr;
    uint4* d_tile_fn = nullptr;
    unsigned long long* d_tile_sum = nullptr;
    uint64_t dec_seg_cap = 0, dec_tile_cap = 0;

    // ---- ... and of sbc_decompress_average (positions and marks go to the candidate lists' space) ----
    AvgTensor* d_avg_tensor = nullptr;    // followed by the streams of each decoding workgroup
    AvgTensor* h_avg_tensor = nullptr;
    uint2* d_avg_chunk = nullptr;         // chunk -> (tensor, its first chunk)
    uint2* h_avg_chunk = nullptr;
    bool avg_valid = false;
    double avg_p = 0.0;
    std::vector<float*> avg_out;
    std::vector<int64_t> avg_numel;
    uint32_t avg_blocks = 0, avg_chunks = 0, avg_pos = 0;
    uint64_t avg_marks = 0;
    hipEvent_t ev_average = nullptr;      // the end of the last such call's last kernel,
    bool avg_running = false;             // which may not have come when the call returns
    bool avg_clears = false;              // the chunk table holds the call's tensors
    bool avg_fits = false;                // and no stream is too long for one workgroup

    // ---- pinned host staging ----
    TensorDesc* h_desc = nullptr;
    uint2* h_chunk_tensor = nullptr;
    uint2* h_sched = nullptr;
    uint32_t* h_order = nullptr;
    WideIds wide_ids = {};
    int max_wide = 0;
    unsigned long long* h_result = nullptr;       // compress: see publish
    unsigned long long* h_result_dev = nullptr;   // ... as the device addresses it
    uint32_t result_seq = 0;              // number of the latest launch of the kernel that completes the message
    unsigned long long* h_result_dec = nullptr;   // decode (its own: a decode call may come between begin and end)
    unsigned long long* h_result_dec_dev = nullptr;
    uint32_t dec_seq = 0;
    DecBlock* h_dec_blocks = nullptr;
    uint32_t n_dec_blocks = 0;
    DecWides dec_wides = {};              // long streams decoded tile by tile
    TensorState* h_state = nullptr;

    // ---- plan of the last compress call: everything that depends on sizes and p only ----
    bool cache_valid = false; int cache_T = 0; double cache_p = 0.0;
    std::vector<int64_t> cache_numel;
    uint64_t cache_total = 0, cache_chunks = 0, cache_stage_words = 0, cache_kept_total = 0, cache_max_bound = 0;
    uint32_t cache_scan_tiles = 1;        // most tiles of the chunk scan that a tensor has
    bool cache_all_inline = false;        // every tensor is finished inside the streaming kernel
    int cache_force_exact = 0;
    std::vector<TensorDesc> plan;         // without the pointers
    std::vector<uint32_t> plan_order;
    int n_wide = 0;                       // tensors whose lists the sweeps can take, and which calls have sweeps:
    bool sweep_always = false, sweep_sampled = false;      // all; those that sample
    uint32_t wide_blocks = 0;
    DescSlot slot[kDescSlots];            // which pointer lists the device tables hold
    uint64_t slot_clock = 0;

    // ---- what the decode tables currently hold ----
    int dev_dec_T = 0;
    bool dev_dec_valid = false;
    double dec_p = 0.0;
    uint32_t dec_tiles = 0;
    std::vector<float*> dec_out;
    std::vector<int64_t> dec_numel;

    // ---- options ----
    int force_exact = 0;
    int carry_keys = 1;
    int carry_stale_run = 0;                 // sampled calls in a row that found the previous call's keys stale
    int carry_backoff = 0, carry_hold = 0;   // sampled calls after a call whose carried keys let a flood pass
    uint32_t flow_looks = kFlowLooks;     // (tests lower it)
    int fused_step = 0;                   // the streaming kernel finishes the tensors it can by itself
    int sampled = 0;                      // subsampled variant: the sampled threshold decides what is kept
    int defer_decode = 0;                 // decode calls return once enqueued; sbc_decode_status reports
    bool deferred_pending = false;        // some deferred decode has not been waited for yet
    bool deferred_dirty = true;           // block [4] must be cleared before the next deferred decode
    uint32_t wide_min_kept = kWideMinKept;
    bool sweep_all = false;               // tensors that keep that many have sweeps in every call

    // filter keys carried over from the previous successful call (same tensor sizes, same p)
    bool hist_valid = false;
    bool hist_long = false;               // that call had a long list
    double hist_p = 0.0;
    std::vector<uint32_t> hist_n;

    // result blocks: calls alternate between two, and a kernel of each call clears the other one
    int result_idx = 0;
    bool result_dirty = true;             // the next compress call must clear its result blocks itself
    int dec_result_idx = 0;
    bool dec_result_dirty = true;

    // optional per-kernel timing: start/stop events of the dispatches
    int profile_level = 0;
    hipEvent_t ev[2 * kNumStages] = {};
    bool ev_ok = false;
    hipEvent_t ev_result = nullptr;       // recorded behind the copy of a client step's result block
    const char* emit_name = "k_emit";     // the kernel that completed the latest step's message
    double stage_ms[kNumStages] = {};
    int64_t stage_calls[kNumStages] = {};

    // a client step that has been enqueued (sbc_compress_begin) and not yet completed
    struct Pending {
        bool active = false;
        hipStream_t stream = nullptr;
        int T = 0, b = 0, slot = 0, force_exact = 0, carry = 0;
        double p = 0.0;
        bool slot_is_new = false, use_history = false, sampled = false, all_inline = false, sweeps = false;
        bool in_one = false;          // k_emit_all completes the step
        bool left = false;            // ... and has not applied every tensor that it has selected
        bool wait_on_event = false;   // begin/end form: the wait ends with this step, not with the stream
        bool timed[kNumStages] = {};
        ResultBlock* res_now = nullptr;
        ResultBlock* res_next = nullptr;
        TensorDesc* d_desc = nullptr;
        uint8_t* msg8 = nullptr;
        size_t msg_capacity = 0, need = 0;
        uint32_t n_chunks = 0;
        unsigned gather_y = 1, scan_tiles = 1;
    } pend;

    // last compress call, for the inspection entry points
    int last_T = 0, last_b = 0;
    bool last_ok = false;
    bool last_used_exact_path = false;
    bool last_used_history = false;
    bool last_used_wide = false;
    bool last_loose = false;
    bool last_deferred = false;
    std::chrono::steady_clock::time_point last_begin;     // when it was enqueued
    hipStream_t last_stream = nullptr;    // stream of the last client step (its last kernel may still be draining)
};

namespace {

constexpr double kPhi = 1.6180339887498948482;

struct DeviceGuard {
    int prev = -1;
    bool changed = false;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) == hipSuccess && prev != dev) changed = (hipSetDevice(dev) == hipSuccess);
    }
    ~DeviceGuard() { if (changed) (void)hipSetDevice(prev); }
};

int bstar_of(double p) {
    const double b = 1.0 + std::floor(std::log2(std::log(kPhi - 1.0) / std::log(1.0 - p)));
    if (b < 0.0) return 0;
    return (int)b;
}

bool valid_p(double p) { return p > 0.0 && p < 1.0; }

int64_t kept_of(int64_t n, double p) {
    int64_t k = (int64_t)std::floor(p * (double)n);
    if (k < 1) k = 1;
    if (k > n) k = n;
    return k;
}

// Most entries a side may keep: k, or in the subsampled variant min(n, 2k + 64).
int64_t cap_of(int64_t n, int64_t k, bool sampled) {
    return sampled ? std::min<int64_t>(n, 2 * k + 64) : k;
}

uint64_t bound_words_of(int64_t n, int64_t k, int b) {
    const uint64_t bits = (uint64_t)k * (uint64_t)(1 + b) + ((uint64_t)(n - k) >> b);
    return (bits + 31) >> 5;
}

template <typename T>
hipError_t dev_alloc(T** p, size_t count) { return hipMalloc(reinterpret_cast<void**>(p), count * sizeof(T)); }
template <typename T>
hipError_t host_alloc(T** p, size_t count) { return hipHostMalloc(reinterpret_cast<void**>(p), count * sizeof(T), hipHostMallocDefault); }

void free_all(sbc_ctx* c) {
    (void)hipFree(c->d_desc); (void)hipFree(c->d_chunk_tensor); (void)hipFree(c->d_sched); (void)hipFree(c->d_group); (void)hipFree(c->d_order); (void)hipFree(c->d_hist);
    (void)hipFree(c->d_state); (void)hipFree(c->d_counters); (void)hipFree(c->d_cand); (void)hipFree(c->d_bitmap); (void)hipFree(c->d_stage);
    (void)hipFree(c->d_kept); (void)hipFree(c->d_sum); (void)hipFree(c->d_head); (void)hipFree(c->d_gap); (void)hipFree(c->d_bitoff); (void)hipFree(c->d_tile);
    (void)hipFree(c->d_flow); (void)hipFree(c->d_result); (void)hipFree(c->d_dec_blocks);
    if (c->h_dec_blocks) (void)hipHostFree(c->h_dec_blocks);
    (void)hipFree(c->d_seg_pack); (void)hipFree(c->d_tile_fn); (void)hipFree(c->d_tile_sum);
    (void)hipFree(c->d_wide_state); (void)hipFree(c->d_wide_hist); (void)hipFree(c->d_wide_acc); (void)hipFree(c->d_runs);
    if (c->h_desc) (void)hipHostFree(c->h_desc);
    if (c->h_chunk_tensor) (void)hipHostFree(c->h_chunk_tensor);
    if (c->h_sched) (void)hipHostFree(c->h_sched);
    (void)hipFree(c->d_avg_tensor); (void)hipFree(c->d_avg_chunk);
    if (c->h_avg_tensor) (void)hipHostFree(c->h_avg_tensor);
    if (c->h_avg_chunk) (void)hipHostFree(c->h_avg_chunk);
    if (c->h_order) (void)hipHostFree(c->h_order);
    if (c->h_result) (void)hipHostFree(c->h_result);
    if (c->h_result_dec) (void)hipHostFree(c->h_result_dec);
    if (c->h_state) (void)hipHostFree(c->h_state);
    if (c->ev_ok) for (hipEvent_t e : c->ev) (void)hipEventDestroy(e);
    if (c->ev_result) (void)hipEventDestroy(c->ev_result);
    if (c->ev_average) (void)hipEventDestroy(c->ev_average);
    c->ev_result = c->ev_average = nullptr;
    c->ev_ok = false;
}

int status_of_err(uint32_t err) {
    if (err & kErrInternal) return SBC_EINTERNAL;
    if (err & kErrNonFinite) return SBC_ENONFINITE;
    if (err & kErrOverflow) return SBC_ECAPACITY;
    if (err & kErrCorrupt) return SBC_ECORRUPT;
    return SBC_OK;
}

// Kernels are timed only when profiling was asked for: the launch then carries a start and a
// stop event that take the dispatch's own begin and end time stamps (event 2s and 2s+1 for
// stage s), so the figure is the kernel's duration without the gaps between dispatches.
// Expects c (context), lvl (profile level), stream and timed[] in scope.
#define SBC_LAUNCH(stage, on, kernel, grid, block, ...) SBC_LAUNCH_LDS(stage, on, kernel, grid, block, 0, __VA_ARGS__)
#define SBC_LAUNCH_LDS(stage, on, kernel, grid, block, lds, ...)                                           \
    do {                                                                                                   \
        if ((on) && (lvl >= 2 || (lvl == 1 && ((stage) == kStAccumulate || (stage) == kStSample)))) {      \
            hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, c->ev[2 * (stage)], c->ev[2 * (stage) + 1], 0, \
                                  __VA_ARGS__);                                                            \
            timed[stage] = true;                                                                           \
        } else {                                                                                           \
            hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__);                             \
        }                                                                                                  \
    } while (0)

// From the candidate lists to the message, for the pending client step: thresholds and sums (pass
// 0: of every tensor the streaming kernel has not finished itself; pass 1: of those handed over),
// side decision, residual update and bitmap, Alg. 3, message assembly.
void launch_selection_and_encode(sbc_ctx* c, int pass) {
    sbc_ctx::Pending& P = c->pend;
    const bool profile = pass == 0;
    const int lvl = c->profile_level;
    hipStream_t stream = P.stream;
    bool* timed = P.timed;
    const int T = P.T, b = P.b;
    if (pass != 0 || !P.all_inline) {
        const bool sweeps = pass == 0 && P.sweeps;
        if (sweeps) {
            const dim3 sweep(c->wide_blocks, 2u * (unsigned)c->n_wide);
            if (lvl >= 2) {
                hipExtLaunchKernelGGL(k_wide_count, sweep, dim3(kWideThreads), 0, stream, c->ev[2 * kStWide], nullptr, 0,
                                      P.d_desc, c->wide_ids, c->d_state, c->d_counters, c->cand(), c->d_wide_hist, c->d_wide_acc, c->d_wide_state);
                hipExtLaunchKernelGGL(k_wide_collect, sweep, dim3(kWideThreads), 0, stream, nullptr, c->ev[2 * kStWide + 1], 0,
                                      P.d_desc, c->wide_ids, c->d_state, c->d_counters, c->cand(), c->d_bitmap, c->d_wide_hist, c->d_wide_acc,
                                      c->d_wide_state);
                timed[kStWide] = true;
            } else {
                hipLaunchKernelGGL(k_wide_count, sweep, dim3(kWideThreads), 0, stream, P.d_desc, c->wide_ids, c->d_state,
                                   c->d_counters, c->cand(), c->d_wide_hist, c->d_wide_acc, c->d_wide_state);
                hipLaunchKernelGGL(k_wide_collect, sweep, dim3(kWideThreads), 0, stream, P.d_desc, c->wide_ids, c->d_state,
                                   c->d_counters, c->cand(), c->d_bitmap, c->d_wide_hist, c->d_wide_acc, c->d_wide_state);
            }
        }
        // (c->d_order: see compress_begin)
        const uint32_t* const order = T > kComputeUnits / 2 ? c->d_order : nullptr;
        const dim3 per_chunk((P.n_chunks + kEncWaves - 1u) / kEncWaves), block(kEncThreads);
        if (P.in_one && pass == 0) {
            // the rest of the step in one launch
            if (++c->flow_tag > kTagMask) {
                // the numbers start over: none of the words that launches have left may carry one of them
                c->flow_tag = 1u;
                hipLaunchKernelGGL(k_zero_words, dim3(64), dim3(256), 0, stream, reinterpret_cast<uint32_t*>(c->d_flow), 2ull * c->flow_words());
                c->flow_sides = c->flow_taken = 0u;
            }
            const StepSweeps swept = {c->d_wide_state, c->d_wide_hist, c->d_wide_acc, sweeps ? 1 : 0};
            const StepChunks chunks = {c->d_chunk_tensor, c->d_runs, c->d_bitmap, c->d_sum, c->d_head, c->cand_entries};
            const StepSizes sizes = {T, b, P.n_chunks, P.carry, c->flow_looks};
            const auto launch = [&](auto kernel, uint32_t per) {
                const uint32_t takers = (P.n_chunks + per - 1u) / per;
                SBC_LAUNCH(kStEmit, profile, kernel, dim3(2u * (unsigned)T + takers), dim3(kEmitThreads), P.d_desc, order,
                           c->d_state, c->d_counters, c->cand(), swept, chunks, c->flow(), sizes, P.msg8, (uint64_t)P.msg_capacity, P.res_now,
                           P.res_next, c->h_result_dev, ++c->result_seq);
                c->flow_sides += 2u * (unsigned)T; c->flow_taken += takers;
            };
            if (P.n_chunks <= kEmitFew) launch(k_emit_all<8u>, 8u);
            else launch(k_emit_all<16u>, 16u);
            return;
        }
        const bool pairs = pass != 0 && c->fused_step;     // (of the tensors that are left, some may have lists in pairs)
        const auto threshold = pairs ? k_threshold<true> : k_threshold<false>;
        const auto apply = pairs ? k_apply<true> : k_apply<false>;
        SBC_LAUNCH(kStThreshold, profile, threshold, dim3(2u * (unsigned)T), dim3(kThThreads), P.d_desc, order, c->d_state, c->d_counters,
                   c->cand(), c->d_bitmap, c->d_wide_state, c->d_wide_hist, c->d_wide_acc, pass, sweeps ? 1 : 0, P.carry, P.res_now);
        SBC_LAUNCH(kStApply, profile, apply, per_chunk, block, P.d_desc, c->d_chunk_tensor, c->d_runs, c->d_state, c->d_state,
                   c->cand(), c->cand_entries, c->d_bitmap, c->d_sum, c->d_head, b, P.left ? kPassAll : pass, P.n_chunks, P.res_now);
        if (!c->fused_step && P.n_chunks <= kScanAllChunks) {
            // (the workgroups that write the codes scan the summaries of all chunks themselves.  Two sizes: few chunks want
            // many small workgroups, the scan over many wants large ones.)
            const size_t lds = 2u * sizeof(uint32_t) * P.n_chunks;
            const auto launch = [&](auto kernel, unsigned threads) {
                SBC_LAUNCH_LDS(kStEmit, profile, kernel, dim3((P.n_chunks + threads / 64u - 1u) / (threads / 64u)), dim3(threads), lds, c->d_chunk_tensor,
                               c->d_sum, c->d_bitmap, c->d_head, c->d_state, c->d_counters, T, b, P.n_chunks, P.msg8, (uint64_t)P.msg_capacity,
                               P.res_now, P.res_next, c->h_result_dev, ++c->result_seq);
            };
            if (P.n_chunks <= kScanFew) launch(k_emit_scan<256>, 256u);
            else launch(k_emit_scan<1024>, 1024u);
            return;
        }
        if (P.scan_tiles > 1)
            hipLaunchKernelGGL(k_tile_summary, dim3(T, P.scan_tiles), dim3(kScanThreads), 0, stream, P.d_desc, c->d_state,
                               c->d_sum, c->d_tile, b, pass);
        SBC_LAUNCH(kStTensorScan, profile, k_tensor_scan, dim3(T, P.scan_tiles), dim3(kScanThreads), P.d_desc, c->d_sum,
                   c->d_tile, c->d_gap, c->d_bitoff, c->d_state, b, pass, P.res_now);
        if (!c->fused_step) {
            SBC_LAUNCH(kStEmit, profile, k_emit<true>, per_chunk, block, P.d_desc, c->d_chunk_tensor, c->d_sum, c->d_bitmap, c->d_head,
                       c->d_gap, c->d_bitoff, c->d_state, c->d_counters, T, b, pass, P.n_chunks, c->d_stage, P.msg8, (uint64_t)P.msg_capacity, P.res_now,
                       P.res_next, c->h_result_dev, ++c->result_seq);
            return;
        }
        SBC_LAUNCH(kStEmit, profile, k_emit<false>, per_chunk, block, P.d_desc, c->d_chunk_tensor, c->d_sum, c->d_bitmap, c->d_head,
                   c->d_gap, c->d_bitoff, c->d_state, c->d_counters, T, b, pass, P.n_chunks, c->d_stage, P.msg8, (uint64_t)P.msg_capacity, P.res_now,
                   P.res_next, c->h_result_dev, 0u);
    }
    SBC_LAUNCH(kStGather, profile, k_finish_message, dim3(T, P.gather_y), dim3(256), P.d_desc, c->d_state, T, b,
               c->d_stage, c->d_kept, c->d_group, P.msg8, (uint64_t)P.msg_capacity, P.res_now, P.res_next,
               c->h_result_dev, ++c->result_seq);
}

// The last average returned when its status was known, before its last kernel had ended: what works on the context's
// scratch comes after that.  An event of the context's own stands for that kernel, for its stream may be gone
// by now.  (Where the caller records a graph on this stream, which must not wait for anything outside, the host waits;
// in that thread only the relaxed mode admits to look at events.)
int settle_average(sbc_ctx* c, hipStream_t stream) {
    if (!c->avg_running) return SBC_OK;
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    hipError_t e = hipEventQuery(c->ev_average);
    if (e == hipErrorNotReady) {
        (void)hipGetLastError();
        hipStreamCaptureStatus recording = hipStreamCaptureStatusNone;
        e = hipStreamIsCapturing(stream, &recording);
        if (e == hipSuccess && recording == hipStreamCaptureStatusNone) {
            e = hipStreamWaitEvent(stream, c->ev_average, 0);          // (still running for calls on further streams)
        } else if (e == hipSuccess) {
            e = hipEventSynchronize(c->ev_average);
            c->avg_running = false;
        }
    } else {
        c->avg_running = false;
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e == hipSuccess) return SBC_OK;
    (void)hipGetLastError();
    c->avg_running = false;                               // (no call fails for it twice)
    return SBC_EHIP;
}

// The pending step's result block on its way to the host / waited for.
int enqueue_result_copy(sbc_ctx* c) {
    if (hipGetLastError() != hipSuccess) return SBC_EHIP;
    // In the begin/end form an event lets the wait end when this step is done, whatever the caller
    // has enqueued behind it; the one-call form waits for the stream, which is cheaper.
    // (the step's last kernel sends the result to pinned host memory itself)
    if (hipGetLastError() != hipSuccess ||
        (c->pend.wait_on_event && hipEventRecord(c->ev_result, c->pend.stream) != hipSuccess)) {
        (void)hipGetLastError();
        return SBC_EHIP;
    }
    return SBC_OK;
}

// The call's result in pinned host memory (see publish).
uint32_t result_seq_of(unsigned long long w) { return (uint32_t)(w >> 50); }
uint32_t result_err_of(unsigned long long w) { return (uint32_t)(w >> 40) & 0x3FFu; }
uint64_t result_bytes_of(unsigned long long w) { return w & ((1ull << 40) - 1ull); }

// Looks for sequence number `want` there for up to 0.3 ms.
bool result_arrived(const unsigned long long* word, uint32_t want) {
    const auto t0 = std::chrono::steady_clock::now();
    for (int spin = 0;; ++spin) {
        if (result_seq_of(__atomic_load_n(word, __ATOMIC_ACQUIRE)) == (want & kSeqMask)) return true;
        if ((spin & 63) == 63 && std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(300)) return false;
    }
}

// Until the result numbered `seq` is there.  Looking for the number takes a microsecond or two once it is,
// where the runtime's wait (for the event, or without one for the stream) returns several microseconds after
// the stream has drained; calls that run longer than a fraction of a millisecond fall through to that wait.
// A kernel that has ended without sending its result has found an invariant violated: the word then still
// holds the call before's.
int wait_result(const unsigned long long* word, uint32_t seq, bool look, hipStream_t stream, hipEvent_t event = nullptr) {
    if (look && result_arrived(word, seq)) return SBC_OK;
    if ((event ? hipEventSynchronize(event) : hipStreamSynchronize(stream)) != hipSuccess) {
        (void)hipGetLastError();
        return SBC_EHIP;
    }
    return result_seq_of(__atomic_load_n(word, __ATOMIC_ACQUIRE)) == (seq & kSeqMask) ? SBC_OK : SBC_EINTERNAL;
}

// The pending step's result.  (Not looked for while kernels carry timing events: those are read right after
// this, and must be complete.)
int wait_result(sbc_ctx* c) {
    return wait_result(c->h_result, c->result_seq, c->profile_level == 0, c->pend.stream, c->pend.wait_on_event ? c->ev_result : nullptr);
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// Server step without any allocation, for callers that cannot call hipMalloc (code under HIP graph
// capture, tight serving loops, harnesses that forbid allocation).  What the decode kernel works on
// travels in its arguments, and its errors go straight to the caller's status word, which a dispatch
// of one thread sets to SBC_OK before it.  Nothing is copied to or from the host and nothing waits.
// ---------------------------------------------------------------------------------------------
namespace {

// What the decode kernel of the context-free call works on, in its arguments (4 KiB at the most).
struct ArgBlocks {
    float* out[SBC_NOALLOC_MAX_TENSORS];
    uint32_t n[SBC_NOALLOC_MAX_TENSORS];
    uint16_t block[SBC_NOALLOC_MAX_TENSORS + kMaxDecExtra];   // tensor, share and shares - 1 of a workgroup in 8 + 3 + 3 bits
    int32_t* status;
    __device__ __forceinline__ DecBlock at(uint32_t i) const {
        const uint32_t v = block[i], t = v & 255u;
        DecBlock b;
        b.out = out[t]; b.n = n[t]; b.t = t; b.share = (v >> 8) & 7u; b.shares = ((v >> 11) & 7u) + 1u;
        return b;
    }
    __device__ __forceinline__ ResultBlock* errors() const { return nullptr; }
    __device__ __forceinline__ int32_t* status_word() const { return status; }
    __device__ __forceinline__ void begin() const {}
};
static_assert(SBC_NOALLOC_MAX_TENSORS <= 256 && kDecShareMax <= 8, "a workgroup's word holds its numbers");
static_assert(sizeof(ArgBlocks) <= 4096 - 256, "must fit the kernel argument segment");
constexpr int kNoAllocMaxDevices = 64;

__global__ void k_status_ok(int32_t* __restrict__ status) { if (threadIdx.x == 0) *status = SBC_OK; }

// The decode kernel for b.
template <typename Blocks, typename Wides>
void launch_decode(hipStream_t stream, uint32_t n_blocks, uint32_t n_tiles, const uint8_t* msg, unsigned long long msg_bytes,
                   const Blocks& blocks, int T, int b, float scale, const Wides& dw, uint4* tile_fn) {
    const dim3 grid(n_blocks + n_tiles), block(kDecThreads);
    if (b <= 7) hipLaunchKernelGGL((k_decode<2, Blocks, Wides>), grid, block, 0, stream, msg, msg_bytes, blocks, n_blocks, T, b, scale, dw, tile_fn);
    else if (b <= 11) hipLaunchKernelGGL((k_decode<3, Blocks, Wides>), grid, block, 0, stream, msg, msg_bytes, blocks, n_blocks, T, b, scale, dw, tile_fn);
    else if (b <= kPackedMaxB) hipLaunchKernelGGL((k_decode<4, Blocks, Wides>), grid, block, 0, stream, msg, msg_bytes, blocks, n_blocks, T, b, scale, dw, tile_fn);
    else hipLaunchKernelGGL((k_decode_generic<Blocks>), grid, block, 0, stream, msg, msg_bytes, blocks, T, b, scale);
}

uint32_t decode_shares(int64_t kept) {
    return (uint32_t)std::min<int64_t>(kDecShareMax, std::max<int64_t>(1, kept / kDecSharePer));
}

}  // namespace

#ifdef SBC_PHASE_TIMING
#include <chrono>
static double g_host_ts[16];
#define SBC_HOST_TS(i) (g_host_ts[i] = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now().time_since_epoch()).count())
#else
#define SBC_HOST_TS(i) ((void)0)
#endif

extern "C" {

const char* sbc_strerror(int code) {
    switch (code) {
        case SBC_OK: return "ok";
        case SBC_EINVAL: return "invalid argument";
        case SBC_ECAPACITY: return "buffer or context too small";
        case SBC_EHIP: return "HIP runtime error";
        case SBC_ECORRUPT: return "corrupt message";
        case SBC_ENONFINITE: return "non-finite accumulated update";
        case SBC_EINTERNAL: return "internal invariant violated";
        default: return "unknown status";
    }
}

int sbc_golomb_bstar(double p) {
    if (!valid_p(p)) return SBC_EINVAL;
    return bstar_of(p);
}

int64_t sbc_num_kept(int64_t numel, double p) {
    if (!valid_p(p) || numel < 1) return SBC_EINVAL;
    return kept_of(numel, p);
}

static size_t msg_bound(const int64_t* numel, int n_tensors, double p, bool sampled) {
    if (!numel || n_tensors <= 0 || !valid_p(p)) return 0;
    const int b = bstar_of(p);
    if (b > kMaxB) return 0;
    uint64_t words = 0;
    for (int t = 0; t < n_tensors; ++t) {
        if (numel[t] < 1 || numel[t] >= (int64_t)1 << 32) return 0;
        words += bound_words_of(numel[t], cap_of(numel[t], kept_of(numel[t], p), sampled), b);
    }
    return (size_t)(32 + 24ull * (unsigned)n_tensors + 4ull * words);
}

size_t sbc_msg_bound(const int64_t* numel, int n_tensors, double p) { return msg_bound(numel, n_tensors, p, false); }

size_t sbc_msg_bound_sampled(const int64_t* numel, int n_tensors, double p) { return msg_bound(numel, n_tensors, p, true); }

static int create_context(sbc_ctx** out, int device, int64_t max_total_elems, int max_tensors, bool compact) {
    if (!out || max_total_elems < 1 || max_tensors < 1 || max_tensors >= (1 << 24)) return SBC_EINVAL;
    *out = nullptr;
    int n_dev = 0;
    if (hipGetDeviceCount(&n_dev) != hipSuccess) return SBC_EHIP;
    if (device < 0 || device >= n_dev) return SBC_EINVAL;
    sbc_ctx* c = new (std::nothrow) sbc_ctx();
    if (!c) return SBC_EHIP;
    c->device = device;
    c->max_elems = max_total_elems;
    c->max_tensors = max_tensors;
    c->compact = compact;
    // full: both sides' lists of every tensor hold every entry; compact: half an entry per entry in all
    // (plus the lists' fixed part), shared out by the plan of each call
    c->cand_entries = compact ? (uint64_t)max_total_elems / 2 + 2048ull * (uint64_t)max_tensors : 2ull * (uint64_t)max_total_elems;
    c->cand_entries = std::max<uint64_t>(c->cand_entries, 128u);      // (k_apply reads a run's first 64 ahead)
    c->max_chunks = (uint64_t)max_total_elems / kChunk + (uint64_t)max_tensors;
    c->kept_cap = std::min<uint64_t>((uint64_t)max_total_elems, (uint64_t)std::max(kInlineMaxK, kSmallMaxN) * (uint64_t)max_tensors);
    // A tensor's stream is at most k(1+b*) + (n-k)/2^b* bits, which stays below 1.3 n for every p
    // (b* shrinks as p grows); n/16 words plus rounding per tensor is ample, and sbc_compress
    // checks the actual need against this capacity.
    c->stage_cap = (uint64_t)max_total_elems / 16 + 64ull * (uint64_t)max_tensors + 64ull;
    DeviceGuard guard(device);
    const size_t T = (size_t)max_tensors;
    bool ok = true;
    ok = ok && dev_alloc(&c->d_desc, (size_t)kDescSlots * T) == hipSuccess;
    ok = ok && dev_alloc(&c->d_chunk_tensor, (size_t)c->max_chunks) == hipSuccess;
    c->max_groups = c->max_chunks / kGroupChunks + (uint64_t)max_tensors;
    ok = ok && dev_alloc(&c->d_sched, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && dev_alloc(&c->d_group, (size_t)c->max_groups) == hipSuccess;
    ok = ok && hipMemset(c->d_group, 0, sizeof(GroupState) * c->max_groups) == hipSuccess;
    ok = ok && host_alloc(&c->h_sched, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && dev_alloc(&c->d_order, T) == hipSuccess;
    ok = ok && dev_alloc(&c->d_hist, T * kL1Bins) == hipSuccess;
    ok = ok && dev_alloc(&c->d_state, T) == hipSuccess;
    ok = ok && hipMemset(c->d_state, 0, sizeof(TensorState) * T) == hipSuccess;
    ok = ok && dev_alloc(&c->d_counters, T * kSegs * kCounterStride) == hipSuccess;
    ok = ok && hipMemset(c->d_counters, 0, sizeof(unsigned long long) * T * kSegs * kCounterStride) == hipSuccess;
    ok = ok && dev_alloc(&c->d_cand, 2u * (size_t)c->cand_entries + 8u) == hipSuccess;       // (see cand())
    ok = ok && dev_alloc(&c->d_runs, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && dev_alloc(&c->d_bitmap, (size_t)c->max_chunks * kChunkWords) == hipSuccess;
    ok = ok && dev_alloc(&c->d_stage, (size_t)c->stage_cap) == hipSuccess;
    ok = ok && dev_alloc(&c->d_kept, (size_t)c->kept_cap) == hipSuccess;
    ok = ok && dev_alloc(&c->d_sum, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && dev_alloc(&c->d_head, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && dev_alloc(&c->d_gap, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && dev_alloc(&c->d_bitoff, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && dev_alloc(&c->d_tile, (size_t)(c->max_chunks / kScanTile) + T + 1) == hipSuccess;
    ok = ok && dev_alloc(&c->d_flow, c->flow_words()) == hipSuccess;
    ok = ok && hipMemset(c->d_flow, 0, sizeof(unsigned long long) * c->flow_words()) == hipSuccess;
    ok = ok && dev_alloc(&c->d_result, 6) == hipSuccess;
    ok = ok && dev_alloc(&c->d_dec_blocks, T + kMaxDecExtra) == hipSuccess;
    const size_t avg_room = T + (sizeof(uint32_t) * kDecWaves * (T + kMaxDecExtra) + sizeof(AvgTensor) - 1) / sizeof(AvgTensor);
    ok = ok && dev_alloc(&c->d_avg_tensor, avg_room) == hipSuccess;
    ok = ok && host_alloc(&c->h_avg_tensor, avg_room) == hipSuccess;
    ok = ok && dev_alloc(&c->d_avg_chunk, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && host_alloc(&c->h_avg_chunk, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && host_alloc(&c->h_dec_blocks, T + kMaxDecExtra) == hipSuccess;
    // tile decode: a stream of w words has w/2 segments; every stream is rounded up to whole tiles
    c->dec_seg_cap = c->stage_cap / 2 + (uint64_t)(kMaxWideDec + 1) * kDecThreads;
    c->dec_tile_cap = c->dec_seg_cap / kDecThreads + kMaxWideDec;
    ok = ok && dev_alloc(&c->d_seg_pack, (size_t)c->dec_seg_cap) == hipSuccess;
    ok = ok && dev_alloc(&c->d_tile_fn, (size_t)c->dec_tile_cap) == hipSuccess;
    ok = ok && dev_alloc(&c->d_tile_sum, (size_t)c->dec_tile_cap) == hipSuccess;
    c->max_wide = std::min(kMaxWide, max_tensors);
    ok = ok && dev_alloc(&c->d_wide_state, (size_t)c->max_wide * 2) == hipSuccess;
    ok = ok && dev_alloc(&c->d_wide_hist, (size_t)c->max_wide * 2 * kThBins) == hipSuccess;
    ok = ok && dev_alloc(&c->d_wide_acc, (size_t)c->max_wide * 2 * 256) == hipSuccess;
    // the histograms start out zero; the kernel that reads them leaves them zero
    ok = ok && hipMemset(c->d_wide_hist, 0, sizeof(uint32_t) * c->max_wide * 2 * kThBins) == hipSuccess;
    ok = ok && host_alloc(&c->h_desc, T) == hipSuccess;
    ok = ok && host_alloc(&c->h_chunk_tensor, (size_t)c->max_chunks) == hipSuccess;
    ok = ok && host_alloc(&c->h_order, T) == hipSuccess;
    ok = ok && host_alloc(&c->h_result, 1) == hipSuccess;
    ok = ok && hipHostGetDevicePointer(reinterpret_cast<void**>(&c->h_result_dev), c->h_result, 0) == hipSuccess;
    // (pinned memory may come back from an earlier context with that context's sequence number in it)
    if (ok) *c->h_result = 0ull;
    ok = ok && host_alloc(&c->h_result_dec, 1) == hipSuccess;
    ok = ok && hipHostGetDevicePointer(reinterpret_cast<void**>(&c->h_result_dec_dev), c->h_result_dec, 0) == hipSuccess;
    if (ok) *c->h_result_dec = 0ull;
    ok = ok && host_alloc(&c->h_state, T) == hipSuccess;
    if (ok) {
        int made = 0;
        for (; made < 2 * kNumStages; ++made)
            if (hipEventCreate(&c->ev[made]) != hipSuccess) break;
        if (made < 2 * kNumStages) {
            for (int i = 0; i < made; ++i) (void)hipEventDestroy(c->ev[i]);
            ok = false;
        } else {
            c->ev_ok = true;
        }
        for (hipEvent_t* ev : {&c->ev_result, &c->ev_average})
            // (ev_average orders work of this device alone: the fence for the host and other devices is the caller's
            // synchronisation, as without an event; with it 32 messages of the ResNet-50 shape take 48.6 us, without 47.0)
            if (ok && hipEventCreateWithFlags(ev, ev == &c->ev_average ? hipEventDisableTiming | hipEventDisableSystemFence : hipEventDisableTiming) != hipSuccess) {
                *ev = nullptr;
                ok = false;
            }
    }
    if (!ok) {
        (void)hipGetLastError();
        free_all(c);
        delete c;
        return SBC_EHIP;
    }
    *out = c;
    return SBC_OK;
}

int sbc_create(sbc_ctx** out, int device, int64_t max_total_elems, int max_tensors) {
    return create_context(out, device, max_total_elems, max_tensors, false);
}

int sbc_create_compact(sbc_ctx** out, int device, int64_t max_total_elems, int max_tensors) {
    return create_context(out, device, max_total_elems, max_tensors, true);
}

void sbc_destroy(sbc_ctx* c) {
    if (!c) return;
    DeviceGuard guard(c->device);
    free_all(c);
    delete c;
}

int sbc_set_option(sbc_ctx* c, int option, int value) {
    if (!c || c->pend.active) return SBC_EINVAL;      // not between sbc_compress_begin and sbc_compress_end
    switch (option) {
        case SBC_OPT_FORCE_EXACT_PATH:
            c->force_exact = value ? 1 : 0;
            c->hist_valid = false;
            c->cache_valid = false;                    // which tensors the streaming kernel finishes is part of the plan
            return SBC_OK;
        case SBC_OPT_CARRY_FILTER_KEYS:
            c->carry_keys = value ? 1 : 0; c->hist_valid = false; c->carry_backoff = c->carry_hold = 0;
            return SBC_OK;
        case SBC_OPT_FUSED_STEP:
            c->fused_step = value ? 1 : 0;
            c->hist_valid = false;
            c->cache_valid = false;                    // which tensors the streaming kernel finishes is part of the plan
            return SBC_OK;
        case SBC_OPT_SAMPLED_THRESHOLD:
            c->sampled = value ? 1 : 0;
            c->cache_valid = false;                    // the capacities of the plan depend on it
            c->dev_dec_valid = false;
            c->hist_valid = false;
            return SBC_OK;
        case SBC_OPT_DEFER_DECODE_STATUS:
            if (c->deferred_pending) return SBC_EINVAL;    // collect the outstanding status first
            c->defer_decode = value ? 1 : 0;
            return SBC_OK;
        case SBC_OPT_WIDE_MIN_KEPT:
            if (value < 0) return SBC_EINVAL;
            c->wide_min_kept = value ? (uint32_t)value : kWideMinKept;
            c->sweep_all = value != 0;
            c->cache_valid = false;                    // which tensors are wide is part of both plans
            c->dev_dec_valid = false;
            return SBC_OK;
        case SBC_OPT_WAIT_LOOKS:
            if (value < 0) return SBC_EINVAL;
            c->flow_looks = value ? (uint32_t)value : kFlowLooks;
            return SBC_OK;
        default: return SBC_EINVAL;
    }
}

// What a step's streaming pass sends past the last-level cache (no result depends on it): update and residual,
// for whatever runs until the next step, other clients' steps or a training step, displaces the residual, and
// where that has written, the cache's dirty lines leave it in the middle of this pass.  Only where the residual is read
// again before that can happen is it kept: by the histogram route of this very call, or by the next step if that follows
// at once.  That is taken from the time since the step before this one: what such a step takes by itself (12 bytes per
// entry at 6 TB/s, 40 us, 35 us per million kept entries) and 100 us, about the time of one other client's step
// and less than two of them take; in the begin/end form, where other clients' steps overlap this one's, 25 us
// (ResNet-50 shape, three clients in flight 57 us a step, with the residual kept 64).  A residual larger than the cache always goes past it, and so does the update of
// a step that does not fit it as a whole, for nobody reads that again.
// Steps of 14e6 to 66e6 entries at p = 0.001, whole ones of one client back to back and of several in turn, and the pass alone
// (us) behind other traffic, residual kept / sent past (25.6e6: the ResNet-50 shape, else one tensor; up to 22e6 the
// update kept as well):
//     entries   one client    two in turn    three         five         0.6 GiB read   0.3 GiB read and written
//     14e6       66.7 / 74.5   64.8 / 71.8   70.4 / 71.6   76.6 / 70.6    31.4 / 35.0    45.4 / 34.8
//     20e6       86.5 / 90.4   85.3 / 90.9   96.2 / 92.3   95.3 / 91.9    44.2 / 47.8    62.1 / 46.6
//     25.6e6     82.5 / 84.3   81.9 / 85.0   90.3 / 85.0   97.2 / 85.2    51.6 / 55.6    65.5 / 55.3
//     45e6      152   / 154   170   / 153   174   / 153                   87.7 / 90.4   108.0 / 91.0
//     66e6      203   / 205   222   / 200   217   / 200                  123.2 / 126.5  146.8 / 128.7
//     100e6     320   / 276   319   / 273   313   / 273                  180.3 / 186.7  218.0 / 188.8
// Steps of up to 160 MiB leave it all in the cache, where a few clients in turn still find part of it (12e6 entries: one
// client 61.7 / 63.5, three 62.5 / 65.0, eight 68.6 / 63.7).
constexpr uint64_t kCacheBytes = 256ull << 20, kKeptBytes = 160ull << 20;
// Entries from which the streaming pass has two workgroups to a compute unit instead of four (see kRun): where the residual
// goes past the cache, and where it is kept, for loads that hit the cache want more of them in flight.  Whole steps at p =
// 0.001 in us, four / two: sent past 24e6 106.2 / 104.9, 30e6 124.9 / 124.4, 45e6 152.1 / 149.0, 66e6 196 / 192; kept
// ResNet-50 shape 82.7 / 84.3, 30e6 120.6 / 125.4 (in twenty tensors 90.1 / 92.2), 45e6 151.3 / 150.3 (117.7 / 120.1), 55e6
// 169.9 / 168.5, 66e6 201 / 198.
constexpr uint64_t kPairsFrom = 24000000, kPairsKeptFrom = 55000000;
static int accumulate_past_cache(sbc_ctx* c, uint64_t total, double p, bool force_exact, bool overlapped) {
    const auto now = std::chrono::steady_clock::now();
    const std::chrono::duration<double> since = now - c->last_begin;
    c->last_begin = now;
    if (total * 12ull <= kKeptBytes) return kPastNothing;
    const double alone = (double)total * 12.0 / 6e12 + 40e-6 + p * (double)total * 35e-12;
    const bool again = force_exact || (c->last_T > 0 && since.count() <= alone + (overlapped ? 25e-6 : 100e-6));
    if (again && total * 12ull <= kCacheBytes) return kPastNothing;
    return again && total * 4ull <= kCacheBytes ? kPastUpdate : kPastAll;
}

static int compress_begin(sbc_ctx* c, void* hip_stream, const float* const* dW, float* const* residual,
                          const int64_t* numel, int n_tensors, double p, void* msg, size_t msg_capacity,
                          bool wait_on_event) {
    if (!c || !dW || !residual || !numel || !msg || n_tensors <= 0 || !valid_p(p))
        return SBC_EINVAL;
    if (c->pend.active) return SBC_EINVAL;            // one step at a time per context
    if (((uintptr_t)msg & 7u) != 0) return SBC_EINVAL;
    if (n_tensors > c->max_tensors) return SBC_ECAPACITY;
    const int T = n_tensors;
    const int b = bstar_of(p);
    if (b > kMaxB) return SBC_EINVAL;
    c->last_ok = false;
    SBC_HOST_TS(0);

    // ---- plan: tensor table, chunk numbering, staging layout ----
    // Everything but the pointers depends only on the tensor sizes and p, and is kept from call
    // to call while those stay the same.  The tensor table itself (sizes, offsets and the
    // pointers) lives in one of kDescSlots device copies keyed by the pointer lists, so a caller
    // that alternates between a few sets of buffers uploads nothing in the steady state.
    uint64_t total = 0, chunks = 0, stage_words = 0, kept_total = 0, max_bound = 0, groups = 0, cand_total = 0;
    bool all_inline = true;
    uint32_t scan_tiles = 1;
    // in the subsampled variant the keys must come from this call's sample
    const bool sampled = c->sampled != 0;
    const int force_exact = sampled ? 0 : c->force_exact;
    bool use_history = !sampled && c->hist_valid && !force_exact && !c->result_dirty && c->hist_p == p &&
                       c->hist_n.size() == (size_t)T;
    if (use_history)
        for (int t = 0; t < T; ++t) if ((int64_t)c->hist_n[t] != numel[t]) { use_history = false; break; }
    const bool sizes_same = c->cache_valid && c->cache_T == T && c->cache_p == p && c->cache_force_exact == force_exact &&
                            std::memcmp(c->cache_numel.data(), numel, sizeof(int64_t) * T) == 0;
    auto pointers_ok = [&](int t) -> bool {
        if (!dW[t] || !residual[t]) return false;
        const uintptr_t a = (uintptr_t)dW[t], r = (uintptr_t)residual[t];
        if ((a & 3u) || (r & 3u)) return false;
        const uintptr_t bytes = (uintptr_t)numel[t] * 4u;
        return !(a < r + bytes && r < a + bytes);     // dW must not overlap the residual
    };
    int slot = -1;
    if (sizes_same) {
        total = c->cache_total; chunks = c->cache_chunks; stage_words = c->cache_stage_words;
        kept_total = c->cache_kept_total; max_bound = c->cache_max_bound;
        scan_tiles = c->cache_scan_tiles;
        all_inline = c->cache_all_inline;
        for (int i = 0; i < kDescSlots; ++i) {
            const DescSlot& sl = c->slot[i];
            if (sl.valid && std::memcmp(sl.dW.data(), dW, sizeof(float*) * T) == 0 &&
                std::memcmp(sl.R.data(), residual, sizeof(float*) * T) == 0) { slot = i; break; }
        }
        if (slot < 0)
            for (int t = 0; t < T; ++t) if (!pointers_ok(t)) return SBC_EINVAL;
    } else {
        c->cache_valid = false;
        for (int i = 0; i < kDescSlots; ++i) c->slot[i].valid = false;
        if (c->plan.size() < (size_t)T) c->plan.resize(T);
        int n_wide = 0;
        // (where some tensor has sweeps, so have all that can: the launches are there anyway)
        c->sweep_always = c->sweep_sampled = false;
        uint64_t wide_longest = 0;
        for (int t = 0; t < T; ++t) {
            const int64_t n = numel[t];
            if (n < 1 || n >= (int64_t)1 << 32) return SBC_EINVAL;
            if (!pointers_ok(t)) return SBC_EINVAL;
            TensorDesc d;
            std::memset(&d, 0, sizeof(d));
            d.n = (uint32_t)n;
            d.k = (uint32_t)kept_of(n, p);
            d.kcap = (uint32_t)cap_of(n, d.k, sampled);
            d.chunk0 = (uint32_t)chunks;
            d.nchunks = (uint32_t)((n + kChunk - 1) / kChunk);
            // compact: a quarter of the tensor per side (the whole budget of half an entry per entry), more
            // if k asks for it (then the budget may not do, and the call is refused below)
            d.cand_cap = c->compact ? (uint32_t)std::min<uint64_t>((uint64_t)n, std::max<uint64_t>((uint64_t)n / 4u, 4ull * d.kcap + 1024ull))
                                    : (uint32_t)n;
            // (the streaming kernel that finishes tensors reads lists in one piece; in the subsampled variant there is no
            // second pass for a segment of a compact context that overflows)
            const bool cut = !c->fused_step && d.nchunks >= (d.cand_cap < d.n ? (sampled ? 0xFFFFFFFFu : kSegMinCompact) : kSegMinChunks);
            d.segs = cut ? kSegs : 1u;
            d.cand_off = cand_total;
            cand_total += 2ull * d.cand_cap;
            d.stage_off = stage_words;
            const uint64_t bw = bound_words_of(n, d.kcap, b);
            if (bw >= (1ull << 32)) return SBC_ECAPACITY;
            d.bound_words = (uint32_t)bw;
            // finished inside the streaming kernel: exact mode, and few enough kept entries and stream
            // words for one workgroup's LDS (a one-chunk tensor: any k, encoded from a bitmap)
            const uint32_t n_groups = (d.nchunks + kGroupChunks - 1u) / kGroupChunks;
            const bool inl = c->fused_step && !sampled && !force_exact && n_groups <= (uint32_t)kMaxGroups &&
                             (d.nchunks == 1u && d.n <= kSmallMaxN ? bw <= kSmallMaxWords
                                                                   : (d.kcap <= kInlineMaxK && bw <= kInlineMaxWords));
            d.flags = (sampled ? kDescSampled : 0u) | (inl ? kDescInline : 0u);
            all_inline = all_inline && inl;
            d.grp0 = (uint32_t)groups;
            if (inl) groups += n_groups;
            if (!inl && d.kcap >= c->wide_min_kept && n_wide < c->max_wide) {
                d.flags |= kDescWide;
                const uint32_t rank = sampled || n <= kSampleMax ? 0u : sample_rank(d.k, kSampleMax, d.n);
                const uint64_t by_sample = rank >= (uint32_t)kSampleMax ? (uint64_t)n : rank ? (uint64_t)rank * (uint64_t)n / kSampleMax : d.k;
                c->sweep_always = c->sweep_always || c->sweep_all || (!sampled && d.k >= kSweepMinKept);
                c->sweep_sampled = c->sweep_sampled || by_sample > kLongList;
                d.wide = (uint32_t)n_wide;
                c->wide_ids.id[n_wide++] = (uint32_t)t;
                wide_longest = std::max<uint64_t>(wide_longest, std::max<uint64_t>((uint64_t)n / 16u, std::min<uint64_t>((uint64_t)n, 4ull * d.k)));
            }
            d.kept_off = (uint32_t)kept_total;
            if (inl) kept_total += d.kcap;
            total += (uint64_t)n;
            chunks += d.nchunks;
            stage_words += bw;
            max_bound = std::max<uint64_t>(max_bound, bw);
            scan_tiles = std::max<uint32_t>(scan_tiles, (d.nchunks + kScanTile - 1u) / kScanTile);
            if (total > (uint64_t)c->max_elems || cand_total > c->cand_entries || chunks > c->max_chunks || kept_total > c->kept_cap ||
                stage_words > c->stage_cap || groups > c->max_groups)
                return SBC_ECAPACITY;
            c->plan[t] = d;
        }
        if (chunks >= (1ull << 31)) return SBC_ECAPACITY;
        c->n_wide = n_wide;
        // Sweeps over a candidate list: enough workgroups for four times the kept entries of the largest tensor, or a
        // sixteenth of it, as far as the chip holds those of all lists at once (512), for the ones that a list has
        // no use for cost, too: 64 for each of the ResNet-50 shape's 122 lists at p = 0.1 42 + 89 us, eight 29 + 40.
        // One tensor of 2^22 entries at p = 0.1 (64; lists of 1.0e6) 9 + 11 us, with eight 23 + 22.
        const uint64_t useful = (wide_longest + kWidePerWorkgroup - 1) / kWidePerWorkgroup, room = 256u / (unsigned)std::max(n_wide, 1);
        c->wide_blocks = (uint32_t)std::max<uint64_t>(kWideFew, std::min(useful + kWideFew - 1, room) / kWideFew * kWideFew);
    }
    const size_t need = (size_t)(32 + 24ull * (unsigned)T + 4ull * stage_words);
    if (msg_capacity < need) return SBC_ECAPACITY;

    DeviceGuard guard(c->device);
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    // The previous step returned when its size was known, possibly before its last kernel had
    // ended: a step on another stream must not touch the context's scratch before that.
    if (c->last_T > 0 && c->last_stream != stream && hipStreamSynchronize(c->last_stream) != hipSuccess) {
        (void)hipGetLastError();
        return SBC_EHIP;
    }
    if (const int rc = settle_average(c, stream)) return rc;
    if (!sizes_same) {
        // tables that depend on the sizes only: tensors by decreasing size, chunk -> tensor
        c->plan_order.resize(T);
        std::iota(c->plan_order.begin(), c->plan_order.end(), 0u);
        std::stable_sort(c->plan_order.begin(), c->plan_order.end(),
                         [&](uint32_t x, uint32_t y) { return c->plan[x].n > c->plan[y].n; });
        // k_threshold's workgroups, two per tensor: largest tensors first if there are more of them than compute
        // units; if only some compute units get two (the first ones, from the 257th workgroup on), small tensors stand
        // at both of their places, and the large ones have a compute unit each (ResNet-50 shape, 322 workgroups, in
        // the list's order, which ends with the largest: step 0.75 us more; largest first: 0.3 us more).  Only time
        // depends on where a workgroup lands.
        const int twice = T > kComputeUnits / 2 && T <= kComputeUnits ? T - kComputeUnits / 2 : 0;
        for (int i = 0; i < T; ++i) c->h_order[i] = c->plan_order[i < twice ? T - 2 * twice + i : i < T - twice ? i - twice : i];
        for (int t = 0; t < T; ++t) {
            uint2* ct = c->h_chunk_tensor + c->plan[t].chunk0;
            for (uint32_t j = 0; j < c->plan[t].nchunks; ++j) ct[j] = make_uint2((uint32_t)t, c->plan[t].chunk0);
        }
        // Order of the streaming kernel's workgroups: the one-chunk tensors it finishes on the spot
        // go first (their selection then runs beside the streaming of everything else), the others
        // follow by decreasing size, so that the tensors whose completion costs most complete early
        // and the last workgroups to finish belong to tensors with little left to do.
        if (c->fused_step) {
            uint64_t w = 0;
            for (int pass = 0; pass < 2; ++pass)
                for (int i = 0; i < T; ++i) {
                    const TensorDesc& d = c->plan[c->plan_order[i]];
                    const bool first = (d.flags & kDescInline) && d.nchunks == 1u && d.n <= kSmallMaxN;
                    if (first != (pass == 0)) continue;
                    for (uint32_t j = 0; j < d.nchunks; ++j) c->h_sched[w++] = make_uint2(d.chunk0 + j, c->plan_order[i]);
                }
        }
        if (hipMemcpyAsync(c->d_order, c->h_order, sizeof(uint32_t) * T, hipMemcpyHostToDevice, stream) != hipSuccess ||
            (c->fused_step && hipMemcpyAsync(c->d_sched, c->h_sched, sizeof(uint2) * chunks, hipMemcpyHostToDevice, stream) != hipSuccess) ||
            hipMemcpyAsync(c->d_chunk_tensor, c->h_chunk_tensor, sizeof(uint2) * chunks, hipMemcpyHostToDevice, stream) != hipSuccess) {
            (void)hipGetLastError();
            return SBC_EHIP;
        }
        c->cache_numel.assign(numel, numel + T);
        c->cache_T = T; c->cache_p = p;
        c->cache_total = total; c->cache_chunks = chunks; c->cache_stage_words = stage_words;
        c->cache_kept_total = kept_total; c->cache_max_bound = max_bound;
        c->cache_scan_tiles = scan_tiles;
        c->cache_all_inline = all_inline; c->cache_force_exact = force_exact;
        // (cache_valid is set once this call has completed: the uploads above must have happened)
    }
    bool slot_is_new = false;
    if (slot < 0) {
        // the least recently used slot receives this call's table
        slot = 0;
        for (int i = 0; i < kDescSlots; ++i) {
            if (!c->slot[i].valid) { slot = i; break; }
            if (c->slot[i].stamp < c->slot[slot].stamp) slot = i;
        }
        DescSlot& sl = c->slot[slot];
        sl.valid = false;
        for (int t = 0; t < T; ++t) {
            c->h_desc[t] = c->plan[t];
            c->h_desc[t].dW = dW[t];
            c->h_desc[t].R = residual[t];
        }
        if (hipMemcpyAsync(c->d_desc + (size_t)slot * c->max_tensors, c->h_desc, sizeof(TensorDesc) * T,
                           hipMemcpyHostToDevice, stream) != hipSuccess) {
            (void)hipGetLastError();
            return SBC_EHIP;
        }
        sl.dW.assign(dW, dW + T);
        sl.R.assign(residual, residual + T);
        slot_is_new = true;
    }
    c->slot[slot].stamp = ++c->slot_clock;
    TensorDesc* const d_desc = c->d_desc + (size_t)slot * c->max_tensors;

    uint8_t* msg8 = static_cast<uint8_t*>(msg);
    const uint32_t n_chunks = (uint32_t)chunks;
    if (c->result_dirty) {                            // after an error, or on the first call
        hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t*>(c->d_result),
                           (uint64_t)(2 * sizeof(ResultBlock) / 4));
        hipLaunchKernelGGL(k_zero_words, dim3(64), dim3(256), 0, stream, reinterpret_cast<uint32_t*>(c->d_group),
                           (uint64_t)c->max_groups * (sizeof(GroupState) / 4));
        hipLaunchKernelGGL(k_zero_words, dim3(64), dim3(256), 0, stream, reinterpret_cast<uint32_t*>(c->d_counters),
                           (uint64_t)c->max_tensors * kSegs * kCounterStride * 2u);
        // (what follows is left as it should be only if all of the call's kernels have run; k_emit_all's words are
        // clean until its first launch, whatever the number of that one)
        if (c->flow_sides | c->flow_taken)
            hipLaunchKernelGGL(k_zero_words, dim3(64), dim3(256), 0, stream, reinterpret_cast<uint32_t*>(c->d_flow), 2ull * c->flow_words());
        c->flow_sides = c->flow_taken = 0u;
        hipLaunchKernelGGL(k_zero_words, dim3(64), dim3(256), 0, stream, c->d_wide_hist, (uint64_t)c->max_wide * 2 * kThBins);
    }
    c->result_dirty = true;                           // until this call has completed normally
    c->hist_valid = false;
    ResultBlock* const res_now = c->d_result + c->result_idx;
    ResultBlock* const res_next = c->d_result + (c->result_idx ^ 1);
    c->result_idx ^= 1;
    const unsigned gather_y = (unsigned)std::min<uint64_t>(64, std::max<uint64_t>(1, (max_bound + 1023) / 1024));

    // what sbc_compress_end and the launch helpers need
    sbc_ctx::Pending& P = c->pend;
    P.stream = stream; P.T = T; P.b = b; P.p = p; P.slot = slot; P.slot_is_new = slot_is_new;
    P.force_exact = force_exact; P.use_history = use_history; P.sampled = sampled;
    P.all_inline = all_inline; P.left = false;
    P.in_one = !c->fused_step && n_chunks <= kEmitAllChunks && T <= (int)kEmitAllTensors && p * (double)kChunk <= (double)kFewKept;
    c->emit_name = P.in_one ? "k_emit_all" : !c->fused_step && n_chunks <= kScanAllChunks ? "k_emit_scan" : "k_emit";
    P.sweeps = c->n_wide > 0 && (c->sweep_always || (use_history ? c->hist_long : c->sweep_sampled));
    for (int st = 0; st < kNumStages; ++st) P.timed[st] = false;
    P.res_now = res_now; P.res_next = res_next; P.d_desc = d_desc; P.msg8 = msg8;
    P.msg_capacity = msg_capacity; P.need = need; P.n_chunks = n_chunks; P.gather_y = gather_y; P.scan_tiles = scan_tiles;
    P.wait_on_event = wait_on_event;
    const int lvl = c->profile_level;
    bool* timed = P.timed;

    SBC_HOST_TS(1);
    // ---- [sample ->] accumulate + filter [-> sweeps over long lists] -> thresholds -> apply -> emit -> message ----
    // The sampling kernel is skipped when the previous call left filter keys for the same tensor
    // sizes and sparsity (k_threshold derives them from the ranks it counted).
    if (!use_history) {
        SBC_LAUNCH(kStSample, true, k_sample_thresholds, dim3(T), dim3(kSampleThreads), d_desc, c->d_state,
                   res_now, force_exact, sampled ? p : 0.0);
    }
    const int carry = c->carry_keys && !sampled && !force_exact ? 1 : 0;
    P.carry = carry;
    if (!c->fused_step) {
        const int past = accumulate_past_cache(c, total, p, force_exact != 0, wait_on_event);
        const size_t room = total >= (past == kPastAll ? kPairsFrom : kPairsKeptFrom) ? kStreamRoom : 0;
        if (past == kPastAll) {
            SBC_LAUNCH_LDS(kStAccumulate, true, k_accumulate_filter<kPastAll>, dim3(n_chunks), dim3(kStreamThreads), room, d_desc,
                       c->d_chunk_tensor, c->d_state, c->d_counters, c->cand(), c->d_runs, res_now);
        } else if (past == kPastUpdate) {
            SBC_LAUNCH_LDS(kStAccumulate, true, k_accumulate_filter<kPastUpdate>, dim3(n_chunks), dim3(kStreamThreads), room, d_desc,
                       c->d_chunk_tensor, c->d_state, c->d_counters, c->cand(), c->d_runs, res_now);
        } else {
            SBC_LAUNCH(kStAccumulate, true, k_accumulate_filter<kPastNothing>, dim3(n_chunks), dim3(kStreamThreads), d_desc,
                       c->d_chunk_tensor, c->d_state, c->d_counters, c->cand(), c->d_runs, res_now);
        }
    } else if (total * 12ull > (512ull << 20)) {
        SBC_LAUNCH(kStAccumulate, true, k_client_step<true>, dim3(n_chunks), dim3(kStepThreads), d_desc, c->d_sched,
                   c->d_state, c->cand(), c->d_runs, c->d_stage, c->d_kept, c->d_group, b, carry, res_now);
    } else {
        SBC_LAUNCH(kStAccumulate, true, k_client_step<false>, dim3(n_chunks), dim3(kStepThreads), d_desc, c->d_sched,
                   c->d_state, c->cand(), c->d_runs, c->d_stage, c->d_kept, c->d_group, b, carry, res_now);
    }
    launch_selection_and_encode(c, 0);
    SBC_HOST_TS(2);
    const int rc = enqueue_result_copy(c);
    if (rc != SBC_OK) return rc;
    SBC_HOST_TS(3);
    P.active = true;
    return SBC_OK;
}

int sbc_compress_begin(sbc_ctx* c, void* hip_stream, const float* const* dW, float* const* residual,
                       const int64_t* numel, int n_tensors, double p, void* msg, size_t msg_capacity) {
    return compress_begin(c, hip_stream, dW, residual, numel, n_tensors, p, msg, msg_capacity, true);
}

int sbc_compress_end(sbc_ctx* c, size_t* msg_bytes) {
    if (!c || !msg_bytes || !c->pend.active) return SBC_EINVAL;
    sbc_ctx::Pending& P = c->pend;
    P.active = false;
    DeviceGuard guard(c->device);
    hipStream_t stream = P.stream;
    const int T = P.T;
    TensorDesc* const d_desc = P.d_desc;
    ResultBlock* const res_now = P.res_now;
    int rc = wait_result(c);
    SBC_HOST_TS(4);
    if (rc != SBC_OK) return rc;
    c->cache_valid = true;
    if (P.slot_is_new) c->slot[P.slot].valid = true;
    c->last_T = T;
    c->last_b = P.b;
    c->last_stream = stream;
    for (int st = 0; st < kNumStages; ++st) {
        if (!P.timed[st]) continue;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, c->ev[2 * st], c->ev[2 * st + 1]) == hipSuccess) {
            c->stage_ms[st] += (double)ms;
            c->stage_calls[st] += 1;
        } else {
            (void)hipGetLastError();
        }
    }
    uint32_t err = result_err_of(*c->h_result);
    if (P.in_one && (err & kErrDeferred)) {
        // k_emit_all has left the step because sides were not being selected yet when its word went out.  They are once
        // it has ended, and what they raise (a filter that fell short, a list that overflowed) stands in the error word
        // only: that word again, behind the kernel.
        hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, stream, c->h_result_dev, res_now, ++c->result_seq);
        rc = enqueue_result_copy(c);
        if (rc == SBC_OK) rc = wait_result(c);
        if (rc != SBC_OK) return rc;
        err |= result_err_of(*c->h_result);
    }
    c->last_used_exact_path = false;
    c->last_used_wide = (err & kErrWide) != 0u;

    // ---- second pass: the histogram route for the tensors whose filter kept fewer than k candidates,
    // and the selection for the tensors the streaming kernel left to it ----
    const uint32_t loose = err & (kErrLoose | kErrStaleKeys | kErrLong);
    c->last_deferred = (err & kErrDeferred) != 0u;
    if ((err & (kErrPrefilter | kErrDeferred)) && !(err & (kErrInternal | kErrNonFinite | kErrOverflow))) {
        c->last_used_exact_path = (err & kErrPrefilter) != 0u;
        P.left = P.in_one && (err & kErrDeferred) != 0u;
        hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t*>(res_now),
                           (uint64_t)(sizeof(ResultBlock) / 4));
        if (err & kErrPrefilter) {
            const uint32_t hist_words = (uint32_t)T * kL1Bins;
            hipLaunchKernelGGL(k_zero_words, dim3((hist_words + 2047) / 2048), dim3(256), 0, stream, c->d_hist,
                               (uint64_t)hist_words);
            hipLaunchKernelGGL(k_hist_flagged, dim3(P.n_chunks), dim3(kStreamThreads), 0, stream, d_desc,
                               c->d_chunk_tensor, c->d_state, c->d_hist);
            hipLaunchKernelGGL(k_pick_bins, dim3(T), dim3(256), 0, stream, d_desc, c->d_hist, c->d_state, res_now);
            hipLaunchKernelGGL(k_extract, dim3(P.n_chunks), dim3(kStreamThreads), 0, stream, d_desc,
                               c->d_chunk_tensor, c->d_state, c->cand(), c->d_runs);
        }
        launch_selection_and_encode(c, 1);
        rc = enqueue_result_copy(c);
        if (rc == SBC_OK) rc = wait_result(c);
        if (rc != SBC_OK) return rc;
        err = result_err_of(*c->h_result) | loose;
        if (err & (kErrPrefilter | kErrDeferred)) return SBC_EINTERNAL;
    }
    const int status = status_of_err(err);
    if (status != SBC_OK) return status;
    const uint64_t bytes = result_bytes_of(*c->h_result);
    if (bytes > P.need) return SBC_EINTERNAL;
    *msg_bytes = (size_t)bytes;
    c->last_ok = true;
    c->last_used_history = P.use_history;
    c->last_loose = (err & kErrLoose) != 0u;
    c->result_dirty = false;
    // the next call may start from this call's thresholds unless they proved unhelpful
    // (a sampled call with long lists says nothing about the keys it leaves: those go by rank)
    const bool flood = (err & kErrLoose) && P.use_history;
    c->hist_valid = c->carry_keys && !P.sampled && !P.force_exact && !c->last_used_exact_path && !flood;
    // While the data still grows from call to call (the first rounds of a run, when the residual
    // builds up) carried keys let floods of candidates pass.  After such a call the next calls
    // sample, and each of their samples also tells whether the keys the call before it left would
    // have held on its data (kErrStaleKeys if not): sampling goes on until they would (for at most
    // 64 calls in a row, then a carried call is tried whatever the samples say).  Should carried
    // calls flood again and again all the same, each flood doubles the number of sampled calls
    // that follow it at the least; a carried call that goes well ends that.
    if (flood) {
        c->carry_backoff = std::min(64, std::max(1, 2 * c->carry_backoff));
        c->carry_hold = c->carry_backoff;
        c->carry_stale_run = 0;
    } else if (P.use_history) {
        c->carry_backoff = 0;
    } else if (c->carry_hold > 1) {
        --c->carry_hold;
        c->hist_valid = false;
    } else if (c->carry_hold == 1) {
        if ((err & kErrStaleKeys) && ++c->carry_stale_run <= 64) {
            c->hist_valid = false;
        } else {
            c->carry_hold = 0;
            c->carry_stale_run = 0;
        }
    }
    if (c->hist_valid) {
        c->hist_long = (err & kErrLong) != 0u;
        c->hist_p = P.p;
        c->hist_n.resize(T);
        for (int t = 0; t < T; ++t) c->hist_n[t] = c->plan[t].n;
    }
    return SBC_OK;
}

int sbc_compress(sbc_ctx* c, void* hip_stream, const float* const* dW, float* const* residual,
                 const int64_t* numel, int n_tensors, double p, void* msg, size_t msg_capacity,
                 size_t* msg_bytes) {
    if (!msg_bytes) return SBC_EINVAL;
    const int rc = compress_begin(c, hip_stream, dW, residual, numel, n_tensors, p, msg, msg_capacity, false);
    if (rc != SBC_OK) return rc;
    return sbc_compress_end(c, msg_bytes);
}

int sbc_decompress_accumulate(sbc_ctx* c, void* hip_stream, const void* msg, size_t msg_bytes,
                              const int64_t* numel, int n_tensors, double p, float scale,
                              float* const* out) {
    if (!c || !msg || !numel || !out || n_tensors <= 0 || !valid_p(p)) return SBC_EINVAL;
    if (((uintptr_t)msg & 7u) != 0) return SBC_EINVAL;
    if (n_tensors > c->max_tensors) return SBC_ECAPACITY;
    const int T = n_tensors;
    const int b = bstar_of(p);
    if (b > kMaxB) return SBC_EINVAL;
    SBC_HOST_TS(8);
    if (msg_bytes < 32 + 24ull * (unsigned)T) return SBC_ECORRUPT;
    bool same = c->dev_dec_valid && c->dev_dec_T == T && c->dec_p == p;
    if (same)
        same = std::memcmp(c->dec_numel.data(), numel, sizeof(int64_t) * T) == 0 && std::memcmp(c->dec_out.data(), out, sizeof(float*) * T) == 0;
    if (!same)
        for (int t = 0; t < T; ++t)
            if (numel[t] < 1 || numel[t] >= (int64_t)1 << 32 || !out[t] || ((uintptr_t)out[t] & 3u)) return SBC_EINVAL;
    DeviceGuard guard(c->device);
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    const bool deferred = c->defer_decode != 0;
    if (const int rc = settle_average(c, stream)) return rc;
    if (!same && c->deferred_pending) {
        // the pinned table below may still be read by an upload of an earlier deferred call
        if (hipStreamSynchronize(stream) != hipSuccess) { (void)hipGetLastError(); return SBC_EHIP; }
    }
    if (!same) {
        // Streams of tensors that keep very many entries are decoded tile by tile by many
        // workgroups, as far as the places and the scratch arrays reach; all others by one workgroup each.
        // If there are any, so are the streams of more than one tile, which a single workgroup would take
        // one after another: the launches are there anyway (ResNet-50 shape at p = 0.01: k_decode 14.8
        // us with streams of up to three tiles).  The longest come first, wherever they stand in the list: one
        // workgroup takes a stream's tiles one after another (the 19-tile stream of a 51e6-entry tensor behind
        // 48 two-tile ones at p = 0.001: 149 us a call where it is left without a place, 65 with one; 79
        // ragged tensors of 6e7 entries at p = 0.02 in tensor order 119 us, the longest first 94).
        DecWides& dw = c->dec_wides;
        dw = DecWides{};
        struct Long { uint32_t t, tiles; };
        Long longs[kMaxWideDec];                          // the longest so far, by decreasing length
        int n_longs = 0;
        bool any_wide = false;
        for (int t = 0; t < T && b <= kPackedMaxB; ++t) {
            // (a context that expects messages of the subsampled variant reserves for its cap)
            const int64_t k = cap_of(numel[t], kept_of(numel[t], p), c->sampled != 0);
            const bool wide = (uint64_t)k >= (uint64_t)c->wide_min_kept;
            any_wide = any_wide || wide;
            const uint64_t max_seg = (bound_words_of(numel[t], k, b) + 1) / 2, max_tiles = (max_seg + kDecThreads - 1) / kDecThreads;
            if (!(wide || max_tiles > 1) || max_tiles == 0 || max_tiles >= (1ull << 29)) continue;
            int at = n_longs;
            while (at > 0 && longs[at - 1].tiles < max_tiles) --at;
            if (at == kMaxWideDec) continue;
            n_longs = std::min(n_longs + 1, kMaxWideDec);
            std::copy_backward(longs + at, longs + n_longs - 1, longs + n_longs);
            longs[at] = {(uint32_t)t, (uint32_t)max_tiles};
        }
        if (!any_wide) n_longs = 0;
        std::sort(longs, longs + n_longs, [](const Long& x, const Long& y) { return x.t < y.t; });
        uint64_t segs = 0, tiles = 0;
        for (int i = 0; i < n_longs; ++i) {
            const Long& l = longs[i];
            if (segs + (uint64_t)l.tiles * kDecThreads > c->dec_seg_cap || tiles + l.tiles > c->dec_tile_cap) continue;
            DecWide& w = dw.w[dw.count++];
            w.out = out[l.t]; w.n = (uint32_t)numel[l.t]; w.t = l.t;
            w.tile0 = (uint32_t)tiles; w.max_tiles = l.tiles; w.seg0 = segs;
            segs += (uint64_t)l.tiles * kDecThreads; tiles += l.tiles;
        }
        uint32_t n_blocks = 0, extra = 0;
        for (int t = 0, i = 0; t < T; ++t) {
            if (i < dw.count && dw.w[i].t == (uint32_t)t) { ++i; continue; }
            // One workgroup decodes a stream; the scattered updates of a stream with many codes are
            // shared among several workgroups that each decode it (a compute unit sustains only so
            // many scattered accesses at a time, and decoding again costs no more time than once).
            uint32_t shares = decode_shares(cap_of(numel[t], kept_of(numel[t], p), c->sampled != 0));
            if (extra + shares - 1u > kMaxDecExtra) shares = 1u;
            extra += shares - 1u;
            for (uint32_t sh = 0; sh < shares; ++sh) {
                DecBlock& blk = c->h_dec_blocks[n_blocks++];
                blk.out = out[t]; blk.n = (uint32_t)numel[t]; blk.t = (uint32_t)t; blk.share = sh; blk.shares = shares;
            }
        }
        c->dec_tiles = (uint32_t)tiles; c->dec_p = p;
        c->n_dec_blocks = n_blocks;
        c->dev_dec_valid = false;
        if (n_blocks > 0 && hipMemcpyAsync(c->d_dec_blocks, c->h_dec_blocks, sizeof(DecBlock) * n_blocks, hipMemcpyHostToDevice, stream) != hipSuccess) {
            (void)hipGetLastError();
            return SBC_EHIP;
        }
        c->dec_out.assign(out, out + T);
        c->dec_numel.assign(numel, numel + T);
        c->dev_dec_T = T;
    }
    // the decode kernel leaves the other of its two result blocks clean for the next call; calls
    // whose status is deferred all raise their error bits in block [4] and clear the spare
    ResultBlock* res_dec;
    ResultBlock* res_dec_next;
    if (deferred) {
        if (c->deferred_dirty) {
            hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t*>(c->d_result + 4),
                               (uint64_t)(sizeof(ResultBlock) / 4));
            c->deferred_dirty = false;
        }
        res_dec = c->d_result + 4;
        res_dec_next = c->d_result + 5;
    } else {
        if (c->dec_result_dirty) {                    // after an error, or on the first call
            hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t*>(c->d_result + 2),
                               (uint64_t)(2 * sizeof(ResultBlock) / 4));
        }
        c->dec_result_dirty = true;                   // until this call has completed normally
        res_dec = c->d_result + 2 + c->dec_result_idx;
        res_dec_next = c->d_result + 2 + (c->dec_result_idx ^ 1);
        c->dec_result_idx ^= 1;
    }
    SBC_HOST_TS(9);
    const uint8_t* m8 = static_cast<const uint8_t*>(msg);
    const unsigned long long mb = (unsigned long long)msg_bytes;
    MemBlocks blocks;
    blocks.table = c->d_dec_blocks; blocks.result = res_dec; blocks.next_result = res_dec_next;
    launch_decode(stream, c->n_dec_blocks, c->dec_tiles, m8, mb, blocks, T, b, scale, c->dec_wides, c->d_tile_fn);
    if (c->dec_tiles > 0) {
        const dim3 tiles(c->dec_tiles), block(kDecThreads);
        if (b <= 7) hipLaunchKernelGGL(k_dec_tile_sums<2>, tiles, block, 0, stream, m8, mb, c->dec_wides, T, b, c->d_tile_fn, c->d_seg_pack, c->d_tile_sum, res_dec);
        else if (b <= 11) hipLaunchKernelGGL(k_dec_tile_sums<3>, tiles, block, 0, stream, m8, mb, c->dec_wides, T, b, c->d_tile_fn, c->d_seg_pack, c->d_tile_sum, res_dec);
        else hipLaunchKernelGGL(k_dec_tile_sums<4>, tiles, block, 0, stream, m8, mb, c->dec_wides, T, b, c->d_tile_fn, c->d_seg_pack, c->d_tile_sum, res_dec);
        hipLaunchKernelGGL(k_dec_tile_place, dim3(c->dec_tiles * kPlacePer), dim3(kPlaceThreads), 0, stream, m8, mb, c->dec_wides, T, b, scale,
                           c->d_seg_pack, c->d_tile_sum, res_dec);
    }
    SBC_HOST_TS(10);
    if (hipGetLastError() != hipSuccess) return SBC_EHIP;
    if (deferred) {
        // (the uploads above precede every later kernel on this stream)
        c->deferred_pending = true;
        c->dev_dec_valid = true;
        return SBC_OK;
    }
    // the status goes to pinned host memory by a small dispatch, and the call looks for it there (as
    // the client step does): it returns when the status is known; `out` is complete for everything
    // enqueued on the stream afterwards
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, stream, c->h_result_dec_dev, res_dec, ++c->dec_seq);
    if (hipGetLastError() != hipSuccess) return SBC_EHIP;
    if (const int rc = wait_result(c->h_result_dec, c->dec_seq, true, stream)) return rc;
    SBC_HOST_TS(11);
    c->dev_dec_valid = true;
    const uint32_t err = result_err_of(*c->h_result_dec);
    if (err == 0u) c->dec_result_dirty = false;
    return status_of_err(err);
}

// out <- the sum of the messages, one after another: the general way of sbc_decompress_average.
static int average_in_turn(sbc_ctx* c, hipStream_t stream, const void* const* msgs, const size_t* msg_bytes, int n_msgs,
                           const int64_t* numel, int T, double p, float scale, float* const* out) {
    if (c->avg_clears) {
        hipLaunchKernelGGL(k_average_clear, dim3(c->avg_chunks), dim3(256), 0, stream, c->d_avg_chunk, c->d_avg_tensor,
                           c->deferred_dirty && !c->deferred_pending ? c->d_result + 4 : nullptr);
        if (!c->deferred_pending) c->deferred_dirty = false;
    } else {
        for (int t = 0; t < T; ++t)
            hipLaunchKernelGGL(k_zero_words, dim3((unsigned)std::min<uint64_t>(4096, ((uint64_t)numel[t] + 2047) / 2048)), dim3(256), 0,
                               stream, reinterpret_cast<uint32_t*>(out[t]), (uint64_t)numel[t]);
    }
    // one status check at the end, unless the caller still has the status of deferred calls to ask for
    const int before = c->defer_decode;
    c->defer_decode = c->deferred_pending ? 0 : 1;
    int rc = SBC_OK;
    for (int m = 0; m < n_msgs && rc == SBC_OK; ++m)
        rc = sbc_decompress_accumulate(c, stream, msgs[m], msg_bytes[m], numel, T, p, scale, out);
    const int status = c->defer_decode ? sbc_decode_status(c, stream) : SBC_OK;
    c->defer_decode = before;
    return rc != SBC_OK ? rc : status;
}

int sbc_decompress_average(sbc_ctx* c, void* hip_stream, const void* const* msgs, const size_t* msg_bytes, int n_msgs,
                           const int64_t* numel, int n_tensors, double p, float scale, float* const* out) {
    if (!c || !msgs || !msg_bytes || n_msgs <= 0 || !numel || !out || n_tensors <= 0 || !valid_p(p)) return SBC_EINVAL;
    for (int m = 0; m < n_msgs; ++m)
        if (!msgs[m] || ((uintptr_t)msgs[m] & 7u) != 0) return SBC_EINVAL;
    if (n_tensors > c->max_tensors) return SBC_ECAPACITY;
    const int T = n_tensors;
    const int b = bstar_of(p);
    if (b > kMaxB) return SBC_EINVAL;
    for (int m = 0; m < n_msgs; ++m)
        if (msg_bytes[m] < 32 + 24ull * (unsigned)T) return SBC_ECORRUPT;
    const bool same = c->avg_valid && c->avg_p == p && c->avg_numel.size() == (size_t)T &&
                      std::memcmp(c->avg_numel.data(), numel, sizeof(int64_t) * T) == 0 &&
                      std::memcmp(c->avg_out.data(), out, sizeof(float*) * T) == 0;
    DeviceGuard guard(c->device);
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    if (!same)
        for (int t = 0; t < T; ++t)
            if (numel[t] < 1 || numel[t] >= (int64_t)1 << 32 || !out[t] || ((uintptr_t)out[t] & 3u)) return SBC_EINVAL;
    if (const int rc = settle_average(c, stream)) return rc;
    if (!same) {
        // (every earlier call has waited for its uploads from the pinned tables)
        c->avg_valid = false;
        uint64_t pos = 0, marks = 0, chunks = 0;
        for (int t = 0; t < T; ++t) chunks += ((uint64_t)numel[t] + kChunk - 1) / kChunk;
        c->avg_clears = chunks <= c->max_chunks && chunks < (1ull << 31);
        c->avg_fits = c->avg_clears && b >= kAvgMinB && b <= kPackedMaxB;
        c->avg_chunks = (uint32_t)chunks;
        uint32_t* const ids = reinterpret_cast<uint32_t*>(c->h_avg_tensor + T);
        uint32_t n_ids = 0, chunk0 = 0, n_small = 0, extra = 0;
        const auto most_segs = [&](int t) { return (bound_words_of(numel[t], cap_of(numel[t], kept_of(numel[t], p), true), b) + 1) / 2; };
        for (int t = 0; t < T && c->avg_clears; ++t) {
            // (room for the cap of the subsampled variant, whichever of the two the senders use)
            const int64_t n = numel[t], k = cap_of(n, kept_of(n, p), true);
            const uint64_t segs = most_segs(t);
            AvgTensor& a = c->h_avg_tensor[t];
            a.out = out[t]; a.n = (uint32_t)n; a.kcap = (uint32_t)k; a.pos_off = (uint32_t)pos; a.mark_off = (uint32_t)marks;
            const uint32_t nchunks = (uint32_t)(((uint64_t)n + kChunk - 1) / kChunk);
            for (uint32_t j = 0; j < nchunks; ++j) c->h_avg_chunk[chunk0 + j] = make_uint2((uint32_t)t, chunk0);
            chunk0 += nchunks;
            pos += (uint64_t)k;
            marks += ((uint64_t)n + kAvgBlock - 1) / kAvgBlock + 1;
            c->avg_fits = c->avg_fits && segs <= (uint64_t)kAvgMaxTiles * kDecThreads && pos < (1ull << 31) && marks < (1ull << 31);
            if (!c->avg_fits || segs <= kAvgWaveSegs) continue;
            const uint32_t tiles = (uint32_t)((segs + kDecThreads - 1) / kDecThreads);
            const uint32_t shares = extra + tiles - 1u <= kMaxDecExtra ? tiles : 1u;
            extra += shares - 1u;
            for (uint32_t share = 0; share < shares; ++share) {
                uint32_t* const w = ids + (size_t)kDecWaves * n_ids++;
                std::fill_n(w, (size_t)kDecWaves, kAvgNone);
                w[0] = (uint32_t)t; w[1] = kAvgWhole; w[2] = share; w[3] = shares;
            }
        }
        for (int t = 0; t < T && c->avg_fits; ++t) {
            if (most_segs(t) > kAvgWaveSegs) continue;
            if (n_small % kDecWaves == 0) { std::fill_n(ids + (size_t)kDecWaves * n_ids, (size_t)kDecWaves, kAvgNone); ++n_ids; }
            ids[(size_t)kDecWaves * (n_ids - 1) + n_small++ % kDecWaves] = (uint32_t)t;
        }
        if (c->avg_clears &&
            (hipMemcpyAsync(c->d_avg_tensor, c->h_avg_tensor, sizeof(AvgTensor) * T + sizeof(uint32_t) * kDecWaves * n_ids,
                            hipMemcpyHostToDevice, stream) != hipSuccess ||
             hipMemcpyAsync(c->d_avg_chunk, c->h_avg_chunk, sizeof(uint2) * chunks, hipMemcpyHostToDevice, stream) != hipSuccess)) {
            (void)hipGetLastError();
            return SBC_EHIP;
        }
        c->avg_blocks = n_ids; c->avg_pos = (uint32_t)pos; c->avg_marks = marks; c->avg_p = p;
        c->avg_out.assign(out, out + T);
        c->avg_numel.assign(numel, numel + T);
        c->avg_valid = true;
    }
    // Messages per pass: a lane each, what the scratch memory holds, and what one launch can have (2^32 - 1 work
    // items: from a million streams of one wavefront each on, fewer than 64).  A single message for a large model
    // is added to the cleared result instead: that stores no positions first (ResNet-50 shape at p = 0.001
    // 35 us, 41 the other way; 66e6 entries 68 and 79 us).  Two messages take 45 us in turn and 42 together, at
    // 66e6 entries 93 and 80 us; one message of a small model 30 and 25 us, of 2^20 entries at p = 0.01 39 and
    // 32 us.
    const uint64_t per_msg = (uint64_t)c->avg_pos + c->avg_marks + (uint64_t)T;
    const uint64_t room = 2u * c->cand_entries;
    const uint64_t launchable = 0xFFFFFFFFull / ((uint64_t)kDecThreads * std::max<uint32_t>(c->avg_blocks, 1u));
    const int most = c->avg_fits && !c->pend.active ? (int)std::min<uint64_t>({kAvgMaxMsgs, room / per_msg, launchable}) : 0;
    if (most < 1 || (n_msgs == 1 && c->avg_chunks > kAvgAloneChunks)) return average_in_turn(c, stream, msgs, msg_bytes, n_msgs, numel, T, p, scale, out);
    // (the last client step may still be draining on another stream)
    if (c->last_T > 0 && c->last_stream != stream && hipStreamSynchronize(c->last_stream) != hipSuccess) {
        (void)hipGetLastError();
        return SBC_EHIP;
    }
    if (c->dec_result_dirty)                              // after an error, or on the first call
        hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, stream, reinterpret_cast<uint32_t*>(c->d_result + 2),
                           (uint64_t)(2 * sizeof(ResultBlock) / 4));
    c->dec_result_dirty = true;                           // until this call has completed normally
    ResultBlock* const res = c->d_result + 2 + c->dec_result_idx;
    ResultBlock* const res_next = c->d_result + 2 + (c->dec_result_idx ^ 1);
    c->dec_result_idx ^= 1;
    uint32_t* const positions = c->d_cand;
    const uint32_t* const ids = reinterpret_cast<const uint32_t*>(c->d_avg_tensor + T);
    for (int m0 = 0; m0 < n_msgs; m0 += most) {
        const int M = std::min(most, n_msgs - m0);
        AvgMsgs list = {};
        for (int m = 0; m < M; ++m) { list.msg[m] = static_cast<const uint8_t*>(msgs[m0 + m]); list.bytes[m] = msg_bytes[m0 + m]; }
        uint32_t* const marks = positions + (size_t)M * c->avg_pos;
        float* const addends = reinterpret_cast<float*>(marks + (size_t)M * c->avg_marks);
        const dim3 grid((unsigned)M * c->avg_blocks), block(kDecThreads);
        if (b <= 7) hipLaunchKernelGGL(k_average_decode<2>, grid, block, 0, stream, list, (uint32_t)M, ids, c->d_avg_tensor, T, b, scale, c->avg_pos, positions, marks, addends, res, res_next);
        else if (b <= 11) hipLaunchKernelGGL(k_average_decode<3>, grid, block, 0, stream, list, (uint32_t)M, ids, c->d_avg_tensor, T, b, scale, c->avg_pos, positions, marks, addends, res, res_next);
        else hipLaunchKernelGGL(k_average_decode<4>, grid, block, 0, stream, list, (uint32_t)M, ids, c->d_avg_tensor, T, b, scale, c->avg_pos, positions, marks, addends, res, res_next);
        // The status is what the decoding kernels find: it goes out between the last of them and the kernel that adds
        // the positions up and stores the result, so that the caller gets on with what it enqueues next while that one
        // runs (32 messages of the ResNet-50 shape, a call among others: 59.0 us with the status behind it, 47.0 so; the
        // event as the launch's own takes nothing, recorded behind the launch 1.3).
        if (m0 + M == n_msgs)
            hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, stream, c->h_result_dec_dev, res, ++c->dec_seq);
        constexpr uint32_t kHalf = kAvgBlock / 2u;
        const auto apply = M < kAvgWholeFrom ? (m0 == 0 ? k_average_apply<false, kHalf> : k_average_apply<true, kHalf>)
                                             : (m0 == 0 ? k_average_apply<false, kAvgBlock> : k_average_apply<true, kAvgBlock>);
        hipExtLaunchKernelGGL(apply, dim3(c->avg_chunks), dim3(kEncThreads), 0, stream, nullptr, m0 + M == n_msgs ? c->ev_average : nullptr, 0,
                              c->d_avg_chunk, c->d_avg_tensor, (uint32_t)M, c->avg_pos, positions, marks, addends, res);
    }
    if (hipGetLastError() != hipSuccess) {
        (void)hipStreamSynchronize(stream);               // (of what was launched nobody else knows)
        (void)hipGetLastError();
        return SBC_EHIP;
    }
    c->avg_running = true;
    if (const int rc = wait_result(c->h_result_dec, c->dec_seq, true, stream)) return rc;
    const uint32_t err = result_err_of(*c->h_result_dec);
    if (err == 0u) {
        c->dec_result_dirty = false;
    } else {                                              // (the last kernel looks at that word: nobody clears it before)
        c->avg_running = false;
        if (hipStreamSynchronize(stream) != hipSuccess) {
            (void)hipGetLastError();
            return SBC_EHIP;
        }
    }
    if ((err & kErrDeferred) && !(err & kErrCorrupt))     // a stream of more positions than there is room for
        return average_in_turn(c, stream, msgs, msg_bytes, n_msgs, numel, T, p, scale, out);
    return status_of_err(err & ~kErrDeferred);
}

int sbc_decode_status(sbc_ctx* c, void* hip_stream) {
    if (!c) return SBC_EINVAL;
    if (!c->deferred_pending) return SBC_OK;
    DeviceGuard guard(c->device);
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    c->deferred_pending = false;
    c->deferred_dirty = true;
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, stream, c->h_result_dec_dev, c->d_result + 4, ++c->dec_seq);
    if (hipGetLastError() != hipSuccess) return SBC_EHIP;
    if (const int rc = wait_result(c->h_result_dec, c->dec_seq, true, stream)) return rc;
    return status_of_err(result_err_of(*c->h_result_dec));
}

int sbc_copy_baseline(void* hip_stream, void* dst, const void* src, size_t bytes) {
    if (!dst || !src || bytes == 0 || (bytes & 15u) || (((uintptr_t)dst | (uintptr_t)src) & 15u)) return SBC_EINVAL;
    const uint64_t n16 = bytes / 16;
    const uint64_t per_block = 256ull * 8ull;
    const uint64_t blocks = (n16 + per_block - 1) / per_block;
    if (blocks >= (1ull << 31)) return SBC_EINVAL;
    hipLaunchKernelGGL(k_copy_baseline, dim3((unsigned)blocks), dim3(256), 0, reinterpret_cast<hipStream_t>(hip_stream),
                       static_cast<uint4*>(dst), static_cast<const uint4*>(src), n16);
    return hipGetLastError() == hipSuccess ? SBC_OK : SBC_EHIP;
}

int sbc_profile_enable(sbc_ctx* c, int level) {
    if (!c || level < 0 || level > 2) return SBC_EINVAL;
    c->profile_level = level;
    for (int st = 0; st < kNumStages; ++st) { c->stage_ms[st] = 0.0; c->stage_calls[st] = 0; }
    return SBC_OK;
}

int sbc_profile_level(sbc_ctx* c, int level) {
    if (!c || level < 0 || level > 2) return SBC_EINVAL;
    c->profile_level = level;
    return SBC_OK;
}

int sbc_profile_read(sbc_ctx* c, int stage, const char** name, double* total_ms, int64_t* calls) {
    if (!c || stage < 0 || stage >= kNumStages) return SBC_EINVAL;
    // (the streaming pass is one of two kernels, by SBC_OPT_FUSED_STEP)
    if (name) *name = (stage == kStAccumulate && !c->fused_step) ? "k_accumulate_filter" : stage == kStEmit ? c->emit_name : kStageNames[stage];
    if (total_ms) *total_ms = c->stage_ms[stage];
    if (calls) *calls = c->stage_calls[stage];
    return SBC_OK;
}

int sbc_last_tensor_stats(sbc_ctx* c, int tensor, double* mu_pos, double* mu_neg, int* side,
                          int64_t* nnz, int64_t* bit_len) {
    if (!c || !c->last_ok || tensor < 0 || tensor >= c->last_T) return SBC_EINVAL;
    DeviceGuard guard(c->device);
    if (hipStreamSynchronize(c->last_stream) != hipSuccess ||
        hipMemcpy(c->h_state, c->d_state + tensor, sizeof(TensorState), hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return SBC_EHIP;
    }
    const TensorState& s = c->h_state[0];
    if (s.kc[0] == 0u || s.kc[1] == 0u) return SBC_EINTERNAL;
    if (mu_pos) *mu_pos = s.S[0] / (double)s.kc[0];
    if (mu_neg) *mu_neg = s.S[1] / (double)s.kc[1];
    if (side) *side = s.side;
    if (nnz) *nnz = (int64_t)s.nnz;
    if (bit_len) *bit_len = (int64_t)s.bit_len;
    return SBC_OK;
}

int sbc_last_candidates(sbc_ctx* c, int tensor, int64_t* positive, int64_t* negative) {
    if (!c || !c->last_ok || tensor < 0 || tensor >= c->last_T) return SBC_EINVAL;
    DeviceGuard guard(c->device);
    if (hipStreamSynchronize(c->last_stream) != hipSuccess ||
        hipMemcpy(c->h_state, c->d_state + tensor, sizeof(TensorState), hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return SBC_EHIP;
    }
    if (positive) *positive = (int64_t)c->h_state[0].cand_seen[0];
    if (negative) *negative = (int64_t)c->h_state[0].cand_seen[1];
    return SBC_OK;
}

int sbc_last_mask(sbc_ctx* c, int tensor, uint32_t* mask_words, size_t n_words) {
    if (!c || !c->last_ok || !mask_words || tensor < 0 || tensor >= c->last_T) return SBC_EINVAL;
    const TensorDesc& d = c->plan[tensor];
    if (n_words != ((size_t)d.n + 31) / 32) return SBC_EINVAL;
    DeviceGuard guard(c->device);
    if (hipStreamSynchronize(c->last_stream) != hipSuccess) { (void)hipGetLastError(); return SBC_EHIP; }
    if (hipMemcpy(c->h_state, c->d_state + tensor, sizeof(TensorState), hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return SBC_EHIP;
    }
    if (c->h_state[0].sorted_kept) {
        // the streaming kernel left the sorted kept indices in scratch
        const uint32_t nnz = c->h_state[0].nnz;
        if (nnz > d.kcap) return SBC_EINTERNAL;
        std::vector<uint32_t> idx(nnz);
        if (hipMemcpy(idx.data(), c->d_kept + d.kept_off, (size_t)nnz * 4, hipMemcpyDeviceToHost) != hipSuccess) {
            (void)hipGetLastError();
            return SBC_EHIP;
        }
        std::memset(mask_words, 0, n_words * 4);
        for (uint32_t j : idx) {
            if (j >= d.n) return SBC_EINTERNAL;
            mask_words[j >> 5] |= 1u << (j & 31u);
        }
        return SBC_OK;
    }
    // from the chunks' codes, which stay where they are until the next step
    std::memset(mask_words, 0, n_words * 4);
    constexpr uint32_t kBatch = 1024;
    struct Batch { ChunkSummary sum[kBatch]; uint32_t words[kBatch * kChunkWords]; };
    std::unique_ptr<Batch> host(new (std::nothrow) Batch);
    if (!host) return SBC_EHIP;
    const int b = c->last_b;
    for (uint32_t f0 = 0; f0 < d.nchunks; f0 += kBatch) {
        const uint32_t count = std::min(kBatch, d.nchunks - f0);
        const size_t at = (size_t)d.chunk0 + f0;
        if (hipMemcpy(host->sum, c->d_sum + at, count * sizeof(ChunkSummary), hipMemcpyDeviceToHost) != hipSuccess ||
            hipMemcpy(host->words, c->d_bitmap + at * kChunkWords, (size_t)count * kChunkWords * 4, hipMemcpyDeviceToHost) != hipSuccess) {
            (void)hipGetLastError();
            return SBC_EHIP;
        }
        for (uint32_t f = 0; f < count; ++f) {
            const ChunkSummary& sm = host->sum[f];
            if (!sum_any(sm)) continue;
            const uint32_t* const w = host->words + (size_t)f * kChunkWords;
            const uint64_t e0 = (uint64_t)(f0 + f) * kChunk;
            if (sum_raw(sm)) {
                const size_t to = (size_t)(f0 + f) * kChunkWords;
                std::memcpy(mask_words + to, w, std::min<size_t>(kChunkWords, n_words - to) * 4);
                continue;
            }
            const auto bit = [&](uint32_t i) { return (w[i >> 5] >> (31u - (i & 31u))) & 1u; };
            uint64_t pos = sum_first(sm);
            for (uint32_t i = 0, end = sum_inner(sm); ; ) {
                if (pos >= (uint64_t)kChunk || e0 + pos >= d.n) return SBC_EINTERNAL;
                mask_words[(e0 + pos) >> 5] |= 1u << (pos & 31u);
                if (i >= end) break;
                uint64_t gap = 0;
                while (i < end && bit(i++)) ++gap;
                for (int j = 0; j < b; ++j) gap = (gap << 1) | (i < end ? bit(i++) : 0u);
                pos += 1 + gap;
            }
        }
    }
    return SBC_OK;
}

int sbc_decompress_accumulate_noalloc(int device, void* hip_stream, const void* msg, size_t msg_bytes,
                                      const int64_t* numel, int n_tensors, double p, float scale,
                                      float* const* out, int32_t* status) {
    if (!msg || !numel || !out || !status || n_tensors <= 0 || !valid_p(p) || device < 0) return SBC_EINVAL;
    if ((((uintptr_t)msg) & 7u) != 0 || (((uintptr_t)status) & 3u) != 0) return SBC_EINVAL;
    if (n_tensors > SBC_NOALLOC_MAX_TENSORS || device >= kNoAllocMaxDevices) return SBC_ECAPACITY;
    int n_dev = 0;
    if (hipGetDeviceCount(&n_dev) != hipSuccess) { (void)hipGetLastError(); return SBC_EHIP; }
    if (device >= n_dev) return SBC_EINVAL;
    const int T = n_tensors;
    const int b = bstar_of(p);
    if (b > kMaxB) return SBC_EINVAL;
    if (msg_bytes < 32 + 24ull * (unsigned)T) return SBC_ECORRUPT;
    ArgBlocks a;
    std::memset(static_cast<void*>(&a), 0, sizeof(a));
    uint32_t n_blocks = 0, extra = 0;
    for (int t = 0; t < T; ++t) {
        if (numel[t] < 1 || numel[t] >= (int64_t)1 << 32 || !out[t] || ((uintptr_t)out[t] & 3u)) return SBC_EINVAL;
        uint32_t shares = decode_shares(kept_of(numel[t], p));
        if (extra + shares - 1u > kMaxDecExtra) shares = 1u;
        extra += shares - 1u;
        a.out[t] = out[t]; a.n[t] = (uint32_t)numel[t];
        for (uint32_t sh = 0; sh < shares; ++sh) a.block[n_blocks++] = (uint16_t)((uint32_t)t | (sh << 8) | ((shares - 1u) << 11));
    }
    a.status = status;
    DeviceGuard guard(device);
    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    hipLaunchKernelGGL(k_status_ok, dim3(1), dim3(64), 0, stream, status);
    launch_decode(stream, n_blocks, 0u, static_cast<const uint8_t*>(msg), (unsigned long long)msg_bytes, a, T, b, scale, NoWides{}, nullptr);
    if (hipGetLastError() != hipSuccess) return SBC_EHIP;
    return SBC_OK;
}

#ifdef SBC_PHASE_TIMING
int sbc_debug_host_times(double* out) { for (int i = 0; i < 16; ++i) out[i] = g_host_ts[i]; return 0; }
// tuning builds only: copies the phase clock tables (3 x 1024 x 16 u64) to host memory
int sbc_debug_phase_clocks(unsigned long long* out) {
    return hipMemcpyFromSymbol(out, HIP_SYMBOL(sbc::g_phase_clock), sizeof(unsigned long long) * 3 * 1024 * 16) == hipSuccess ? 0 : -3;
}
int sbc_debug_step_clocks(unsigned long long* out) {
    return hipMemcpyFromSymbol(out, HIP_SYMBOL(sbc::g_step_clock), sizeof(unsigned long long) * 16384 * 8) == hipSuccess ? 0 : -3;
}
#endif

int sbc_last_route(sbc_ctx* c) {
    if (!c || !c->last_ok) return SBC_EINVAL;
    return (c->last_used_history ? SBC_ROUTE_CARRIED_KEYS : 0) | (c->last_used_exact_path ? SBC_ROUTE_HISTOGRAM : 0) |
           (c->last_used_wide ? SBC_ROUTE_WIDE : 0) | (c->last_loose ? SBC_ROUTE_LOOSE_KEYS : 0) |
           (c->last_deferred ? SBC_ROUTE_TAKEN_OVER : 0);
}

}  // extern "C"
