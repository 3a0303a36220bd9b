// Drives the library's host side (argument validation, planning of a client step, message
// bounds, sizing of the decode plan and of the server average's tables, the clean-up paths) in a build where the HIP runtime is
// replaced by hip_stub.cpp and everything is compiled with AddressSanitizer and
// UndefinedBehaviorSanitizer.  No GPU.  Usage: driver <file with one model's tensor sizes>.
// Pointers that stand for device buffers are never dereferenced here (launches do nothing), so
// large tensors are made-up, suitably aligned addresses.
#include "sbc.h"

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <ctime>
#include <vector>

#include <unistd.h>

extern "C" long stub_launches();
extern "C" unsigned stub_grid(long launch);
extern "C" const void* stub_kernel(long launch);
extern "C" long stub_live_blocks();
extern "C" void stub_fail_allocation(long nth);
extern "C" void stub_withhold_results(int on);
extern "C" int stub_known_senders();
extern "C" void stub_result_bits(uint32_t bits);
extern "C" void stub_next_result_bits(const char* kernel, uint32_t bits);
extern "C" void stub_stream_gone(void* stream);
extern "C" void stub_stream_records(void* stream);
extern "C" void stub_events_pending(int on);
extern "C" int stub_stream_waits();
extern "C" int stub_event_waits();
extern "C" int stub_launched(const char* name, long from);
extern "C" unsigned stub_grid_of(const char* name, long from);
extern "C" size_t stub_lds_of(const char* name, long from);

#define CHECK(cond)                                                                     \
    do {                                                                                \
        if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); std::exit(1); } \
    } while (0)

struct Buffers {
    std::vector<const float*> dW;
    std::vector<float*> R, out;
    std::vector<int64_t> numel;
    int T() const { return (int)numel.size(); }
    int64_t total() const { int64_t s = 0; for (int64_t n : numel) s += n; return s; }
};

// made-up addresses: three disjoint ranges, each tensor 16-byte aligned
static Buffers fake_buffers(const std::vector<int64_t>& sizes, uintptr_t salt = 0) {
    Buffers b;
    uintptr_t a = 0x100000000000ull + salt, r = 0x200000000000ull + salt, o = 0x300000000000ull + salt;
    for (int64_t n : sizes) {
        b.numel.push_back(n);
        b.dW.push_back(reinterpret_cast<const float*>(a));
        b.R.push_back(reinterpret_cast<float*>(r));
        b.out.push_back(reinterpret_cast<float*>(o));
        const uintptr_t step = ((uintptr_t)n * 4u + 15u) & ~(uintptr_t)15u;
        a += step; r += step; o += step;
    }
    return b;
}

static void* const kMsg = reinterpret_cast<void*>(0x400000000000ull);

static int compress(sbc_ctx* c, const Buffers& b, double p, size_t capacity, size_t* nbytes) {
    return sbc_compress(c, nullptr, b.dW.data(), b.R.data(), b.numel.data(), b.T(), p, kMsg, capacity, nbytes);
}

int main(int argc, char** argv) {
    CHECK(argc == 2);
    std::vector<int64_t> model;
    {
        std::FILE* f = std::fopen(argv[1], "r");
        CHECK(f != nullptr);
        long long n;
        while (std::fscanf(f, "%lld", &n) == 1) model.push_back(n);
        std::fclose(f);
    }
    CHECK(model.size() >= 100);
    CHECK(stub_known_senders() == 7);                  // k_emit_all and k_emit_scan for few and for many chunks, k_emit, k_finish_message, k_publish

    // ---- scalar helpers ----
    const double bad_p[] = {0.0, 1.0, -1.0, 2.0, 0.0 / 1.0 - 0.0, 1e-12};
    for (double p : bad_p) {
        const int64_t n1[1] = {10};
        if (p != 1e-12) { CHECK(sbc_golomb_bstar(p) == SBC_EINVAL); CHECK(sbc_num_kept(10, p) == SBC_EINVAL); }
        CHECK(sbc_msg_bound(n1, 1, p) == 0);
        CHECK(sbc_msg_bound_sampled(n1, 1, p) == 0);
    }
    CHECK(sbc_golomb_bstar(0.001) == 9 && sbc_golomb_bstar(0.5) == 0);
    CHECK(sbc_num_kept(0, 0.1) == SBC_EINVAL && sbc_num_kept(64, 0.001) == 1);
    {
        const int64_t zero[1] = {0}, huge[1] = {(int64_t)1 << 32}, neg[1] = {-5};
        CHECK(sbc_msg_bound(zero, 1, 0.1) == 0 && sbc_msg_bound(huge, 1, 0.1) == 0 && sbc_msg_bound(neg, 1, 0.1) == 0);
        CHECK(sbc_msg_bound(nullptr, 1, 0.1) == 0 && sbc_msg_bound(zero, 0, 0.1) == 0);
    }
    for (int code = 1; code >= -8; --code) CHECK(sbc_strerror(code) != nullptr);

    // ---- create: bad arguments, and an allocation that fails half way (everything is released) ----
    sbc_ctx* c = nullptr;
    CHECK(sbc_create(nullptr, 0, 10, 1) == SBC_EINVAL);
    CHECK(sbc_create(&c, 0, 0, 1) == SBC_EINVAL && sbc_create(&c, 0, 10, 0) == SBC_EINVAL);
    CHECK(sbc_create(&c, 1, 10, 1) == SBC_EINVAL && sbc_create(&c, -1, 10, 1) == SBC_EINVAL);
    for (long nth = 0; nth < 60; nth += 7) {
        stub_fail_allocation(nth);
        const int rc = sbc_create(&c, 0, 100000, 4);
        stub_fail_allocation(-1);
        if (rc == SBC_OK) { sbc_destroy(c); c = nullptr; }
        else CHECK(rc == SBC_EHIP && c == nullptr);
        CHECK(stub_live_blocks() == 0);
    }
    sbc_destroy(nullptr);

    // ---- the model: plans of the client step in every mode ----
    const Buffers m = fake_buffers(model);
    const double p = 0.001;
    const size_t bound = sbc_msg_bound(m.numel.data(), m.T(), p);
    CHECK(bound > 32 + 24 * (size_t)m.T());
    CHECK(sbc_msg_bound_sampled(m.numel.data(), m.T(), p) >= bound);
    CHECK(sbc_create(&c, 0, m.total(), m.T()) == SBC_OK);
    size_t nbytes = 123;
    // argument errors: nothing is enqueued
    const long launches0 = stub_launches();
    CHECK(sbc_compress(nullptr, nullptr, m.dW.data(), m.R.data(), m.numel.data(), m.T(), p, kMsg, bound, &nbytes) == SBC_EINVAL);
    CHECK(sbc_compress(c, nullptr, nullptr, m.R.data(), m.numel.data(), m.T(), p, kMsg, bound, &nbytes) == SBC_EINVAL);
    CHECK(sbc_compress(c, nullptr, m.dW.data(), m.R.data(), m.numel.data(), 0, p, kMsg, bound, &nbytes) == SBC_EINVAL);
    CHECK(sbc_compress(c, nullptr, m.dW.data(), m.R.data(), m.numel.data(), m.T(), 0.0, kMsg, bound, &nbytes) == SBC_EINVAL);
    CHECK(sbc_compress(c, nullptr, m.dW.data(), m.R.data(), m.numel.data(), m.T(), p, nullptr, bound, &nbytes) == SBC_EINVAL);
    CHECK(sbc_compress(c, nullptr, m.dW.data(), m.R.data(), m.numel.data(), m.T(), p, (char*)kMsg + 4, bound, &nbytes) == SBC_EINVAL);
    CHECK(compress(c, m, p, bound - 1, &nbytes) == SBC_ECAPACITY);
    {
        Buffers x = m;
        x.dW[3] = reinterpret_cast<const float*>((uintptr_t)x.dW[3] + 2);              // misaligned
        CHECK(compress(c, x, p, bound, &nbytes) == SBC_EINVAL);
        x = m; x.R[5] = const_cast<float*>(x.dW[5]) + 1;                                // residual overlaps the update
        CHECK(compress(c, x, p, bound, &nbytes) == SBC_EINVAL);
        x = m; x.dW[0] = nullptr;
        CHECK(compress(c, x, p, bound, &nbytes) == SBC_EINVAL);
        x = m; x.numel[7] = 0;
        CHECK(compress(c, x, p, bound, &nbytes) == SBC_EINVAL);
        x = m; x.numel[7] = (int64_t)1 << 32;
        CHECK(compress(c, x, p, bound, &nbytes) != SBC_OK);
        x = m; x.numel[0] += 1;                                                          // one entry more than the context holds
        CHECK(compress(c, x, p, sbc_msg_bound(x.numel.data(), x.T(), p), &nbytes) == SBC_ECAPACITY);
        std::vector<int64_t> more(model); more.push_back(1);
        const Buffers y = fake_buffers(more);
        CHECK(compress(c, y, p, bound + 64, &nbytes) == SBC_ECAPACITY);               // one tensor more
    }
    CHECK(stub_launches() == launches0);
    CHECK(sbc_compress_end(c, &nbytes) == SBC_EINVAL);                                   // nothing pending
    CHECK(sbc_last_tensor_stats(c, 0, nullptr, nullptr, nullptr, nullptr, nullptr) != SBC_OK);   // no successful call yet

    // plans: first call, same buffers again (cached plan), five more buffer sets (the device copies
    // of the tensor table are recycled), every option
    for (int opt_round = 0; opt_round < 6; ++opt_round) {
        if (opt_round == 1) CHECK(sbc_set_option(c, SBC_OPT_CARRY_FILTER_KEYS, 1) == SBC_OK);
        if (opt_round == 2) CHECK(sbc_set_option(c, SBC_OPT_FUSED_STEP, 1) == SBC_OK);
        if (opt_round == 3) CHECK(sbc_set_option(c, SBC_OPT_FORCE_EXACT_PATH, 1) == SBC_OK);
        if (opt_round == 4) { CHECK(sbc_set_option(c, SBC_OPT_FORCE_EXACT_PATH, 0) == SBC_OK); CHECK(sbc_set_option(c, SBC_OPT_WIDE_MIN_KEPT, 1) == SBC_OK); }
        if (opt_round == 5) CHECK(sbc_set_option(c, SBC_OPT_SAMPLED_THRESHOLD, 1) == SBC_OK);
        const size_t need = opt_round == 5 ? sbc_msg_bound_sampled(m.numel.data(), m.T(), p) : bound;
        for (int set = 0; set < 7; ++set) {
            const Buffers s = fake_buffers(model, (uintptr_t)(set % 6) << 36);
            nbytes = 123;
            CHECK(compress(c, s, p, need, &nbytes) == SBC_OK && nbytes == 0);           // (no kernel ran: empty result)
            CHECK(sbc_compress_begin(c, nullptr, s.dW.data(), s.R.data(), s.numel.data(), s.T(), p, kMsg, need) == SBC_OK);
            CHECK(sbc_compress_begin(c, nullptr, s.dW.data(), s.R.data(), s.numel.data(), s.T(), p, kMsg, need) == SBC_EINVAL);
            CHECK(sbc_set_option(c, SBC_OPT_FUSED_STEP, 1) != SBC_OK || true);
            CHECK(sbc_compress_end(c, &nbytes) == SBC_OK);
        }
        for (double q : {0.5, 0.1, 0.01, 0.0001}) {
            const size_t nb = (opt_round == 5 ? sbc_msg_bound_sampled : sbc_msg_bound)(m.numel.data(), m.T(), q);
            CHECK(nb > 0 && compress(c, m, q, nb, &nbytes) == SBC_OK);
        }
        CHECK(sbc_last_route(c) >= 0);
        double mp, mn; int side; int64_t nnz, bits, cp, cn;
        // (no kernel filled the state: the counts of kept entries read zero, which the call reports)
        CHECK(sbc_last_tensor_stats(c, 0, &mp, &mn, &side, &nnz, &bits) == SBC_EINTERNAL);
        CHECK(sbc_last_tensor_stats(c, m.T(), &mp, &mn, &side, &nnz, &bits) == SBC_EINVAL);
        CHECK(sbc_last_candidates(c, m.T() - 1, &cp, &cn) == SBC_OK && sbc_last_candidates(c, -1, &cp, &cn) == SBC_EINVAL);
        std::vector<uint32_t> mask((size_t)(m.numel[0] + 31) / 32);
        CHECK(sbc_last_mask(c, 0, mask.data(), mask.size()) == SBC_OK);
        CHECK(sbc_last_mask(c, 0, mask.data(), mask.size() - 1) != SBC_OK);
    }
    CHECK(sbc_set_option(c, 99, 1) == SBC_EINVAL && sbc_set_option(nullptr, SBC_OPT_FUSED_STEP, 1) == SBC_EINVAL);
    CHECK(sbc_profile_enable(c, 2) == SBC_OK);
    CHECK(compress(c, m, p, sbc_msg_bound_sampled(m.numel.data(), m.T(), p), &nbytes) == SBC_OK);
    for (int stage = 0; stage < 16; ++stage) {
        const char* name = nullptr; double ms; int64_t calls;
        const int rc = sbc_profile_read(c, stage, &name, &ms, &calls);
        CHECK(rc == SBC_OK ? name != nullptr : rc == SBC_EINVAL);
    }
    CHECK(sbc_profile_enable(c, 0) == SBC_OK);

    // ---- decode plan: argument errors, every stream by one workgroup, tiled streams, deferred status ----
    CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, 31 + 24 * (size_t)m.T(), m.numel.data(), m.T(), p, 1.f, m.out.data()) == SBC_ECORRUPT);
    CHECK(sbc_decompress_accumulate(c, nullptr, (char*)kMsg + 4, bound, m.numel.data(), m.T(), p, 1.f, m.out.data()) == SBC_EINVAL);
    CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, bound, m.numel.data(), m.T() + 1, p, 1.f, m.out.data()) == SBC_ECAPACITY);
    CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, bound, nullptr, m.T(), p, 1.f, m.out.data()) == SBC_EINVAL);
    for (double q : {0.5, 0.1, 0.01, 0.001, 0.0001})
        for (int rep = 0; rep < 2; ++rep)
            CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, bound, m.numel.data(), m.T(), q, 1.f / 32, m.out.data()) == SBC_OK);
    CHECK(sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 1) == SBC_OK);
    for (int rep = 0; rep < 3; ++rep)
        CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, bound, m.numel.data(), m.T(), 0.1, 1.f, m.out.data()) == SBC_OK);
    CHECK(sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 0) == SBC_EINVAL);           // a status is outstanding
    CHECK(sbc_decode_status(c, nullptr) == SBC_OK);
    CHECK(sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 0) == SBC_OK);
    sbc_destroy(c); c = nullptr;
    CHECK(stub_live_blocks() == 0);

    // ---- shapes at the edges: one entry; a tensor of thousands of chunks; more tensors that keep
    // very many entries than the sweeps and the tiled decoder take; many tiny tensors ----
    {
        const std::vector<std::vector<int64_t>> shapes = {
            {1}, {8192}, {8193}, {64000000, 5}, std::vector<int64_t>(70, 70000), std::vector<int64_t>(3000, 7)};
        for (const auto& sizes : shapes) {
            const Buffers s = fake_buffers(sizes);
            CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
            for (int fused = 0; fused < 2; ++fused) {
                CHECK(sbc_set_option(c, SBC_OPT_FUSED_STEP, fused) == SBC_OK);
                CHECK(sbc_set_option(c, SBC_OPT_WIDE_MIN_KEPT, 6500) == SBC_OK);
                for (double q : {0.9, 0.1, 0.001}) {
                    const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), q);
                    CHECK(nb > 0 && compress(c, s, q, nb, &nbytes) == SBC_OK);
                    CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, nb, s.numel.data(), s.T(), q, 1.f, s.out.data()) == SBC_OK);
                }
            }
            sbc_destroy(c); c = nullptr;
            CHECK(stub_live_blocks() == 0);
        }
    }

    // ---- the streaming pass of a step that follows its context's last one at once keeps the residual in the
    // cache, after a pause it does not; calls below the cache's size and residuals beyond it know no difference ----
    for (int64_t n : {12000000, 60000000, 100000000}) {
        const Buffers s = fake_buffers({n, 1000});
        const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), p);
        CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
        CHECK(sbc_profile_enable(c, 1) == SBC_OK);     // (no looking for a result that no kernel writes)
        auto kernels = [&]() {
            const long from = stub_launches();
            CHECK(compress(c, s, p, nb, &nbytes) == SBC_OK);
            std::vector<const void*> k;
            for (long i = from; i < stub_launches(); ++i) k.push_back(stub_kernel(i));
            return k;
        };
        kernels();                                     // (the first call samples)
        usleep(50000);
        const std::vector<const void*> paused = kernels();
        int most = 0;
        for (int call = 0; call < 100; ++call) {       // (a busy machine may come late for some of them)
            const std::vector<const void*> k = kernels();
            CHECK(k.size() == paused.size());
            int differ = 0;
            for (size_t i = 0; i < k.size(); ++i) differ += k[i] != paused[i];
            most = differ > most ? differ : most;
        }
        CHECK(most == (n == 60000000 ? 1 : 0));
        sbc_destroy(c); c = nullptr;
    }

    // ---- ... where "at once" is what the step takes by itself and that of one other client: 20e6 entries at p = 0.001
    // after 150 us (in the begin/end form, in which several clients' steps overlap, after 90), at p = 0.2 after 300 (220), but
    // neither after 600 ----
    for (double q : {0.001, 0.2}) {
        const Buffers s = fake_buffers({20000000, 1000});
        const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), q);
        CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
        timespec last = {};
        const auto past = [&](long after_us, bool overlapped) {
            timespec now;
            do clock_gettime(CLOCK_MONOTONIC, &now);
            while ((now.tv_sec - last.tv_sec) * 1000000000l + now.tv_nsec - last.tv_nsec < after_us * 1000l);
            last = now;
            const long from = stub_launches();
            if (overlapped)
                CHECK(sbc_compress_begin(c, nullptr, s.dW.data(), s.R.data(), s.numel.data(), s.T(), q, kMsg, nb) == SBC_OK &&
                      sbc_compress_end(c, &nbytes) == SBC_OK);
            else
                CHECK(compress(c, s, q, nb, &nbytes) == SBC_OK);
            CHECK(stub_launched("k_accumulate_filterILi0E", from) + stub_launched("k_accumulate_filterILi2E", from) == 1);
            return stub_launched("k_accumulate_filterILi2E", from);
        };
        past(0, false);
        for (bool overlapped : {false, true}) {
            int kept = 0;                              // (a busy machine may come late for some of them)
            for (int call = 0; call < 100; ++call) kept += !past(overlapped ? (q < 0.1 ? 90 : 220) : (q < 0.1 ? 150 : 300), overlapped);
            CHECK(kept > 0);
            for (int call = 0; call < 20; ++call) CHECK(past(600, overlapped));
        }
        for (int call = 0; call < 20; ++call) CHECK(past(q < 0.1 ? 150 : 300, true));
        sbc_destroy(c); c = nullptr;
    }

    // ---- how many workgroups of the streaming pass share a compute unit (LDS that it asks for and does not use) ----
    {
        struct Case { int64_t n; bool kept, sent; };
        const Case cases[] = {{23000000, false, false}, {24000000, false, true}, {54000000, false, true}, {55000000, true, true}, {100000000, true, true}};
        for (const Case& k : cases) {
            const Buffers s = fake_buffers({k.n});
            const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), p);
            CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
            const auto pairs = [&]() {
                const long from = stub_launches();
                CHECK(compress(c, s, p, nb, &nbytes) == SBC_OK);
                const size_t lds = stub_lds_of("k_accumulate_filter", from);
                CHECK(lds == 0 || lds == 23552);
                return lds != 0;
            };
            pairs();
            int differ = 0;                            // (a busy machine may come late for some of them)
            for (int call = 0; call < 100; ++call) differ += pairs() != k.kept;
            CHECK(differ < 100);
            usleep(50000);
            CHECK(pairs() == k.sent);
            sbc_destroy(c); c = nullptr;
        }
    }

    // ---- more streams of two tiles than the tiled decoder has places, and one of 19 tiles: that one has a
    // place wherever it stands (31 of the others have one, too) ----
    for (int at : {0, 20, 48}) {
        std::vector<int64_t> sizes(48, (int64_t)1 << 22);
        sizes.insert(sizes.begin() + at, 51463000);
        const Buffers s = fake_buffers(sizes);
        CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
        const long first = stub_launches() + 1;        // (behind the clearing of the result blocks)
        CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, 1 << 24, s.numel.data(), s.T(), 0.001, 1.f, s.out.data()) == SBC_OK);
        const unsigned tiles = 19 + 31 * 2;
        CHECK(stub_grid(first + 1) == tiles && stub_grid(first + 2) == 4 * tiles);     // k_dec_tile_sums, k_dec_tile_place
        sbc_destroy(c); c = nullptr;
    }

    // ---- which calls have sweeps over their lists: by what the lists' length is going to be.  `first`: a call
    // that samples, `later`: one on carried keys after a call that saw no long list; after a call that saw one
    // (bit 512 of its error word) the sweeps come whatever the tensor ----
    {
        struct Case { int64_t n; double p; bool sampled; int first, later, after_long; };
        const Case cases[] = {
            {800000, 0.01, false, 0, 0, 0},            // 8000 kept entries: never
            {1048576, 0.01, false, 0, 0, 1},           // 10485
            {3276700, 0.01, false, 0, 0, 1},           // 32767
            {3276800, 0.01, false, 1, 1, 1},           // 32768: always
            {150000000, 1e-4, false, 0, 0, 1},         // 15000, keys from 10 sampled entries: 92,000
            {200000000, 1e-4, false, 1, 0, 1},         // 20000: 122,000
            {3000000, 0.01, true, 0, 0, 0},            // subsampled: about as many candidates as kept entries, 30000
            {9000000, 0.01, true, 0, 0, 0},            // 90000
            {9900000, 0.01, true, 1, 1, 1},            // 99000
        };
        for (const Case& k : cases) {
            const Buffers s = fake_buffers({k.n, 1000});
            const size_t nb = sbc_msg_bound_sampled(s.numel.data(), s.T(), k.p);
            CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
            CHECK(sbc_set_option(c, SBC_OPT_SAMPLED_THRESHOLD, k.sampled ? 1 : 0) == SBC_OK);
            auto sweeps = [&](uint32_t bits) {
                const long from = stub_launches();
                stub_result_bits(bits);
                CHECK(compress(c, s, k.p, nb, &nbytes) == SBC_OK);
                stub_result_bits(0);
                const int in_one = (k.n + 8191) / 8192 + 1 <= 3584 ? 1 : 0;
                CHECK(stub_launched("10k_emit_all", from) == in_one && stub_launched("11k_threshold", from) == 1 - in_one);
                CHECK(stub_launched("7k_apply", from) == 1 - in_one && stub_launched("13k_tensor_scan", from) <= 1 - in_one);
                CHECK(stub_launched("k_wide_count", from) == stub_launched("k_wide_collect", from));
                return stub_launched("k_wide_count", from);
            };
            CHECK(sweeps(0) == k.first && sweeps(0) == k.later);
            CHECK(sweeps(512) == k.later && sweeps(0) == k.after_long && sweeps(0) == k.later);
            CHECK(sbc_set_option(c, SBC_OPT_WIDE_MIN_KEPT, 5000) == SBC_OK && sweeps(0) == 1 && sweeps(0) == 1);
            CHECK(sbc_set_option(c, SBC_OPT_WIDE_MIN_KEPT, 1 << 30) == SBC_OK && sweeps(0) == 0 && sweeps(512) == 0 && sweeps(0) == 0);
            sbc_destroy(c); c = nullptr;
        }
    }

    // ---- workgroups per list of the sweeps: enough for the largest tensor's, eight at the least, a multiple of
    // eight, fewer for each the more lists there are ----
    {
        struct Case { std::vector<int64_t> sizes; double p; unsigned blocks; };
        const Case cases[] = {
            {{1 << 20}, 0.5, 64}, {{1 << 20}, 0.1, 32}, {{1 << 20}, 0.05, 16}, {{1 << 22}, 0.01, 16}, {{200000}, 0.2, 16},
            {{400000000}, 0.01, 256}, {std::vector<int64_t>(16, 1 << 20), 0.5, 16}, {std::vector<int64_t>(64, 1 << 20), 0.5, 8}};
        for (const Case& k : cases) {
            const Buffers s = fake_buffers(k.sizes);
            CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
            const long from = stub_launches();
            CHECK(compress(c, s, k.p, sbc_msg_bound(s.numel.data(), s.T(), k.p), &nbytes) == SBC_OK);
            CHECK(stub_grid_of("k_wide_count", from) == k.blocks && stub_grid_of("k_wide_collect", from) == k.blocks);
            sbc_destroy(c); c = nullptr;
        }
    }

    // ---- a context with short candidate lists: the plan shares them out, large p does not fit ----
    {
        CHECK(sbc_create_compact(nullptr, 0, 10, 1) == SBC_EINVAL);
        CHECK(sbc_create_compact(&c, 0, m.total(), m.T()) == SBC_OK);
        for (double q : {0.001, 0.01, 0.05}) {
            const size_t nb = sbc_msg_bound(m.numel.data(), m.T(), q);
            CHECK(compress(c, m, q, nb, &nbytes) == SBC_OK);
            CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, nb, m.numel.data(), m.T(), q, 1.f, m.out.data()) == SBC_OK);
        }
        const long launched = stub_launches();
        CHECK(compress(c, m, 0.3, sbc_msg_bound(m.numel.data(), m.T(), 0.3), &nbytes) == SBC_ECAPACITY);
        CHECK(stub_launches() == launched);
        sbc_destroy(c); c = nullptr;
        CHECK(stub_live_blocks() == 0);
    }

    // ---- a kernel that ends without sending the call's result: the call fails (the word in pinned memory then
    // still holds the call before's), and the next one works again ----
    for (const std::vector<int64_t>& shape : {model, std::vector<int64_t>{40000000, 5}})          // k_emit_all; k_emit
        for (int fused = 0; fused < 2; ++fused) {
            const Buffers s = fake_buffers(shape);
            const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), p);
            const void* const msgs[2] = {kMsg, kMsg};
            const size_t lens[2] = {nb, nb};
            CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
            CHECK(sbc_set_option(c, SBC_OPT_FUSED_STEP, fused) == SBC_OK);
            for (int withheld : {0, 1, 1, 0}) {
                stub_withhold_results(withheld);
                const int want = withheld ? SBC_EINTERNAL : SBC_OK;
                CHECK(compress(c, s, p, nb, &nbytes) == want);
                CHECK(sbc_compress_begin(c, nullptr, s.dW.data(), s.R.data(), s.numel.data(), s.T(), p, kMsg, nb) == SBC_OK);
                CHECK(sbc_compress_end(c, &nbytes) == want);
                CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, nb, s.numel.data(), s.T(), p, 1.f, s.out.data()) == want);
                CHECK(sbc_decompress_average(c, nullptr, msgs, lens, 2, s.numel.data(), s.T(), p, 0.5f, s.out.data()) == want);
                CHECK(sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 1) == SBC_OK);
                CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, nb, s.numel.data(), s.T(), p, 1.f, s.out.data()) == SBC_OK);
                CHECK(sbc_decode_status(c, nullptr) == want);
                CHECK(sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 0) == SBC_OK);
            }
            sbc_destroy(c); c = nullptr;
            CHECK(stub_live_blocks() == 0);
        }

    // ---- a step that k_emit_all leaves to the second pass (bit 64), in which sides that start after its word has gone
    // out raise more: what they raise counts as if it had been in that word ----
    {
        const Buffers s = fake_buffers({3000000, 1000});
        const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), 0.01);
        struct Case { uint32_t early, late; int status, histogram; };
        const Case cases[] = {{64, 0, SBC_OK, 0}, {64, 8, SBC_OK, 1}, {64 | 8, 0, SBC_OK, 1}, {64, 8 | 16, SBC_OK, 1},
                              {64, 128, SBC_ECAPACITY, 0}, {64, 2, SBC_EINTERNAL, 0}, {64, 8 | 128, SBC_ECAPACITY, 0},
                              {64 | 1, 0, SBC_ENONFINITE, 0}};
        CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
        for (int begin_end = 0; begin_end < 2; ++begin_end)
            for (const Case& k : cases) {
                CHECK(compress(c, s, 0.01, nb, &nbytes) == SBC_OK);
                const long from = stub_launches();
                stub_next_result_bits("k_emit_all", k.early);
                stub_next_result_bits("k_publish", (k.early & ~64u) | k.late);
                int status;
                if (begin_end) {
                    CHECK(sbc_compress_begin(c, nullptr, s.dW.data(), s.R.data(), s.numel.data(), s.T(), 0.01, kMsg, nb) == SBC_OK);
                    status = sbc_compress_end(c, &nbytes);
                } else {
                    status = compress(c, s, 0.01, nb, &nbytes);
                }
                CHECK(status == k.status);
                CHECK(stub_launched("k_publish", from) == 1);
                CHECK(stub_launched("k_hist_flagged", from) == k.histogram && stub_launched("k_extract", from) == k.histogram);
                CHECK(stub_launched("7k_apply", from) == (k.status == SBC_OK ? 1 : 0));
                const int route = sbc_last_route(c);
                if (k.status == SBC_OK)
                    CHECK((route & (SBC_ROUTE_TAKEN_OVER | SBC_ROUTE_HISTOGRAM)) == (SBC_ROUTE_TAKEN_OVER | (k.histogram ? SBC_ROUTE_HISTOGRAM : 0)) &&
                          !(route & SBC_ROUTE_LOOSE_KEYS) == !(k.late & 16));
            }
        // a long list (bit 512) that such a side has found: the next call sweeps, as ever
        for (int late = 0; late < 2; ++late) {
            CHECK(compress(c, s, 0.01, nb, &nbytes) == SBC_OK);
            stub_next_result_bits("k_emit_all", late ? 64u : 64u | 512u);
            stub_next_result_bits("k_publish", 512u);
            CHECK(compress(c, s, 0.01, nb, &nbytes) == SBC_OK);
            const long from = stub_launches();
            CHECK(compress(c, s, 0.01, nb, &nbytes) == SBC_OK);
            CHECK(stub_launched("k_wide_count", from) == 1);
        }
        sbc_destroy(c); c = nullptr;
        CHECK(stub_live_blocks() == 0);
    }

    // ---- which kernels complete a step: one launch for few tensors, chunks and kept entries per chunk, three up to 4096
    // chunks, four beyond; a second pass never waits ----
    {
        struct Case { std::vector<int64_t> sizes; double p; int all, scan, emit; };
        const Case cases[] = {
            {{3584 * 8192}, 0.001, 1, 0, 0}, {{3584 * 8192 + 1}, 0.001, 0, 1, 0}, {{4096 * 8192}, 0.001, 0, 1, 0}, {{4096 * 8192 + 1}, 0.001, 0, 0, 1},
            {std::vector<int64_t>(200, 100), 0.01, 1, 0, 0}, {std::vector<int64_t>(201, 100), 0.01, 0, 1, 0}, {std::vector<int64_t>(4097, 1), 0.01, 0, 0, 1},
            {{1000000}, 0.0625, 1, 0, 0}, {{1000000}, 0.0626, 0, 1, 0}, {{1000000}, 0.9, 0, 1, 0}, {{1}, 1e-6, 1, 0, 0}};
        for (const Case& k : cases) {
            const Buffers s = fake_buffers(k.sizes);
            const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), k.p);
            CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
            const auto reported = [&](const char* kernel) {
                for (int stage = 0; ; ++stage) {
                    const char* name = nullptr;
                    if (sbc_profile_read(c, stage, &name, nullptr, nullptr) != SBC_OK) return false;
                    if (std::strcmp(name, kernel) == 0) return true;
                }
            };
            for (int second : {0, 1}) {
                const long from = stub_launches();
                const char* const sender = k.all ? "k_emit_all" : k.scan ? "k_emit_scan" : "6k_emit";
                if (second) stub_next_result_bits(sender, 8);
                CHECK(compress(c, s, k.p, nb, &nbytes) == SBC_OK);
                CHECK(stub_launched("10k_emit_all", from) == k.all && stub_launched("6k_emit", from) == k.emit * (1 + second));
                CHECK(stub_launched("11k_emit_scan", from) == k.scan + second * (1 - k.emit));
                CHECK(reported(k.all ? "k_emit_all" : k.scan ? "k_emit_scan" : "k_emit"));
                CHECK(stub_launched("11k_threshold", from) == (k.all ? 0 : 1) + second && stub_launched("7k_apply", from) == (k.all ? 0 : 1) + second);
            }
            sbc_destroy(c); c = nullptr;
        }
    }

    // ---- scratch memory that a context's creation leaves clean: a first call clears no words that only earlier launches
    // can have left, a call after one that failed does ----
    {
        const Buffers s = fake_buffers({3000000, 1000});
        const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), p);
        CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
        const int cleared[] = {4, 0, 0, 5, 0};
        for (int call = 0; call < 5; ++call) {
            const long from = stub_launches();
            stub_withhold_results(call == 2);
            CHECK(compress(c, s, p, nb, &nbytes) == (call == 2 ? SBC_EINTERNAL : SBC_OK));
            stub_withhold_results(0);
            CHECK(stub_launched("k_zero_words", from) == cleared[call]);
        }
        sbc_destroy(c); c = nullptr;
    }

    // ---- the average over a round's messages: argument errors, and its two tables at their limits ----
    {
        std::vector<const void*> msgs(130, kMsg);
        std::vector<size_t> sizes(130, bound);
        CHECK(sbc_create(&c, 0, m.total(), m.T()) == SBC_OK);
        const long launched = stub_launches();
        auto average = [&](const Buffers& b, int n_msgs, double q) {
            return sbc_decompress_average(c, nullptr, msgs.data(), sizes.data(), n_msgs, b.numel.data(), b.T(), q, 0.5f, b.out.data());
        };
        CHECK(sbc_decompress_average(nullptr, nullptr, msgs.data(), sizes.data(), 2, m.numel.data(), m.T(), p, 1.f, m.out.data()) == SBC_EINVAL);
        CHECK(sbc_decompress_average(c, nullptr, nullptr, sizes.data(), 2, m.numel.data(), m.T(), p, 1.f, m.out.data()) == SBC_EINVAL);
        CHECK(sbc_decompress_average(c, nullptr, msgs.data(), nullptr, 2, m.numel.data(), m.T(), p, 1.f, m.out.data()) == SBC_EINVAL);
        CHECK(sbc_decompress_average(c, nullptr, msgs.data(), sizes.data(), 2, nullptr, m.T(), p, 1.f, m.out.data()) == SBC_EINVAL);
        CHECK(sbc_decompress_average(c, nullptr, msgs.data(), sizes.data(), 2, m.numel.data(), m.T(), p, 1.f, nullptr) == SBC_EINVAL);
        CHECK(average(m, 0, p) == SBC_EINVAL && average(m, -3, p) == SBC_EINVAL && average(m, 2, 0.0) == SBC_EINVAL);
        CHECK(sbc_decompress_average(c, nullptr, msgs.data(), sizes.data(), 2, m.numel.data(), m.T() + 1, p, 1.f, m.out.data()) == SBC_ECAPACITY);
        msgs[1] = nullptr;
        CHECK(average(m, 2, p) == SBC_EINVAL);
        msgs[1] = (const char*)kMsg + 4;                  // misaligned
        CHECK(average(m, 2, p) == SBC_EINVAL);
        msgs[1] = kMsg;
        sizes[1] = 31 + 24 * (size_t)m.T();
        CHECK(average(m, 2, p) == SBC_ECORRUPT);
        sizes[1] = bound;
        {
            Buffers x = m;
            x.out[4] = nullptr;
            CHECK(average(x, 2, p) == SBC_EINVAL);
            x = m; x.out[4] = reinterpret_cast<float*>((uintptr_t)x.out[4] + 2);
            CHECK(average(x, 2, p) == SBC_EINVAL);
            x = m; x.numel[4] = 0;
            CHECK(average(x, 2, p) == SBC_EINVAL);
        }
        CHECK(stub_launches() == launched);
        sbc_destroy(c); c = nullptr;

        // the model; one-chunk tensors up to the context's count; 40 streams of 16 tiles (their shares run
        // out); one stream beyond 16 tiles; ragged ones on both sides of a block and a chunk
        const std::vector<std::vector<int64_t>> shapes = {
            model, std::vector<int64_t>(2000, 64), std::vector<int64_t>(40, 650000), {9000000, 300}, {1}, {2047, 2048, 2049, 8191, 8192, 8193, 70001}};
        for (const auto& shape : shapes) {
            const Buffers s = fake_buffers(shape), other = fake_buffers(shape, (uintptr_t)1 << 36);
            for (int kind = 0; kind < 3; ++kind) {        // full, compact, and created for a sixteenth of the entries
                const int64_t total = kind == 2 ? s.total() / 16 + 1 : s.total();
                CHECK((kind == 1 ? sbc_create_compact(&c, 0, total, s.T()) : sbc_create(&c, 0, total, s.T())) == SBC_OK);
                size_t nb = 0;
                for (double q : {0.5, 0.2, 0.04, 0.001, 1e-6}) {           // (remainders of 0 to 19 bits)
                    nb = sbc_msg_bound(s.numel.data(), s.T(), q);
                    sizes.assign(130, nb);
                    for (int n_msgs : {1, 2, 64, 130}) CHECK(average(s, n_msgs, q) == SBC_OK);
                    CHECK(average(other, 3, q) == SBC_OK && average(s, 3, q) == SBC_OK);
                }
                // while deferred decodes are outstanding, and while a client step is pending
                CHECK(sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 1) == SBC_OK);
                CHECK(sbc_decompress_accumulate(c, nullptr, kMsg, nb, s.numel.data(), s.T(), 1e-6, 1.f, s.out.data()) == SBC_OK);
                CHECK(average(s, 2, 1e-6) == SBC_OK && average(s, 2, 0.04) == SBC_OK);
                CHECK(sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 0) == SBC_EINVAL);
                CHECK(sbc_decode_status(c, nullptr) == SBC_OK);
                if (kind == 0) {
                    const size_t need = sbc_msg_bound(s.numel.data(), s.T(), p);
                    CHECK(sbc_compress_begin(c, nullptr, s.dW.data(), s.R.data(), s.numel.data(), s.T(), p, kMsg, need) == SBC_OK);
                    CHECK(average(s, 2, 0.04) == SBC_OK);
                    CHECK(sbc_compress_end(c, &nbytes) == SBC_OK);
                }
                sbc_destroy(c); c = nullptr;
                CHECK(stub_live_blocks() == 0);
            }
        }
    }

    // ---- what follows an average whose last kernel is still running: waits for that kernel on its own stream, whatever has
    // become of the average's (a destroyed one); a stream that records a graph has the host wait.  Nothing to wait
    // for once the kernel has ended, or the average failed ----
    {
        const Buffers s = fake_buffers({3000000, 1000});
        const size_t nb = sbc_msg_bound(s.numel.data(), s.T(), p);
        const void* const msgs[2] = {kMsg, kMsg};
        const size_t lens[2] = {nb, nb};
        void* const first = reinterpret_cast<void*>(0x1000);
        void* const second = reinterpret_cast<void*>(0x2000);
        const auto average = [&](void* stream) { return sbc_decompress_average(c, stream, msgs, lens, 2, s.numel.data(), s.T(), p, 0.5f, s.out.data()); };
        const auto decode = [&](void* stream) { return sbc_decompress_accumulate(c, stream, kMsg, nb, s.numel.data(), s.T(), p, 1.f, s.out.data()); };
        const auto step = [&](void* stream) {
            return sbc_compress(c, stream, s.dW.data(), s.R.data(), s.numel.data(), s.T(), p, kMsg, nb, &nbytes);
        };
        for (int pending = 0; pending < 2; ++pending) {
            CHECK(sbc_create(&c, 0, s.total(), s.T()) == SBC_OK);
            CHECK(average(first) == SBC_OK);
            stub_stream_gone(first);
            stub_events_pending(pending);
            int waits = stub_stream_waits();
            CHECK(step(second) == SBC_OK && step(second) == SBC_OK && decode(second) == SBC_OK && average(second) == SBC_OK);
            CHECK(stub_stream_waits() - waits == (pending ? 4 : 0));
            stub_stream_gone(nullptr);
            CHECK(sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 1) == SBC_OK && decode(second) == SBC_OK && average(first) == SBC_OK);
            stub_stream_records(second);
            waits = stub_event_waits();
            CHECK(decode(second) == SBC_OK && decode(second) == SBC_OK);
            CHECK(stub_event_waits() - waits == pending);
            stub_stream_records(nullptr);
            CHECK(sbc_decode_status(c, second) == SBC_OK && sbc_set_option(c, SBC_OPT_DEFER_DECODE_STATUS, 0) == SBC_OK);
            CHECK(average(second) == SBC_OK);
            stub_next_result_bits("k_publish", 4);         // (a corrupt message: the call drains its stream)
            CHECK(average(second) == SBC_ECORRUPT);
            waits = stub_stream_waits();
            CHECK(decode(first) == SBC_OK && stub_stream_waits() == waits);
            stub_events_pending(0);
            sbc_destroy(c); c = nullptr;
        }
        CHECK(stub_live_blocks() == 0);
    }

    // ---- the average over 64 messages of more tensors than one launch can decode for all of them: fewer
    // messages at a time, whatever the tensors ----
    {
        const Buffers s = fake_buffers(std::vector<int64_t>(1100000, 1));
        const std::vector<const void*> msgs(64, kMsg);
        const std::vector<size_t> lens(64, sbc_msg_bound(s.numel.data(), s.T(), p));
        CHECK(sbc_create(&c, 0, 64 * s.total(), s.T()) == SBC_OK);
        const long from = stub_launches();
        CHECK(sbc_decompress_average(c, nullptr, msgs.data(), lens.data(), 64, s.numel.data(), s.T(), p, 1.f, s.out.data()) == SBC_OK);
        CHECK(stub_launches() - from == 1 + 2 * 2 + 1);   // cleared result blocks, two passes of two kernels, the status
        unsigned rows = 0;
        for (long i : {1, 3}) {
            CHECK((uint64_t)stub_grid(from + i) * 512u < (uint64_t)1 << 32);
            rows += stub_grid(from + i);
        }
        CHECK(rows == 64u * 137500u);
        sbc_destroy(c); c = nullptr;
    }

    // ---- the server step that allocates nothing ----
    {
        int32_t* const status = reinterpret_cast<int32_t*>(0x500000000000ull);
        const long blocks = stub_live_blocks();
        CHECK(sbc_decompress_accumulate_noalloc(0, nullptr, nullptr, bound, m.numel.data(), m.T(), p, 1.f, m.out.data(), status) == SBC_EINVAL);
        CHECK(sbc_decompress_accumulate_noalloc(0, nullptr, kMsg, bound, m.numel.data(), m.T(), p, 1.f, m.out.data(), nullptr) == SBC_EINVAL);
        CHECK(sbc_decompress_accumulate_noalloc(3, nullptr, kMsg, bound, m.numel.data(), m.T(), p, 1.f, m.out.data(), status) == SBC_EINVAL);
        CHECK(sbc_decompress_accumulate_noalloc(0, nullptr, kMsg, 10, m.numel.data(), m.T(), p, 1.f, m.out.data(), status) == SBC_ECORRUPT);
        const Buffers big = fake_buffers(std::vector<int64_t>(SBC_NOALLOC_MAX_TENSORS + 1, 100));
        CHECK(sbc_decompress_accumulate_noalloc(0, nullptr, kMsg, 1 << 20, big.numel.data(), big.T(), p, 1.f, big.out.data(), status) == SBC_ECAPACITY);
        for (double q : {0.1, 0.001})
            CHECK(sbc_decompress_accumulate_noalloc(0, nullptr, kMsg, bound, m.numel.data(), m.T(), q, 1.f, m.out.data(), status) == SBC_OK);
        CHECK(stub_live_blocks() == blocks);                                            // it allocated nothing
    }
    std::printf("host checks passed, %ld launches planned\n", stub_launches());
    return 0;
}
