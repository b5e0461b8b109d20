// When the library's host side lets go of the caller's arrays, shown without a device (tests/test_sanitized_host.py
// compiles and runs it).  The device operations of kernels.hip are replaced: an asynchronous copy reads its source as
// late as it may, when the stream is next waited for or after the caller has overwritten the array it passed.  What the
// replay would then find on the device must be what was passed.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "internal.h"

namespace {

struct Copy {
    void* dst;
    const void* src;
    size_t bytes;
};
std::vector<Copy> pending;
const uint64_t* launched_seeds = nullptr;
int launched = 0;

void perform() {
    for (const Copy& c : pending) std::memcpy(c.dst, c.src, c.bytes);
    pending.clear();
}

}  // namespace

namespace gorgo {

bool pack_replays(const Plan&, int64_t) { return false; }
Workgroups replay_workgroups(const Plan&, int32_t, int32_t, bool, bool) { return {1, 4}; }
int launch_replay(const gorgo_trace*, const Plan&, const double*, const double*, const double*, uint8_t*, uint16_t*, double*,
                  double*, void*, void*, const OnlineLaunch*, const PolicyLaunch* policy, const EngineLaunch*, const ProxyLaunch*,
                  unsigned long long*) {
    // (the small inputs travel as arguments of the launch: nothing here waits for the stream)
    launched_seeds = policy ? policy->seeds : nullptr;
    ++launched;
    return GORGO_OK;
}
int last_eval_kernel_ms(double*, double*, double*) { return GORGO_OK; }
int upload_trace(const gorgo_trace*) { return GORGO_OK; }
bool trace_is_resident(const gorgo_trace*) { return true; }
int static_scratch(void**, size_t*) { return GORGO_ERR_DEVICE; }
void set_event_marks(bool) {}
void release_device_trace(gorgo_trace*) {}
int copy_small_to_device(void* dst, const void* src, size_t bytes, void*) {
    pending.push_back(Copy{dst, src, bytes});
    return GORGO_OK;
}
int wait_for_copies(void*) {
    perform();
    return GORGO_OK;
}
int copy_small_to_host_sync(void*, const void*, size_t, void*) { return GORGO_OK; }

}  // namespace gorgo

#define CHECK(cond)                                                                                     \
    do {                                                                                                \
        if (!(cond)) {                                                                                  \
            std::fprintf(stderr, "host_copies: check failed at line %d: %s (last error: %s)\n", __LINE__, #cond, \
                         gorgo_last_error());                                                           \
            std::exit(3);                                                                               \
        }                                                                                               \
    } while (0)

// The random policy's seeds, under the linear replica model and under the engine model.
static void seeds_outlive_the_callers_array(const gorgo_trace* t, const gorgo_model& m, int P, bool engine) {
    gorgo_outputs want;
    std::memset(&want, 0, sizeof want);
    size_t bytes = 0;
    CHECK(gorgo_workspace_bytes(t, &m, nullptr, P, &want, &bytes) == GORGO_OK);
    void* ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    CHECK(ws != nullptr);
    const std::vector<double> rtt((size_t)m.R, 10.0), scale((size_t)P, 1.0), rate((size_t)m.R, 0.05);
    std::vector<uint64_t>* const seeds = new std::vector<uint64_t>((size_t)P);
    for (int p = 0; p < P; ++p) (*seeds)[p] = 0x9E3779B97F4A7C15ull * (uint64_t)(p + 1);
    const std::vector<uint64_t> passed = *seeds;
    launched = 0;
    if (engine) {
        gorgo_engine e;
        std::memset(&e, 0, sizeof e);
        e.prefill_ms_per_token = rate.data();
        e.decode_ms_per_token = rate.data();
        CHECK(gorgo_eval_engine(t, &m, nullptr, &e, rtt.data(), GORGO_POLICY_RANDOM, nullptr, seeds->data(), nullptr, scale.data(), P,
                                &want, ws, bytes, nullptr) == GORGO_OK);
    } else {
        CHECK(gorgo_eval_policy(t, &m, nullptr, rtt.data(), GORGO_POLICY_RANDOM, seeds->data(), scale.data(), P, &want, ws, bytes,
                                nullptr) == GORGO_OK);
    }
    CHECK(launched == 1 && launched_seeds != nullptr);
    std::fill(seeds->begin(), seeds->end(), 0);       // the caller's array is the caller's again
    for (const Copy& c : pending) CHECK(c.src != seeds->data());
    perform();
    CHECK(std::memcmp(launched_seeds, passed.data(), sizeof(uint64_t) * passed.size()) == 0);
    delete seeds;
    std::free(ws);
}

int main() {
    const int64_t ts[3] = {0, 10, 20}, off[4] = {0, 2, 4, 7}, ids[7] = {1, 2, 1, 2, 1, 2, 3};
    const int32_t in_len[3] = {1000, 1000, 1500}, out_len[3] = {10, 20, 30};
    gorgo_trace* t = nullptr;
    CHECK(gorgo_load_trace_arrays(3, ts, in_len, out_len, off, ids, 512, &t) == GORGO_OK);
    gorgo_model m;
    std::memset(&m, 0, sizeof m);
    m.R = 3;
    m.batch = 2;
    m.block_tokens = 512;
    m.cache_blocks = 0;
    m.prefill_ms_per_token = 0.05;
    m.decode_ms_per_token = 20.0;
    int calls = 0;
    for (int P : {1, 2, 111, 112, 300})               // (either side of where the small inputs stop being arguments)
        for (bool engine : {false, true}) {
            seeds_outlive_the_callers_array(t, m, P, engine);
            ++calls;
        }
    gorgo_free_trace(t);
    std::printf("%d calls\n", calls);
    return 0;
}
