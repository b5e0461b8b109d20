// Internal declarations shared by the host-side translation units of libgorgo.
#pragma once
#include <cstdint>
#include <cstddef>
#include <string>
#include <vector>

#include "gorgo.h"

namespace gorgo {

// thread-local error text behind gorgo_last_error()
int fail(int code, const std::string& msg);
void clear_error();

// One segment of a request's block list: segment id and the number of the request's blocks up to and
// including this segment.
struct SegRef {
    int32_t id;       // in the loaded trace: the row slot the segment occupies while it is referenced
    int32_t end;      // | SEG_FRESH where this is the segment's first reference (its row slot starts over there)
};
constexpr int32_t SEG_FRESH = 1 << 30;
constexpr int32_t SEG_END_MASK = 0xFFFF;     // (a request has fewer than 2^16 blocks)

// One block of a request, for the block formulation over rows: the row slot of its id, and marks.
constexpr uint32_t ROW_SLOT = (1u << 27) - 1;
constexpr uint32_t ROW_FIRST = 1u << 27;         // first occurrence within the request
constexpr uint32_t ROW_FRESH = 1u << 28;         // the id's first request in the trace: its row starts over there
constexpr uint32_t ROW_NEW_BEFORE = 1u << 29;    // ... was the request before this one
constexpr uint32_t ROW_IN_BEFORE = 1u << 30;     // the request before this one has the id as well

// Device-resident copy of a trace (filled lazily by the first evaluation).
struct DeviceTrace {
    int device = -1;
    void* base = nullptr;          // one allocation holding every array below
    const int64_t* ts = nullptr;   // [N]
    const int32_t* in_len = nullptr;
    const int32_t* out_len = nullptr;
    const int64_t* blk_off = nullptr;   // [N+1]
    const uint32_t* key = nullptr;      // [total] dense block key (1-based)
    const uint8_t* first = nullptr;     // [total] 1 = first occurrence of its key inside the request
    const int64_t* seg_off = nullptr;   // [N+1] (chain-consistent traces only)
    const SegRef* seg = nullptr;        // [seg_off[N]]
    const uint32_t* first_hash = nullptr;   // [N] hash of the request's first block (session-affinity policy)
    const int32_t* seg_prev = nullptr;      // [seg_off[N]] latest request before with the same segment, -1: none
    const uint32_t* row_ref = nullptr;      // [total] (traces that do not go by segments only)
};

}  // namespace gorgo

// The opaque handle of the C ABI.
struct gorgo_trace {
    int64_t N = 0;
    int32_t block_tokens = 0;
    std::vector<int64_t> ts;
    std::vector<int32_t> in_len, out_len;
    std::vector<int64_t> blk_off;
    std::vector<uint32_t> key;       // dense remap of hash ids: 1 + order of first appearance in the file
    std::vector<uint8_t> first;
    std::vector<uint32_t> first_hash;   // per request: high word of SplitMix64's output for its first block id
    int64_t total_blocks = 0;
    int32_t max_blocks = 0;          // largest n_r
    int32_t max_distinct = 0;        // largest number of distinct ids in one request
    int64_t unique_ids = 0;
    bool chain_consistent = true;
    std::vector<int64_t> seg_off;    // chain-consistent traces: request -> its segments
    std::vector<gorgo::SegRef> seg;
    std::vector<int32_t> seg_prev;
    int64_t n_segments = 0;
    int64_t n_slots = 0;             // rows a replay needs: the most segments in use at one time
    std::vector<uint32_t> row_ref;   // traces that do not go by segments: row slot and marks of every block
    int64_t n_row_slots = 0;         // the most ids in use at one time
    gorgo::DeviceTrace dev;
};

namespace gorgo {

// whether a chain-consistent trace's requests are few segments long (each then costs a handful of row reads)
inline bool segments_suit(const gorgo_trace* t) { return (int64_t)t->seg.size() <= 16 * (t->N > 0 ? t->N : 1); }

// Geometry of one evaluation, computed on the host and handed to the launchers.
enum ReplayPath { PATH_AUTO = 0, PATH_BLOCKS = 1, PATH_SEGMENTS = 2 };

// A share of a chunk's requests (replay_each.h): segment references, blocks, requests.
struct EachCount {
    int64_t segs, blocks, count;
};

// Workspace of replay_each.h (byte offsets): P replays of N requests with T segment references on R replicas.
struct EachSpace {
    size_t where, count, from, list, ts, seg_off, blk_off, in_len, out_len, seg, hit, ttft, e2e, total;
    EachSpace(size_t P, size_t N, size_t T, size_t R) {
        total = 0;
        auto take = [&](size_t bytes) {
            const size_t at = total;
            total += (bytes + 255) & ~(size_t)255;
            return at;
        };
        where = take(P * N);
        count = take(P * ((N + 1023) / 1024) * R * sizeof(EachCount));
        from = take(P * (R + 1) * 4);
        list = take(P * N * 4);
        ts = take(P * N * 8);
        seg_off = take(P * (N + R) * 8);
        blk_off = take(P * (N + R) * 8);
        in_len = take(P * N * 4);
        out_len = take(P * N * 4);
        seg = take(P * (T + 1) * sizeof(SegRef));
        hit = take(P * N * 2);
        ttft = take(P * N * 8);
        e2e = take(P * N * 8);
    }
};

struct Plan {
    int32_t path = PATH_BLOCKS;      // PATH_BLOCKS: hashed block tables; PATH_SEGMENTS: dense segment rows
    int64_t nseg = 0;
    int32_t P = 0, R = 0, B = 0;
    int64_t N = 0, C = 0;
    double requests_held = 0;        // by a replica's cache, requests of the trace's mean length
    int64_t cap = 0;                 // slots per (replay, replica) table, power of two
    int64_t row_slots = 0;           // block formulation: rows of stamps instead of tables where not 0
    bool each = false;               // segment formulation: a workgroup per replay and replica (routes that a policy dictates)
    int32_t row_words = 0;           // ... and words of a log record
    int32_t block_tokens = 0;
    double a_pf = 0, a_dec = 0;
    int32_t packing = 2;             // gorgo_options::replay_packing of the call
    // workspace carve-up (byte offsets from the workspace base)
    size_t off_tables = 0, off_spare = 0, off_rec = 0, off_route = 0, off_ttft = 0, off_e2e = 0, off_small = 0, off_each = 0;
    size_t total = 0;
    // [P] nearest-rank percentiles to be computed (device pointers), or null
    double *p95_ttft = nullptr, *p95_e2e = nullptr;
    // the small inputs on the host, which the launch brings to d_rtt, d_params and d_scale (adjacent, in this order);
    // keep_copies: they are the library's own and go away when the call returns
    const double *h_rtt = nullptr, *h_params = nullptr, *h_scale = nullptr;
    bool keep_copies = false;
};

// Online tuner of one launch (device pointers; see gorgo_online in gorgo.h).
struct OnlineLaunch {
    int32_t window = 0, hop = 0;
    int64_t steps = 0;
    const double* tuner = nullptr;       // lo[3], hi[3], ln lo[3], ln hi[3], sigma0, exp(0.4), exp(-0.1)
    const double* ln_theta0 = nullptr;   // [P][3]
    const double* z = nullptr;
    double* theta_step = nullptr;
    double* fitness_step = nullptr;
    double* theta_final = nullptr;
    double* sigma_final = nullptr;
    int32_t* accepted = nullptr;
};
constexpr int TUNER_CONSTS = 16;         // doubles reserved for OnlineLaunch::tuner

// How a replay picks replicas (gorgo_policy in gorgo.h) and, for the random policy, the seeds of the replays.
struct PolicyLaunch {
    int32_t policy = 0;
    const uint64_t* seeds = nullptr;     // device [P]
};

// Engine model of a replica of one launch (device pointers; see gorgo_engine in gorgo.h).
struct EngineLaunch {
    const double* a_pf = nullptr;        // [R]
    const double* a_dec = nullptr;       // [R]
    const double* budget = nullptr;      // [R] KV tokens as doubles, 0 = none
    double slowdown = 0.0;
    double least_dec = 0.0;              // smallest decode rate
};

// Imperfect proxy knowledge of one launch (device pointers; see gorgo_proxy in gorgo.h).
struct ProxyLaunch {
    int32_t epochs = 0, probe_ms = 0;
    const double* rtt_true = nullptr;    // [epochs][R]
    double* rtt_est = nullptr;           // [epochs][R], written by the launch before the replay
    double alpha = 1.0;
    int64_t index_blocks = -1;
    uint16_t* believed = nullptr;        // [P][N], nullable
};

// kernels.hip
bool pack_replays(const Plan& pl, int64_t rows);     // rows of one replay: its segments + 2
struct Workgroups {
    int32_t replays, wavefronts;         // of a workgroup (0 replays: a workgroup for each replica of a replay)
};
Workgroups replay_workgroups(const Plan& pl, int32_t policy, int32_t window, bool engine, bool proxy);      // window 0: no tuner
int launch_replay(const gorgo_trace* t, const Plan& pl, const double* d_rtt, const double* d_params,
                  const double* d_scale, uint8_t* route, uint16_t* hit, double* ttft, double* e2e,
                  void* workspace, void* stream, const OnlineLaunch* online = nullptr,
                  const PolicyLaunch* policy = nullptr, const EngineLaunch* engine = nullptr,
                  const ProxyLaunch* proxy = nullptr, unsigned long long* sections = nullptr);
int last_eval_kernel_ms(double* fill_ms, double* replay_ms, double* select_ms);
int upload_trace(const gorgo_trace* t);
bool trace_is_resident(const gorgo_trace* t);          // on the current device
int static_scratch(void** ptr, size_t* bytes);         // device address and size of the library's static scratch array
void set_event_marks(bool on);                         // whether this thread's evaluations record timing events
void release_device_trace(gorgo_trace* t);
int copy_small_to_device(void* dst, const void* src, size_t bytes, void* stream);
int wait_for_copies(void* stream);
int copy_small_to_host_sync(void* dst, const void* src, size_t bytes, void* stream);

}  // namespace gorgo
