// Device side: the launches of the replay kernels (segment rows: replay_segments.h; block
// tables: replay_blocks.h), the exact percentile selection, and the trace upload.
//
// Decision arithmetic is fp64 with every product and sum rounded separately (built with -ffp-contract=off)
// in the association (w_rtt*rtt + w_prefill*pf) + w_queue*qd, so that routes are reproducible bit for bit.
#include <atomic>
#include <hip/hip_runtime.h>
#include <mutex>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <new>
#include <string>

#include "device_common.h"
#include "internal.h"
#include "replay_apart.h"
#include "replay_blocks.h"
#include "replay_each.h"
#include "replay_rows.h"
#include "replay_segments.h"

namespace gorgo {

namespace {

// What a launch needs before its replays start: the small inputs (round trip times, weights, time scales), which travel as
// arguments of the kernel where they fit, and the cell value that is below any cursor in the last row but one of every
// replay's rows (the one no request touches; rows: null for block tables).  (With three copies
// from pageable host memory and a launch a ten-request replay takes 57.5 us, so 47.3; arguments also are taken when the
// launch is enqueued, so nothing has to be waited for before the library's own arrays go away.)
constexpr int SMALL_INPUTS = 448;      // doubles: the arguments of a launch are limited to 4 KiB
struct SmallInputs {
    double v[SMALL_INPUTS];
};
__global__ void __launch_bounds__(256) prepare_replays(SmallInputs in, int count, double* dst, int32_t* last, int32_t P, int64_t rows,
                                                       int32_t R, int32_t v) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (size_t)count) dst[i] = in.v[i];
    if (last && i < (size_t)P * R) last[((i / R) * (size_t)rows + (size_t)(rows - 2)) * R + i % R] = v;
}

// ---- exact nearest-rank percentile: the k-th smallest of x[p][0..N) on the order-preserving integer image (key) of the
// doubles.  One workgroup per row, and per array where both percentiles are wanted (blockIdx.y).
// A pass counts the keys of the current interval [lo, hi], which holds the k-th, in 2,046 equal bins above a point a, one
// for what is below a and one for what is above the last; the bin with the k-th is the next interval.  The first pass
// over a long row takes a and the bins' width from a sample of 1,024 elements: the latencies of a replay spread over a few
// powers of two, so bins of fixed digits would send nearly all of them to a handful of LDS words, and the atomics on one
// word run one after the other.  Intervals with few enough keys are gathered into LDS and narrowed there, the last 64 by
// counting.  A row is so read twice and sampled once.
constexpr int SEL_THREADS = 1024;
constexpr int SEL_BINS = 2 * SEL_THREADS;
constexpr int SEL_GATHER = 4096;      // keys that are narrowed further in LDS
constexpr int SEL_FEW = WAVE;         // keys that are finished by counting
constexpr int SEL_LOADS = 8;          // loads in flight per thread

__device__ __forceinline__ uint64_t ordered_bits(double x) {
    uint64_t b = (uint64_t)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__global__ void __launch_bounds__(SEL_THREADS) select_kth(const double* x0, const double* x1, int64_t N, int64_t kth /*1-based*/,
                                                          double* out0, double* out1) {
    __shared__ uint32_t hist[SEL_BINS];
    __shared__ uint64_t cand[SEL_GATHER];
    __shared__ uint64_t few[SEL_FEW];
    __shared__ unsigned long long s_lo, s_hi;
    __shared__ uint32_t part[SEL_THREADS / WAVE];
    __shared__ uint32_t s_k, s_m, s_n;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const double* const row = (blockIdx.y ? x1 : x0) + (size_t)blockIdx.x * N;
    double* const out = (blockIdx.y ? out1 : out0) + blockIdx.x;
    if (N <= 0) {
        if (tid == 0) *out = 0.0;
        return;
    }
    // f(key) for every element of the row
    auto each = [&](auto f) {
        for (int64_t i0 = tid; i0 < N; i0 += (int64_t)SEL_LOADS * SEL_THREADS) {
            uint64_t v[SEL_LOADS];
#pragma unroll
            for (int u = 0; u < SEL_LOADS; ++u) {
                const int64_t i = i0 + (int64_t)u * SEL_THREADS;
                v[u] = ordered_bits(row[i < N ? i : N - 1]);
            }
#pragma unroll
            for (int u = 0; u < SEL_LOADS; ++u)
                if (i0 + (int64_t)u * SEL_THREADS < N) f(v[u]);
        }
    };
    if (tid == 0) {
        s_lo = ~0ull;
        s_hi = 0;
        s_n = 0;
    }
    hist[2 * tid] = hist[2 * tid + 1] = 0;
    __syncthreads();
    // the whole of a short row in LDS, a sample of a long one; either's smallest and largest key
    bool in_lds = N <= SEL_GATHER;
    uint32_t n = in_lds ? (uint32_t)N : 0;           // keys in LDS
    unsigned long long least = ~0ull, most = 0;
    if (in_lds) {
        for (int i = tid; i < (int)N; i += SEL_THREADS) {
            const uint64_t v = ordered_bits(row[i]);
            cand[i] = v;
            least = v < least ? v : least;
            most = v > most ? v : most;
        }
    } else {
        least = most = ordered_bits(row[(int64_t)tid * N / SEL_THREADS]);
    }
    for (int d = 1; d < WAVE; d *= 2) {
        const unsigned long long a = __shfl_xor(least, d), b = __shfl_xor(most, d);
        least = a < least ? a : least;
        most = b > most ? b : most;
    }
    if (lane == 0) {
        atomicMin(&s_lo, least);
        atomicMax(&s_hi, most);
    }
    __syncthreads();
    unsigned long long lo = s_lo, hi = s_hi;         // the interval; where the bins start and their width (log2)
    unsigned long long a = lo;
    auto width = [](unsigned long long range) {      // the least with range >> width <= SEL_BINS - 2
        int s = range < SEL_BINS - 1 ? 0 : 64 - __clzll(range) - 11;
        return (range >> s) > SEL_BINS - 2 ? s + 1 : s;
    };
    int shift = width(hi - lo);
    if (!in_lds) {
        lo = 0;
        hi = ~0ull;
    }
    uint32_t m = (uint32_t)N;                        // keys in the interval
    int64_t k = kth;
    unsigned long long answer = lo;
    for (;;) {
        if (lo == hi) {
            answer = lo;
            break;
        }
        if (in_lds && m <= (uint32_t)SEL_FEW) {
            // the one with fewer than k below it and at least k not above it
            for (uint32_t c = tid; c < n; c += SEL_THREADS) {
                const uint64_t v = cand[c];
                if (v >= lo && v <= hi) few[atomicAdd(&s_n, 1u)] = v;
            }
            __syncthreads();
            if (tid < (int)m) {
                const uint64_t mine = few[tid];
                int64_t less = 0, leq = 0;
                for (uint32_t j = 0; j < m; ++j) {
                    less += few[j] < mine ? 1 : 0;
                    leq += few[j] <= mine ? 1 : 0;
                }
                if (less < k && k <= leq) s_lo = mine;               // (every such key has the same value)
            }
            __syncthreads();
            answer = s_lo;
            break;
        }
        if (!in_lds && m <= (uint32_t)SEL_GATHER) {
            each([&](uint64_t v) {
                if (v >= lo && v <= hi) cand[atomicAdd(&s_n, 1u)] = v;
            });
            __syncthreads();
            n = m;
            in_lds = true;
            if (tid == 0) s_n = 0;
            __syncthreads();
            continue;
        }
        auto count = [&](uint64_t v) {
            if (v < lo || v > hi) return;
            const unsigned long long b = v < a ? 0 : 1 + ((v - a) >> shift);
            atomicAdd(&hist[b < SEL_BINS - 1 ? b : SEL_BINS - 1], 1u);
        };
        if (in_lds) {
            for (uint32_t c = tid; c < n; c += SEL_THREADS) count(cand[c]);
        } else {
            each(count);
        }
        __syncthreads();
        // the bin that holds the k-th: sums up to each bin (two per thread), within the wavefront and over wavefronts
        const uint32_t h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
        hist[2 * tid] = hist[2 * tid + 1] = 0;
        uint32_t incl = h0 + h1;
        for (int d = 1; d < WAVE; d *= 2) {
            const uint32_t below = __shfl_up(incl, d);
            incl += lane >= d ? below : 0;
        }
        if (lane == WAVE - 1) part[wave] = incl;
        __syncthreads();
        for (int w = 0; w < wave; ++w) incl += part[w];
        const int64_t before = (int64_t)incl - h0 - h1;
        if (before < k && k <= (int64_t)incl) {
            const bool first = k <= before + h0;
            const unsigned long long b = 2 * tid + (first ? 0 : 1);
            s_k = (uint32_t)(k - before - (first ? 0 : h0));
            s_m = first ? h0 : h1;
            if (b == 0) {
                s_lo = lo;
                s_hi = a - 1;
            } else {
                const unsigned long long from = a + ((b - 1) << shift), span = (1ull << shift) - 1;
                s_lo = from;
                s_hi = b == SEL_BINS - 1 || hi - from < span ? hi : from + span;
            }
        }
        __syncthreads();
        lo = a = s_lo;
        hi = s_hi;
        k = s_k;
        m = s_m;
        shift = width(hi - lo);
        __syncthreads();
    }
    if (tid == 0) {
        const uint64_t b = (answer >> 63) ? (answer & 0x7FFFFFFFFFFFFFFFull) : ~answer;
        *out = __longlong_as_double((long long)b);
    }
}

int hip_fail(hipError_t e, const char* what) {
    return fail(GORGO_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// HIP events bracketing the kernels of the most recent evaluation on this thread (for measurement).
struct Marks {
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};   // before fill, before replay, after replay, after select
    int device = -1;
    bool valid = false;
};
thread_local Marks g_marks;

bool marks_ready() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (g_marks.device == dev) return true;
    for (auto& e : g_marks.ev)
        if (hipEventCreate(&e) != hipSuccess) return false;
    g_marks.device = dev;
    return true;
}

thread_local bool g_marks_on = true;      // off for the evaluation that must not create or record events

void mark(int i, hipStream_t s) {
    if (g_marks_on && g_marks.device >= 0) (void)hipEventRecord(g_marks.ev[i], s);
}

// Device memory for the entry point that allocates nothing: one array per GPU, there from the moment the library
// is loaded until the process ends.  Host code only ever uses its device address, looked up once per device.
static __device__ __align__(256) unsigned char scratch[GORGO_STATIC_SCRATCH_BYTES];

}  // namespace

constexpr size_t UPLOAD_AT_ONCE = (size_t)256 << 10;

int upload_trace(const gorgo_trace* tc) {
    gorgo_trace* t = const_cast<gorgo_trace*>(tc);
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (t->dev.base && t->dev.device == dev) return GORGO_OK;
    if (t->dev.base) release_device_trace(t);
    const size_t N = (size_t)t->N, T = (size_t)t->total_blocks;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t o_ts = 0;
    const size_t o_off = o_ts + up(N * 8);
    const size_t o_il = o_off + up((N + 1) * 8);
    const size_t o_ol = o_il + up(N * 4);
    const size_t o_key = o_ol + up(N * 4);
    const size_t o_first = o_key + up(T * 4);
    const size_t n_sr = t->seg.size();
    const size_t o_soff = o_first + up(T);
    const size_t o_seg = o_soff + up(t->seg_off.size() * 8);
    const size_t o_fh = o_seg + up(n_sr * sizeof(SegRef));
    const size_t o_row = o_fh + up(N * 4);
    const size_t o_prev = o_row + up(t->row_ref.size() * 4);
    const size_t total = o_prev + up(t->seg_prev.size() * 4) + 256;
    char* base = nullptr;
    e = hipMalloc(reinterpret_cast<void**>(&base), total);
    if (e != hipSuccess) return fail(GORGO_ERR_OOM, std::string("hipMalloc(trace): ") + hipGetErrorString(e));
    // (a copy of its own takes some 10 us however small: a small trace is put together on the host and copied once; ten
    // requests, first evaluation: 226 us with eleven copies, 120 so)
    std::unique_ptr<char[]> small(total <= UPLOAD_AT_ONCE ? new (std::nothrow) char[total]() : nullptr);
    auto put = [&](size_t o, const void* src, size_t bytes) {
        if (bytes == 0) return hipSuccess;
        if (!small) return hipMemcpy(base + o, src, bytes, hipMemcpyHostToDevice);
        std::memcpy(small.get() + o, src, bytes);
        return hipSuccess;
    };
    if ((e = put(o_ts, t->ts.data(), N * 8)) != hipSuccess || (e = put(o_off, t->blk_off.data(), (N + 1) * 8)) != hipSuccess ||
        (e = put(o_il, t->in_len.data(), N * 4)) != hipSuccess || (e = put(o_ol, t->out_len.data(), N * 4)) != hipSuccess ||
        (e = put(o_key, t->key.data(), T * 4)) != hipSuccess || (e = put(o_first, t->first.data(), T)) != hipSuccess ||
        (e = put(o_soff, t->seg_off.data(), t->seg_off.size() * 8)) != hipSuccess ||
        (e = put(o_seg, t->seg.data(), n_sr * sizeof(SegRef))) != hipSuccess ||
        (e = put(o_fh, t->first_hash.data(), N * 4)) != hipSuccess ||
        (e = put(o_row, t->row_ref.data(), t->row_ref.size() * 4)) != hipSuccess ||
        (e = put(o_prev, t->seg_prev.data(), t->seg_prev.size() * 4)) != hipSuccess ||
        (small && (e = hipMemcpy(base, small.get(), total, hipMemcpyHostToDevice)) != hipSuccess)) {
        (void)hipFree(base);
        return hip_fail(e, "hipMemcpy(trace)");
    }
    t->dev.device = dev;
    t->dev.base = base;
    t->dev.ts = reinterpret_cast<const int64_t*>(base + o_ts);
    t->dev.blk_off = reinterpret_cast<const int64_t*>(base + o_off);
    t->dev.in_len = reinterpret_cast<const int32_t*>(base + o_il);
    t->dev.out_len = reinterpret_cast<const int32_t*>(base + o_ol);
    t->dev.key = reinterpret_cast<const uint32_t*>(base + o_key);
    t->dev.first = reinterpret_cast<const uint8_t*>(base + o_first);
    t->dev.seg_off = reinterpret_cast<const int64_t*>(base + o_soff);
    t->dev.seg = reinterpret_cast<const SegRef*>(base + o_seg);
    t->dev.first_hash = reinterpret_cast<const uint32_t*>(base + o_fh);
    t->dev.row_ref = reinterpret_cast<const uint32_t*>(base + o_row);
    t->dev.seg_prev = reinterpret_cast<const int32_t*>(base + o_prev);
    return GORGO_OK;
}

void release_device_trace(gorgo_trace* t) {
    if (t->dev.base) (void)hipFree(t->dev.base);
    t->dev = DeviceTrace();
}

int copy_small_to_device(void* dst, const void* src, size_t bytes, void* stream) {
    hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? GORGO_OK : hip_fail(e, "hipMemcpyAsync(H2D)");
}

// Whether a launch of fixed-weight replays runs two replays per workgroup.  A replay is a serial chain whose duration
// hardly depends on how many others run beside it, and a packed pair takes about a third longer per request than a
// lone replay (0.79 us against 0.60, 40,000 requests, 32 replicas, the chip full of either): packing pays when the replays
// would not all be resident at once otherwise.
bool pack_replays(const Plan& pl, int64_t rows) {
    const int32_t mode = pl.packing;       // 0 never, 1 whenever the shape allows, 2 when the replays would not all be resident
    if (mode == 0 || pl.R > HALF || pl.B > 16 || pl.P % 2 != 0 ||
        2ull * (uint64_t)rows * (uint64_t)pl.R * 4u >= (1ull << 32))
        return false;
    if (mode == 1) return true;
    int device = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&device) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, replay_segments_kernel<MODE_COST_MODEL, false, false>,
                                                     seg_threads<1>(), replay_queue_lds_bytes(pl.R, pl.B, false, 0)) != hipSuccess)
        return false;
    // (10,000 requests, 32 replicas of 8 slots, unpacked against packed: 1,280 replays 7.2 / 7.2 ms, 1,282 12.5 / 7.2, 1,536
    // 12.3 / 7.2, 2,048 13.6 / 8.2; where the pairs take two rounds as well: 2,050 13.6 / 14.0, 2,304 14.7 / 13.8, 2,560
    // 14.9 / 14.0.  16 slots, where 1,024 replays are resident either way: 1,026 13.0 / 13.6, 1,536 14.1 / 14.1, 2,048
    // 15.0 / 14.2.  The upper end is what the option says, not where packing stops being the faster: 3,072 20.0 / 15.7,
    // 4,096 26.3 / 21.8, 8,192 47.9 / 37.7.)
    const int64_t resident = (int64_t)cus * per_cu;
    return (int64_t)pl.P > resident && (int64_t)pl.P <= 2 * resident;
}

int wait_for_copies(void* stream) {
    hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    return e == hipSuccess ? GORGO_OK : hip_fail(e, "hipStreamSynchronize");
}

int copy_small_to_host_sync(void* dst, const void* src, size_t bytes, void* stream) {
    hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(D2H)");
    e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
    return e == hipSuccess ? GORGO_OK : hip_fail(e, "hipStreamSynchronize");
}

namespace {

// The proxy's smoothed round trip times (Sec. 2.2: an exponentially weighted moving average of pings), one
// thread per replica: est[0] = x[0], est[e] = alpha x[e] + (1 - alpha) est[e-1], each product and sum rounded
// on its own.
__global__ void smooth_rtt(const double* x, double* est, int epochs, int R, double alpha) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= R) return;
    double prev = x[i];
    est[i] = prev;
    for (int e = 1; e < epochs; ++e) {
        const double fresh = alpha * x[(size_t)e * R + i];
        const double kept = (1.0 - alpha) * prev;
        prev = fresh + kept;
        est[(size_t)e * R + i] = prev;
    }
}

}  // namespace

int static_scratch(void** ptr, size_t* bytes) {
    static std::mutex mu;
    static void* address[64] = {};        // per device: each GPU holds its own copy of the array at its own address
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= 64) return fail(GORGO_ERR_DEVICE, "device index out of range");
    std::lock_guard<std::mutex> lock(mu);
    if (!address[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        address[dev] = p;
    }
    *ptr = address[dev];
    *bytes = sizeof(scratch);
    return GORGO_OK;
}

bool trace_is_resident(const gorgo_trace* t) {
    int dev = 0;
    return hipGetDevice(&dev) == hipSuccess && t->dev.base && t->dev.device == dev;
}

void set_event_marks(bool on) { g_marks_on = on; }

namespace {

// The small inputs on their way to the device, and the never-cached rows filled.  A stream under capture keeps the copies:
// a graph reads the caller's arrays again at every replay.
// (a replay laid out by replica has its rows replica by replica)
int prepare(const Plan& pl, double* d_small, int32_t* last, int64_t rows, hipStream_t s) {
    const size_t R = (size_t)pl.R, P = (size_t)pl.P, count = R + 4 * P;
    SmallInputs in;
    bool as_arguments = count <= (size_t)SMALL_INPUTS;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (as_arguments && (hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone)) {
        (void)hipGetLastError();
        as_arguments = false;
    }
    int rc;
    if (as_arguments) {
        std::memcpy(in.v, pl.h_rtt, R * sizeof(double));
        std::memcpy(in.v + R, pl.h_params, 3 * P * sizeof(double));
        std::memcpy(in.v + R + 3 * P, pl.h_scale, P * sizeof(double));
    } else {
        if ((rc = copy_small_to_device(d_small, pl.h_rtt, R * sizeof(double), s))) return rc;
        if ((rc = copy_small_to_device(d_small + R, pl.h_params, 3 * P * sizeof(double), s))) return rc;
        if ((rc = copy_small_to_device(d_small + R + 3 * P, pl.h_scale, P * sizeof(double), s))) return rc;
        if (pl.keep_copies && (rc = wait_for_copies(s))) return rc;
    }
    const size_t threads = std::max(as_arguments ? count : 0, last ? P * R : 0);
    if (threads == 0) return GORGO_OK;
    hipLaunchKernelGGL(prepare_replays, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, in, as_arguments ? (int)count : 0,
                       d_small, last, pl.each ? pl.P * pl.R : pl.P, rows, pl.each ? 1 : pl.R, NEVER_CACHED);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? GORGO_OK : hip_fail(e, "launch prepare_replays");
}

// Whether a launch of segment rows spreads each replay over six wavefronts instead of four: up to two replays for each of
// the 256 CUs, with few replicas up to three.  A replay's chain is then a tenth to a third shorter; with more replays per CU the
// quarter more vector instructions a request takes is what counts.  (10,000 requests, four / six wavefronts, ms.  Two replays on 2
// replicas: 7.8 / 5.3.  19, caches of 8,000 blocks: 3 replicas 7.3 / 5.3, 16 5.9 / 5.0, 32 5.6 / 4.8, 48 5.9 / 5.3, 64 5.4 / 5.0; of
// 700 blocks 7.5 / 5.8, 6.2 / 5.9, 6.0 / 5.7, 6.2 / 6.1, 5.9 / 6.0.  512, of 8,000: 7.9 / 5.8, 6.6 / 5.6, 6.0 / 5.4, 6.4 / 6.2, 6.0 /
// 5.7; of 700 8.2 / 6.4, 6.8 / 6.5, 6.3 / 6.2, 6.7 / 6.9, 6.3 / 6.6.  768: 2 replicas 8.4 / 6.5, 8 7.5 / 6.7, 12 7.6 / 6.9, proxy 10.9 /
// 10.6, engine model 10.3 / 8.2, tuner 8.6 / 7.4; 16 6.5 / 6.4, proxy 8.6 / 9.8, caches of 700 blocks 6.8 / 7.9; 20 6.3 / 6.7, 32 6.0 /
// 6.4.)  And only where all of them are resident: by their LDS, `lds` bytes of it for the service slots (with 1,024 slots or long
// tuner windows fewer fit a CU), and by their registers, `held` workgroups.  That is half of the wavefronts that fit a SIMD,
// for a workgroup of six takes the room of two on each: three up to 80 registers, two up to 128.  (The time doubles from 768
// replays to 769, 2 replicas 6.5 / 11.6 ms, 32 6.0 / 10.6, and not where the kernel is kept to 64 registers; proxy, engine model
// and tuner together take 85, 3,000 requests on 8 replicas: 512 replays 3.0 ms, 640 5.9, with four wavefronts 4.8.)
// Nor, with fixed weights or session affinity and the linear model, where the cache of one of 24 replicas or more holds about as few
// requests as the look-ahead has records, `least` of them: the deciding wavefront then waits for the evicting one at
// nearly every request.  (6,000 requests of 62 blocks, 300 replays.  48 replicas of 600 blocks 4.00 / 4.17, 800 3.97 / 4.01, 1,000 3.93
// / 3.92, 1,600 3.89 / 3.79; 64 3.99 / 4.18, -, 3.93 / 3.89, 3.90 / 3.77; of 11 blocks, 48 replicas of 60 4.17 / 4.37, 100 4.10 / 4.18, 150 4.04
// / 3.99.  Affinity, 48 of 600 3.88 / 4.09, 1,000 3.81 / 3.85, 1,600 3.77 / 3.75.  32 of 250 3.97 / 4.23, 450 3.85 / 3.95, 600 3.78 / 3.81,
// 750 3.73 / 3.68, affinity 3.89 / 4.19, 3.69 / 3.87, 3.64 / 3.72, 3.59 / 3.60; 24 4.05 / 4.22, 3.90 / 3.99, 3.84 / 3.84, 3.80 / 3.73, affinity 3.96 /
// 4.20, 3.77 / 3.91, 3.72 / 3.79, 3.67 / 3.66; 16 of 250 4.31 / 4.22, affinity 4.33 / 4.28.
// Least-request, random, tuner, engine and proxy, 48 and 64 of 600: six are the faster by 3 to 15 %.)
constexpr int SPREAD_UP_TO = 512, SPREAD_FEW_REPLICAS = 12, SPREAD_FEW_UP_TO = 768;
constexpr int SPREAD_WAITS_FROM = 24;       // replicas
double spread_least_held(const Plan& pl, bool affinity) {
    return pl.R < SPREAD_WAITS_FROM ? 0.0 : pl.R <= HALF ? (affinity ? 12.0 : 10.0) : affinity ? 20.0 : 15.0;
}
int spread_up_to(const Plan& pl, int held) { return std::min(pl.R <= SPREAD_FEW_REPLICAS ? SPREAD_FEW_UP_TO : SPREAD_UP_TO, 256 * held); }
bool spread_replays(const Plan& pl, bool proxy, size_t lds, int held, double least) {
    if (pl.P > spread_up_to(pl, held) || pl.requests_held < least) return false;
    const size_t fixed = proxy ? sizeof(ApartHandover<true>) : sizeof(ApartHandover<false>);
    const size_t per_cu = (size_t)160 * 1024 / ((fixed + lds + 1279) / 1280 * 1280);        // (given out in pieces of 1,280 bytes)
    return pl.P <= 256 * (int)per_cu;
}

// Whether the pairs of a launch, eight wavefronts each, are all resident: two workgroups for each of the 256 CUs, fewer where their
// service slots' LDS, `lds` bytes of a pair, does not leave the room.  (By registers four wavefronts fit a SIMD up to 128.)
bool pairs_resident(const Plan& pl, bool proxy, size_t lds, int64_t rows) {
    if (pl.packing == 0 || pl.R > HALF || 2ull * (uint64_t)rows * (uint64_t)pl.R * 4u >= (1ull << 32)) return false;
    const size_t fixed = proxy ? sizeof(ApartHandover<true, 2>) : sizeof(ApartHandover<false, 2>);
    const size_t per_cu = (size_t)160 * 1024 / ((fixed + lds + 1279) / 1280 * 1280);
    return (pl.P + 1) / 2 <= 256 * std::min((int)per_cu, 2);
}
// Whether they take the launch: it has too many replays for six wavefronts each, and the caches hold enough requests, for two replays
// wait twice as often for the evicting wavefront (PAIR_HELD); or it has more than one for each CU in the variants whose serving or
// deciding wavefront has so much to do that it does better alone on its SIMD, and the caches hold more still.  How often that
// wait comes depends on the trace: the lines are where pairs gain on the mean and lose no more than some five per cent on any
// one (proxy of any index, 16 replicas, 288 replays, 45 held 0.94 to 1.06; 2 replicas, an index that never forgets, 10 held 0.96 to 1.06).
// (us per request.  1,000 replays, four wavefronts each / pairs of eight, users by Zipf's law, caches of 8,000 blocks, 130 requests: 2 replicas 0.844 / 0.671,
// tuner 0.955 / 0.727, engine model 1.075 / 0.867, proxy 1.338 / 0.988; 16 0.676 / 0.607, 0.787 / 0.676, 0.940 / 0.796, 0.862 / 0.787; 32
// 0.606 / 0.574, 0.709 / 0.647, 0.806 / 0.690, 0.739 / 0.684; 513, 600, 768 and 900 replays on 32 0.577 / 0.502, 0.579 / 0.516, 0.574 / 0.516, 0.584 / 0.515.
// How many times as long four wavefronts take as pairs, by requests held, least / mean / most of five traces of 4,000 requests, four of
// them with users drawn evenly, 767 replays (1,023 on 12 replicas).  Fixed weights, 12 replicas: 9 0.98 / 1.00 / 1.02, 12 1.00 / 1.02 / 1.06; 16: 9 0.92 / 0.98 / 1.03,
// 15 0.96 / 1.02 / 1.08, 18 1.00 / 1.05 / 1.09; 32: 12 0.90 / 0.92 / 1.00, 18 0.98 / 1.00 / 1.04, 22 1.01 / 1.03 / 1.05.  Tuner, 16: 9 0.95 / 0.97 / 1.02, 15 1.00 / 1.02 /
// 1.10; 32: 9 0.87 / 0.90 / 0.98, 18 1.00 / 1.02 / 1.07.  Engine model, 24: 6 0.98 / 1.07 / 1.16; 28: 6 0.98 / 1.07 / 1.14 and on other traces from 0.95, 9 1.02 / 1.11 / 1.17; 32: 6 0.91 / 0.96 / 1.01, 12 0.99 / 1.04 / 1.09; with a tuner, 32: 6 0.98 / 1.01 /
// 1.06.  Proxy, 12: 9 0.97 / 0.99 / 1.04, 12 0.97 / 1.02 / 1.09; 16: 12 0.95 / 0.99 / 1.04, 15 0.97 / 1.03 / 1.07; 24: 15 0.93 / 0.99 / 1.05, 22 0.98 / 1.04 / 1.11; with a
// tuner, 16: 9 0.95 / 0.99 / 1.09, 12 1.00 / 1.03 / 1.12; with the engine model, 16: 9 1.03 / 1.09 / 1.13, 32: 9 0.94 / 0.98 / 1.03, 18 1.06 / 1.10 / 1.13.
// Least-request, 32: 6 1.09 / 1.09 / 1.10.
// Six wavefronts and pairs, the same.  Engine model, 24 replicas: 257 replays, 40 held 0.94 / 0.99 / 1.05; 288, 30 0.96 / 1.00 / 1.03; 320, 20 0.99 / 1.02 / 1.04, 30 1.02 /
// 1.04 / 1.07.  Proxy, 16: 257, 60 0.95 / 0.96 / 0.97; 288, 40 1.00 / 1.02 / 1.04; 401, 30 0.95 / 0.98 / 1.02, 40 0.96 / 1.00 / 1.04, 60 1.00 / 1.03 / 1.05; 32: 288, 20 0.94 / 0.98 / 1.02,
// 40 1.03 / 1.06 / 1.08.  Tuner and engine model, 16 and 32, unbounded: 320 0.97 / 0.98 / 0.99, 0.98 / 1.00 / 1.02, 511 0.96 / 0.97 / 0.98, 0.98 / 0.99 / 1.01.  Proxy and engine
// model, 16: 511, 60 0.97 / 0.98 / 0.99; 24: 320, 60 1.00 / 1.03 / 1.04 and on other traces from 0.96, 401, 40 0.98 / 0.99 / 1.01, 60 0.99 / 1.02 / 1.03; with a tuner, 24: 320, 20 0.96 /
// 0.98 / 1.01, 40 1.01 / 1.03 / 1.06.  Least-request and engine model, 24: 257 0.97 / 1.00 / 1.02, 288 1.06 / 1.07 / 1.08.
// Proxy, engine model and tuner together, of which 512 are resident with six wavefronts each; four each / pairs, 513 and 768 replays on 4
// replicas of 8,000 blocks 1.507 / 1.010 and 1.521 / 1.050, on 12 1.449 / 1.002 and 1.442 / 1.028; 768 on 12 of 800 blocks 1.535 / 1.147.)
constexpr double PAIR_HELD[][6] = {       // requests; up to 8, 12, 16, 24, 28 and 32 replicas
    {9, 12, 16, 18, 18, 20},              // fixed weights
    {8, 8, 14, 17, 18, 18},               // tuner
    {6, 6, 6, 6, 9, 10},                  // engine model
    {6, 6, 6, 6, 6, 6},                   // ... and tuner
    {10, 12, 15, 20, 18, 21},             // proxy
    {10, 10, 11, 20, 20, 20},             // ... and tuner
    {10, 10, 10, 20, 20, 20},             // ... and engine model
    {10, 10, 10, 20, 20, 20},             // all three
    {9, 9, 9, 12, 12, 12},                // least-request
    {6, 6, 6, 6, 6, 6}};                  // ... and engine model
bool pair_replays(const Plan& pl, int mode, bool engine, bool proxy, int held) {
    if (pl.packing == 1) return true;
    const bool tuner = mode == MODE_ONLINE, least_request = mode == MODE_LEAST_REQUEST, few = pl.R < 24;       // replicas
    if (pl.P > spread_up_to(pl, held)) {
        const int row = least_request ? (engine ? 9 : 8) : (proxy ? 4 : 0) + (engine ? 2 : 0) + (tuner ? 1 : 0);
        return pl.requests_held >= PAIR_HELD[row][pl.R <= 8 ? 0 : pl.R <= 12 ? 1 : pl.R <= 16 ? 2 : pl.R <= 24 ? 3 : pl.R <= 28 ? 4 : 5];
    }
    if (pl.P < 288 || pl.R < 16) return false;
    if (proxy && engine && !tuner) return pl.P >= 400 && !few && pl.requests_held >= 60.0;
    if (proxy) return pl.requests_held >= (few && !engine ? 45.0 : 35.0);
    return engine && !tuner && pl.requests_held >= (least_request ? 12.0 : 30.0);
}

// Which of the segment-row kernels takes a launch, `window` the tuner's.  (The answer is the launch's, gorgo_query_replay_workgroups'
// and, for want of a timed instantiation of the packed one, nearly the section timing's.)
enum SegmentKernel { FOUR_WAVEFRONTS, SIX_WAVEFRONTS, PAIRS, PACKED };
SegmentKernel segment_kernel(const Plan& pl, int mode, bool engine, bool proxy, int32_t window) {
    const int64_t rows = pl.nseg + 2;
    const size_t lds = replay_queue_lds_bytes(pl.R, pl.B, engine, mode == MODE_ONLINE ? window : 0);
    if (mode == MODE_COST_MODEL && !engine && !proxy && pack_replays(pl, rows)) return PACKED;
    const int held = mode == MODE_ONLINE && engine && proxy ? 2 : 3;         // workgroups of six wavefronts, of a CU's registers
    if ((mode == MODE_COST_MODEL || mode == MODE_ONLINE || mode == MODE_LEAST_REQUEST) && pairs_resident(pl, proxy, 2 * lds, rows) &&
        pair_replays(pl, mode, engine, proxy, held))
        return PAIRS;
    const bool waits = (mode == MODE_COST_MODEL || mode == MODE_AFFINITY) && !engine && !proxy;
    const double least = waits ? spread_least_held(pl, mode == MODE_AFFINITY) : 0.0;
    return spread_replays(pl, proxy, lds, held, least) ? SIX_WAVEFRONTS : FOUR_WAVEFRONTS;
}

int mode_of(int32_t policy, bool online) {
    return online ? MODE_ONLINE
                  : policy == 0 ? MODE_COST_MODEL : policy == 1 ? MODE_LEAST_REQUEST : policy == 2 ? MODE_AFFINITY : MODE_RANDOM;
}

// The segment-row kernels' instantiations: every mode with either replica model; imperfect proxy knowledge concerns the
// cost model (fixed weights or tuned online) only.
template <int MODE>
void launch_segments(SegmentKernel kernel, bool engine, bool proxy, const Plan& pl, hipStream_t s, const SegArgs& a) {
    const size_t lds = replay_queue_lds_bytes(pl.R, pl.B, engine, a.window);
    const dim3 grid((unsigned)pl.P);
    if (kernel == SIX_WAVEFRONTS) {
        const dim3 block(APART_WAVES * WAVE);
        if constexpr (MODE == MODE_COST_MODEL || MODE == MODE_ONLINE) {
            if (proxy) {
                if (engine) hipLaunchKernelGGL((replay_apart_kernel<MODE, true, true>), grid, block, lds, s, a);
                else hipLaunchKernelGGL((replay_apart_kernel<MODE, false, true>), grid, block, lds, s, a);
                return;
            }
        }
        if (engine) hipLaunchKernelGGL((replay_apart_kernel<MODE, true, false>), grid, block, lds, s, a);
        else hipLaunchKernelGGL((replay_apart_kernel<MODE, false, false>), grid, block, lds, s, a);
        return;
    }
    if constexpr (MODE == MODE_COST_MODEL || MODE == MODE_ONLINE || MODE == MODE_LEAST_REQUEST) {
        if (kernel == PAIRS) {
            const dim3 grid2((unsigned)((pl.P + 1) / 2)), block(apart_threads<2>());
            if constexpr (MODE != MODE_LEAST_REQUEST) {
                if (proxy) {
                    if (engine) hipLaunchKernelGGL((replay_apart_pairs_kernel<MODE, true, true>), grid2, block, 2 * lds, s, a);
                    else hipLaunchKernelGGL((replay_apart_pairs_kernel<MODE, false, true>), grid2, block, 2 * lds, s, a);
                    return;
                }
            }
            if (engine) hipLaunchKernelGGL((replay_apart_pairs_kernel<MODE, true, false>), grid2, block, 2 * lds, s, a);
            else hipLaunchKernelGGL((replay_apart_pairs_kernel<MODE, false, false>), grid2, block, 2 * lds, s, a);
            return;
        }
    }
    const dim3 block(seg_threads<1>());
    if constexpr (MODE == MODE_COST_MODEL || MODE == MODE_ONLINE) {
        if (proxy) {
            if (engine) hipLaunchKernelGGL((replay_segments_kernel<MODE, true, true>), grid, block, lds, s, a);
            else hipLaunchKernelGGL((replay_segments_kernel<MODE, false, true>), grid, block, lds, s, a);
            return;
        }
    }
    if (engine) hipLaunchKernelGGL((replay_segments_kernel<MODE, true, false>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((replay_segments_kernel<MODE, false, false>), grid, block, lds, s, a);
}

// Log records of look-ahead per replica with six and eight wavefronts, of the fifteen there is room for.  The deciding wavefront waits for the
// evicting one when it matches blocks of a record in the look-ahead, so a long one is waited for often where a cache holds few
// requests, and a short one runs dry.  (us per request, 64 replays on 32 replicas, 5 / 6 / 8 / 11 / 15 records.  Caches of 700 blocks, 11
// requests: 0.522 / 0.520 / 0.531 / 0.554 / 0.586, proxy 0.769 / 0.745 / 0.741 / 0.759 / 0.794; 1,500: 0.493 / 0.490 / 0.491 / 0.497 /
// 0.510, proxy 0.752 / 0.730 / 0.706 / 0.706 / 0.715; 3,000, 48 requests: 0.480 / 0.484 / 0.486 / 0.483 / 0.487, proxy 0.712 / 0.685 /
// 0.672 / 0.668 / 0.670.  Three replicas, 700: 0.583 / 0.579 / 0.580 / 0.582 / 0.587; 3,000: 0.554 / 0.547 / 0.542 / 0.539 / 0.537.
// Pairs wait for two replays and have the same line.  1,000 replays of 4,000 requests on 3 to 32 replicas, means of three traces, 64 alike: eleven records from
// 15 requests held on instead of 40, 16 held up to 6 % slower, 25 up to 3 %, 35 from 1.4 % slower (tuner, 16 replicas) to 1.4 % faster (fixed weights, 32); from
// 100 on, 60 and 90 held up to 2 % slower.)
constexpr double LOOK_FEW_HELD = 40.0;       // requests
int32_t apart_look(const Plan& pl, bool proxy) { return pl.requests_held < LOOK_FEW_HELD ? (proxy ? 8 : 6) : 11; }
static_assert(APART_LOOK > 11);
// From when on: the longest requests that there is still room for.  (The same launches.  One request instead of four: 16 held up to 4 %
// faster, 100 held up to 1.5 % slower, else within 1.3 %.  Sixteen: 1,000 requests into caches of 25 up to 19 % slower, 4,000 into caches of 60 up to 6 %.)
constexpr int LOOK_FROM = 4;

// Dictated routes: the shares laid out, a replay per share, the outputs back in their order.
int launch_each(const gorgo_trace* t, const Plan& pl, int mode, bool engine, const SegArgs& a, char* ws, hipStream_t s) {
    const size_t P = (size_t)pl.P, N = (size_t)pl.N, R = (size_t)pl.R;
    const EachSpace at(P, N, t->seg.size(), R);
    char* const base = ws + pl.off_each;
    EachArgs e;
    e.ts = a.ts;
    e.seg_off = a.seg_off;
    e.blk_off = a.blk_off;
    e.in_len = a.in_len;
    e.out_len = a.out_len;
    e.seg = a.seg;
    e.seg_prev = t->dev.seg_prev;
    e.first_hash = a.first_hash;
    e.seeds = a.seeds;
    e.N = pl.N;
    e.T = (int64_t)t->seg.size();
    e.R = pl.R;
    e.chunks = (int32_t)((N + EACH_CHUNK - 1) / EACH_CHUNK);
    e.where = reinterpret_cast<uint8_t*>(base + at.where);
    e.count = reinterpret_cast<EachCount*>(base + at.count);
    e.from = reinterpret_cast<int32_t*>(base + at.from);
    e.list = reinterpret_cast<int32_t*>(base + at.list);
    e.s_ts = reinterpret_cast<int64_t*>(base + at.ts);
    e.s_seg_off = reinterpret_cast<int64_t*>(base + at.seg_off);
    e.s_blk_off = reinterpret_cast<int64_t*>(base + at.blk_off);
    e.s_in = reinterpret_cast<int32_t*>(base + at.in_len);
    e.s_out = reinterpret_cast<int32_t*>(base + at.out_len);
    e.s_seg = reinterpret_cast<SegRef*>(base + at.seg);
    e.hit = a.hit ? reinterpret_cast<uint16_t*>(base + at.hit) : nullptr;
    e.ttft = a.ttft ? reinterpret_cast<double*>(base + at.ttft) : nullptr;
    e.e2e = a.e2e ? reinterpret_cast<double*>(base + at.e2e) : nullptr;
    const dim3 chunks((unsigned)e.chunks, (unsigned)P), threads(EACH_CHUNK);
    if (mode == MODE_AFFINITY) hipLaunchKernelGGL((each_route<MODE_AFFINITY>), chunks, threads, 0, s, e);
    else hipLaunchKernelGGL((each_route<MODE_RANDOM>), chunks, threads, 0, s, e);
    hipLaunchKernelGGL(each_begin, dim3((unsigned)P), dim3(WAVE), 0, s, e);
    hipLaunchKernelGGL(each_place, chunks, threads, 0, s, e);
    const dim3 shares((unsigned)(P * R)), block(APART_WAVES * WAVE);
    const size_t lds = replay_queue_lds_bytes(1, pl.B, engine, 0);
    if (engine) hipLaunchKernelGGL((replay_each_kernel<true>), shares, block, lds, s, a, e);
    else hipLaunchKernelGGL((replay_each_kernel<false>), shares, block, lds, s, a, e);
    hipLaunchKernelGGL(each_return, chunks, threads, 0, s, e, a.route, a.hit, a.ttft, a.e2e);
    const hipError_t rc = hipGetLastError();
    return rc == hipSuccess ? GORGO_OK : hip_fail(rc, "launch replay_each_kernel");
}

// The block formulation over rows of stamps: the same instantiations as the block tables'.
template <int MODE>
void launch_rows(bool engine, bool proxy, dim3 grid, size_t lds, hipStream_t s, const RowArgs& b) {
    const dim3 block(ROW_WAVES * WAVE);
    if constexpr (MODE == MODE_COST_MODEL || MODE == MODE_ONLINE) {
        if (proxy) {
            if (engine) hipLaunchKernelGGL((replay_rows_kernel<MODE, true, true>), grid, block, lds, s, b);
            else hipLaunchKernelGGL((replay_rows_kernel<MODE, false, true>), grid, block, lds, s, b);
            return;
        }
    }
    if (engine) hipLaunchKernelGGL((replay_rows_kernel<MODE, true, false>), grid, block, lds, s, b);
    else hipLaunchKernelGGL((replay_rows_kernel<MODE, false, false>), grid, block, lds, s, b);
}

// The block-table kernel's instantiations: every mode with either replica model; imperfect proxy knowledge concerns
// the cost model (fixed weights or tuned online) only.
template <int MODE>
void launch_blocks(bool engine, bool proxy, dim3 grid, size_t lds, hipStream_t s, const BlockArgs& b) {
    const dim3 block(BLOCK_THREADS);
    if constexpr (MODE == MODE_COST_MODEL || MODE == MODE_ONLINE) {
        if (proxy) {
            if (engine) hipLaunchKernelGGL((replay_blocks_kernel<MODE, true, true>), grid, block, lds, s, b);
            else hipLaunchKernelGGL((replay_blocks_kernel<MODE, false, true>), grid, block, lds, s, b);
            return;
        }
    }
    if (engine) hipLaunchKernelGGL((replay_blocks_kernel<MODE, true, false>), grid, block, lds, s, b);
    else hipLaunchKernelGGL((replay_blocks_kernel<MODE, false, false>), grid, block, lds, s, b);
}

}  // namespace

Workgroups replay_workgroups(const Plan& pl, int32_t policy, int32_t window, bool engine, bool proxy) {
    if (pl.path != PATH_SEGMENTS) return {1, pl.row_slots > 0 ? ROW_WAVES : BLOCK_THREADS / WAVE};
    if (pl.each) return {0, APART_WAVES};
    switch (segment_kernel(pl, mode_of(policy, window > 0), engine, proxy, window)) {
        case SIX_WAVEFRONTS: return {1, apart_threads<1>() / WAVE};
        case PAIRS: return {2, apart_threads<2>() / WAVE};
        case PACKED: return {2, seg_threads<2>() / WAVE};
        default: return {1, seg_threads<1>() / WAVE};
    }
}

int launch_replay(const gorgo_trace* t, const Plan& pl, const double* d_rtt, const double* d_params,
                  const double* d_scale, uint8_t* route, uint16_t* hit, double* ttft, double* e2e,
                  void* workspace, void* stream, const OnlineLaunch* online, const PolicyLaunch* policy,
                  const EngineLaunch* engine, const ProxyLaunch* proxy, unsigned long long* sections) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    int rc;
    g_marks.valid = false;
    if (g_marks_on) marks_ready();
    mark(0, s);
    hipError_t e;
    const bool segments = pl.path == PATH_SEGMENTS;
    // what both formulations' kernels read: the trace's scalars, the model, the weights, the outputs, and what the
    // online tuner, the baseline policies, the engine model and the proxy's knowledge bring
    SegArgs a;
    a.ts = t->dev.ts;
    a.in_len = t->dev.in_len;
    a.out_len = t->dev.out_len;
    a.seg_off = segments ? t->dev.seg_off : nullptr;
    a.seg = segments ? t->dev.seg : nullptr;
    a.blk_off = t->dev.blk_off;
    a.N = pl.N;
    a.P = pl.P;
    a.R = pl.R;
    a.B = pl.B;
    a.C = pl.C;
    a.nseg = pl.nseg + 2;             // rows of one replay: one per segment, one that no request touches, a spare
    a.block_tokens = pl.block_tokens;
    a.look = apart_look(pl, proxy != nullptr);
    a.near = LOOK_FROM * t->max_blocks;              // (at most 2^16 of them)
    a.a_pf = pl.a_pf;
    a.a_dec = pl.a_dec;
    a.least_dec = engine ? engine->least_dec : pl.a_dec;
    a.rtt = d_rtt;
    a.params = d_params;
    a.scale = d_scale;
    a.last = segments ? reinterpret_cast<int32_t*>(ws + pl.off_tables) : nullptr;
    a.log = segments ? reinterpret_cast<LogRec*>(ws + pl.off_spare) : nullptr;
    a.rec = reinterpret_cast<Rec*>(ws + pl.off_rec);
    a.route = route;
    a.hit = hit;
    a.ttft = ttft;
    a.e2e = e2e;
    a.window = online ? online->window : 0;
    a.hop = online ? online->hop : 0;
    a.steps = online ? online->steps : 0;
    a.tuner = online ? online->tuner : nullptr;
    a.ln_theta0 = online ? online->ln_theta0 : nullptr;
    a.z = online ? online->z : nullptr;
    a.theta_step = online ? online->theta_step : nullptr;
    a.fitness_step = online ? online->fitness_step : nullptr;
    a.theta_final = online ? online->theta_final : nullptr;
    a.sigma_final = online ? online->sigma_final : nullptr;
    a.accepted = online ? online->accepted : nullptr;
    a.first_hash = t->dev.first_hash;
    a.seeds = policy ? policy->seeds : nullptr;
    a.eng_a_pf = engine ? engine->a_pf : nullptr;
    a.eng_a_dec = engine ? engine->a_dec : nullptr;
    a.eng_budget = engine ? engine->budget : nullptr;
    a.eng_slowdown = engine ? engine->slowdown : 0.0;
    a.epochs = proxy ? proxy->epochs : 0;
    a.probe_ms = proxy ? proxy->probe_ms : 0;
    a.rtt_true = proxy ? proxy->rtt_true : nullptr;
    a.rtt_est = proxy ? proxy->rtt_est : nullptr;
    a.index_blocks = proxy ? proxy->index_blocks : -1;
    a.believed = proxy ? proxy->believed : nullptr;
    a.sections = sections;
    if (sections && (!segments || online || engine || proxy || (policy && policy->policy != 0)))
        return fail(GORGO_ERR_INVALID_ARG, "section timing exists for the fixed-weight cost model with the linear replica "
                                           "model in the segment formulation");
    if (proxy) {
        if (policy && policy->policy != 0)
            return fail(GORGO_ERR_INVALID_ARG, "imperfect proxy knowledge concerns the cost model, not the baseline policies");
        hipLaunchKernelGGL(smooth_rtt, dim3(1), dim3(WAVE), 0, s, proxy->rtt_true, proxy->rtt_est, proxy->epochs, pl.R,
                           proxy->alpha);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch smooth_rtt");
    }
    const int mode = mode_of(policy ? policy->policy : 0, online != nullptr);
    // (a row is written through before it is first read -- the request that brings a segment into a row slot resets the
    // row -- so only the never-cached row needs a value beforehand)
    if ((rc = prepare(pl, const_cast<double*>(d_rtt), segments ? a.last : nullptr, a.nseg, s))) return rc;
    if (segments) {
        mark(1, s);
        if (pl.N > 0 || online) {      // (an empty trace still reports the tuner's initial state)
            const SegmentKernel kernel = pl.each ? SIX_WAVEFRONTS : segment_kernel(pl, mode, engine != nullptr, proxy != nullptr, a.window);
            const size_t lds = replay_queue_lds_bytes(pl.R, pl.B, false, 0);
            if (pl.each) {
                if ((rc = launch_each(t, pl, mode, engine != nullptr, a, ws, s))) return rc;
            } else if (sections && kernel == SIX_WAVEFRONTS) {
                hipLaunchKernelGGL((replay_apart_kernel<MODE_COST_MODEL, false, false, true>), dim3((unsigned)pl.P), dim3(apart_threads<1>()),
                                   lds, s, a);
            } else if (sections && kernel == PAIRS) {
                hipLaunchKernelGGL((replay_apart_pairs_timed_kernel<MODE_COST_MODEL, false, false>), dim3((unsigned)((pl.P + 1) / 2)),
                                   dim3(apart_threads<2>()), 2 * lds, s, a);
            } else if (sections) {
                hipLaunchKernelGGL((replay_segments_kernel<MODE_COST_MODEL, false, false, 1, true>), dim3((unsigned)pl.P), dim3(seg_threads<1>()),
                                   lds, s, a);
            } else if (kernel == PACKED) {
                hipLaunchKernelGGL((replay_segments_kernel<MODE_COST_MODEL, false, false, 2>), dim3((unsigned)(pl.P / 2)),
                                   dim3(seg_threads<2>()), 2 * lds, s, a);
            } else {
                const bool eng = engine != nullptr;
                switch (mode) {
                    case MODE_COST_MODEL: launch_segments<MODE_COST_MODEL>(kernel, eng, proxy != nullptr, pl, s, a); break;
                    case MODE_ONLINE: launch_segments<MODE_ONLINE>(kernel, eng, proxy != nullptr, pl, s, a); break;
                    case MODE_LEAST_REQUEST: launch_segments<MODE_LEAST_REQUEST>(kernel, eng, false, pl, s, a); break;
                    case MODE_AFFINITY: launch_segments<MODE_AFFINITY>(kernel, eng, false, pl, s, a); break;
                    default: launch_segments<MODE_RANDOM>(kernel, eng, false, pl, s, a); break;
                }
            }
            if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch replay_segments_kernel");
        }
    } else if (pl.row_slots > 0) {
        RowArgs b;
        b.q = a;
        b.blk_off = t->dev.blk_off;
        b.ref = t->dev.row_ref;
        b.cells = reinterpret_cast<int64_t*>(ws + pl.off_tables);
        b.log = reinterpret_cast<uint32_t*>(ws + pl.off_spare);
        b.slots = pl.row_slots;
        b.words = pl.row_words;
        mark(1, s);                    // (nothing to be cleared: a row starts over before it is first read)
        if (pl.N > 0 || online) {      // (an empty trace still reports the tuner's initial state)
            const size_t lds = replay_rows_lds_bytes(pl.R, pl.B, engine != nullptr, a.window);
            const dim3 grid((unsigned)pl.P);
            switch (mode) {
                case MODE_COST_MODEL: launch_rows<MODE_COST_MODEL>(engine != nullptr, proxy != nullptr, grid, lds, s, b); break;
                case MODE_ONLINE: launch_rows<MODE_ONLINE>(engine != nullptr, proxy != nullptr, grid, lds, s, b); break;
                case MODE_LEAST_REQUEST: launch_rows<MODE_LEAST_REQUEST>(engine != nullptr, false, grid, lds, s, b); break;
                case MODE_AFFINITY: launch_rows<MODE_AFFINITY>(engine != nullptr, false, grid, lds, s, b); break;
                default: launch_rows<MODE_RANDOM>(engine != nullptr, false, grid, lds, s, b); break;
            }
            if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch replay_rows_kernel");
        }
    } else {
        BlockArgs b;
        b.q = a;
        b.blk_off = t->dev.blk_off;
        b.key = t->dev.key;
        b.first = t->dev.first;
        b.cap = pl.cap;
        b.cap_log2 = 0;
        while ((1ll << b.cap_log2) < pl.cap) ++b.cap_log2;
        b.tables = reinterpret_cast<Slot*>(ws + pl.off_tables);
        b.spare = reinterpret_cast<Slot*>(ws + pl.off_spare);
        b.routed = reinterpret_cast<uint8_t*>(ws + pl.off_route);
        const size_t nslots = (size_t)pl.P * pl.R * pl.cap;
        size_t blocks = (nslots + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(fill_slots, dim3((unsigned)blocks), dim3(256), 0, s, b.tables, nslots);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch fill_slots");
        mark(1, s);
        if (pl.N > 0 || online) {      // (an empty trace still reports the tuner's initial state)
            const size_t lds = replay_blocks_lds_bytes(pl.R, pl.B, engine != nullptr, a.window);
            const dim3 grid((unsigned)pl.P);
            switch (mode) {
                case MODE_COST_MODEL: launch_blocks<MODE_COST_MODEL>(engine != nullptr, proxy != nullptr, grid, lds, s, b); break;
                case MODE_ONLINE: launch_blocks<MODE_ONLINE>(engine != nullptr, proxy != nullptr, grid, lds, s, b); break;
                case MODE_LEAST_REQUEST: launch_blocks<MODE_LEAST_REQUEST>(engine != nullptr, false, grid, lds, s, b); break;
                case MODE_AFFINITY: launch_blocks<MODE_AFFINITY>(engine != nullptr, false, grid, lds, s, b); break;
                default: launch_blocks<MODE_RANDOM>(engine != nullptr, false, grid, lds, s, b); break;
            }
            if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch replay_blocks_kernel");
        }
    }
    mark(2, s);
    if (pl.p95_ttft || pl.p95_e2e) {
        // (one launch for both percentiles)
        const bool both = pl.p95_ttft && pl.p95_e2e;
        hipLaunchKernelGGL(select_kth, dim3((unsigned)pl.P, both ? 2 : 1), dim3(SEL_THREADS), 0, s, pl.p95_ttft ? ttft : e2e,
                           e2e, pl.N, (95 * pl.N + 99) / 100, pl.p95_ttft ? pl.p95_ttft : pl.p95_e2e, pl.p95_e2e);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "launch select_kth");
    }
    mark(3, s);
    g_marks.valid = g_marks_on && g_marks.device >= 0;
    return GORGO_OK;
}

int last_eval_kernel_ms(double* fill_ms, double* replay_ms, double* select_ms) {
    if (!g_marks.valid) return fail(GORGO_ERR_INVALID_ARG, "no evaluation has been enqueued on this thread");
    hipError_t e = hipEventSynchronize(g_marks.ev[3]);
    if (e != hipSuccess) return hip_fail(e, "hipEventSynchronize");
    float a = 0, b = 0, c = 0;
    if ((e = hipEventElapsedTime(&a, g_marks.ev[0], g_marks.ev[1])) != hipSuccess ||
        (e = hipEventElapsedTime(&b, g_marks.ev[1], g_marks.ev[2])) != hipSuccess ||
        (e = hipEventElapsedTime(&c, g_marks.ev[2], g_marks.ev[3])) != hipSuccess)
        return hip_fail(e, "hipEventElapsedTime");
    if (fill_ms) *fill_ms = a;
    if (replay_ms) *replay_ms = b;
    if (select_ms) *select_ms = c;
    return GORGO_OK;
}

}  // namespace gorgo
