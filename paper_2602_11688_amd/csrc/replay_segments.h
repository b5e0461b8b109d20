// Replay kernel, segment formulation (chain-consistent traces).
//
// On a chain-consistent trace every request is a root-to-node path of the key forest and a whole number of
// segments.  With the root-newest stamp order a replica's cache is always closed under taking prefixes,
// every block of a segment carries the same last-touching request, and a block is cached iff its
// (last request, position) is not below the replica's eviction cursor.  The cache state of a replay is
// therefore one 32-bit "last request that touched it" per (segment, replica), stored as dense rows of R
// cells addressed by segment id: no hashing, no probing.
//
// Eviction (least recently used block first) only moves a cursor and writes no cell.  The cursor of a
// replica walks that replica's log of routed requests, oldest first.  A logged request still *owns* the
// blocks of its path that no later request on the same replica has touched again; because paths of a forest
// share prefixes only, that is always a suffix [own, n) of its path.  `own` is kept up to date when a later
// request takes segments over (the cells just read say whom they belonged to), so the walk needs one small
// record per logged request (next request on the replica, own, n) and never re-reads cells.  Records that
// own nothing any more are dropped from the walk as soon as they are seen.
//
// The request loop is one dependent chain per replay: decision r changes the cursor, the cells and the load signal of
// one replica, and decision r + 1 may depend on them.  A dependent vector or scalar instruction costs a wavefront
// eight cycles (an independent one five), a branch on a vector comparison forty, a word handed to another wavefront through
// LDS and a barrier 180.  So only what the next decision needs is on the chain, in the hands of one wavefront, and everything
// else is done beside it by others of the same workgroup, which meet at ONE barrier per request:
//   X(r): the choice of request r is published, and so is what has left the load signals by the arrival of r + 1.
//   The deciding wavefront (lane = replica; two replays in its halves where R <= 32 and the launch packs) holds the
// load signals, the eviction cursors and the row cells of the current and the next request.  Per request it matches,
// scores, takes the minimum, announces the choice, moves the chosen replica's cursor.
//   The queue wavefront (one per replay; lane = service slot or replica) is one request behind: while r + 1 is being
// decided it serves r, keeps the latencies, and retires what completes by the arrival of r + 2.  The deciding
// wavefront adds the tokens of r to the load signal itself, which is right unless r has completed before r + 1 even
// arrives; the trace and the time scale alone can rule that out (r takes at least its decode time) and practically
// always do.
//   The book-keeping wavefront stores: cells, log records, ownership changes, routes and hit counts.
//   The front-end wavefront walks the trace two dozen requests ahead, eight requests at a time, and leaves a descriptor
// of each in an LDS ring; it touches the rows that will be read, so that they are in the L2 by then, and brings the row
// cells of the request after next, and the log records asked for, to LDS.  (A fifth wavefront for the cells frees half of
// its time but nothing on the chain: 1,024 replays of 250,000 requests 166.4 -> 174.5 ms.)
// Where one barrier is not enough -- r may complete before r + 1 arrives, r + 1 has more segments than the deciding
// wavefront preloads, the online tuner changes the weights after r -- the descriptor of r says so (DESC_SYNC), every
// wavefront of the workgroup reads that same word, and all meet once more, Y(r), when the queue and the book-keeping
// wavefront have caught up with r.  The number of barriers a wavefront executes depends on the descriptors alone, so
// none can wait for ever.  The deciding wavefront comes to Y(r) when it has matched r + 1 against the rows in hand, which
// the service of r does not concern; only the load signals, the weights and a longer path's rows wait for it.  (10,000
// requests, 32 replicas, 2 and 1,024 replays, every request with two meetings: a request a minute 11.2 and 12.3 ms with the
// match behind Y(r), so 9.8 and 11.2; without decode time 8.6 and 9.6, so 6.8 and 8.2.)
//
// 1,024 replays of 250,000 requests on 32 replicas: 241 ms with two barriers per request and half of its work between
// them, 154 ms so (0.61 us, some 1,450 cycles a request).  The deciding and the queue wavefront now have chains of
// the same length, each is the last to arrive about half of the time; 2 replays would take 0.53 us (they have six wavefronts).
#pragma once
#include "device_common.h"
#include "internal.h"

namespace gorgo {

// Log record of a routed request: next request routed to the same replica, start of the owned suffix of its
// path, and its number of blocks.  Read and written as one 64-bit word: next | own << 32 | n << 48.
struct LogRec {
    int32_t next;
    uint16_t own;
    uint16_t n;
};

struct SegArgs {
    const int64_t* ts;
    const int32_t* in_len;
    const int32_t* out_len;
    const int64_t* seg_off;
    const int64_t* blk_off;       // [N+1]
    const SegRef* seg;
    int64_t N;
    int32_t P, R, B;
    int64_t C;
    int64_t nseg;
    int32_t block_tokens;
    int32_t look, near;           // six and eight wavefronts: log records of look-ahead per replica, from when on (blocks of room)
    double a_pf, a_dec;
    double least_dec;             // smallest decode time per output token of any replica
    const double* rtt;
    const double* params;
    const double* scale;
    int32_t* last;   // [P][nseg][R], -1 = never touched
    LogRec* log;     // [P][N]
    Rec* rec;        // [P][N]
    uint8_t* route;  // [P][N], nullable
    uint16_t* hit;   // nullable
    double* ttft;    // nullable
    double* e2e;     // nullable
    // online tuner (only read by the kernel's online variant)
    int32_t window, hop;
    int64_t steps;             // tuner steps of one replay
    const double* tuner;       // lo[3], hi[3], ln lo[3], ln hi[3], sigma0, exp(0.4), exp(-0.1)
    const double* ln_theta0;   // [P][3]
    const double* z;           // [P][steps][3]
    double* theta_step;        // [P][steps][3], nullable
    double* fitness_step;      // [P][steps], nullable
    double* theta_final;       // [P][3], nullable
    double* sigma_final;       // [P], nullable
    int32_t* accepted;         // [P], nullable
    // baseline policies
    const uint32_t* first_hash;   // [N] hash of the request's first block
    const uint64_t* seeds;        // [P] seed of the random policy
    // engine model of a replica (only read by the kernel's engine variants)
    const double* eng_a_pf;       // [R] prefill ms per token
    const double* eng_a_dec;      // [R] decode ms per token
    const double* eng_budget;     // [R] KV budget in tokens, 0 = none
    double eng_slowdown;
    // imperfect proxy knowledge (only read by the kernel's proxy variants)
    int32_t epochs, probe_ms;     // probe epochs given, and their length
    const double* rtt_true;       // [epochs][R] round trip time a request dispatched in the epoch experiences
    const double* rtt_est;        // [epochs][R] the proxy's moving average of them: what Eq. 3 scores with
    int64_t index_blocks;         // >= 0: Eq. 3 takes its cached prefix from the proxy's own index (an LRU of this
                                  // many blocks per replica, 0 = it never forgets); < 0: from the replica's cache
    uint16_t* believed;           // [P][N] blocks the proxy believed cached on the chosen replica, nullable
    unsigned long long* sections; // timed instantiation only: [P][3][SECTIONS] cycles per section (deciding; queue; front-end and book-keeping wavefront)
};

// What picks the replica: the cost model of Eq. 3 with fixed weights, the same with the online tuner, or one
// of the baseline policies of Sec. 4 (prefix-cache and proxy-only least-load are the cost model with weights
// (0, 1, 0) and (0, 0, 1)); MODE_GIVEN: there is one replica (a workgroup of replay_each.h).
enum SegMode { MODE_COST_MODEL = 0, MODE_ONLINE = 1, MODE_LEAST_REQUEST = 2, MODE_AFFINITY = 3, MODE_RANDOM = 4, MODE_GIVEN = 5 };

// A 32-bit value spread over R replicas: floor(h * R / 2^32).
__device__ __forceinline__ int spread(uint32_t h, int R) { return (int)(((uint64_t)h * (uint64_t)R) >> 32); }

// First word of Philox-4x32 with 10 rounds (Salmon, Moraes, Dror, Shaw, SC'11) for counter (c0, c1, 0, 0): per
// round two 32x32 -> 64 bit products of counter words 0 and 2 with the generator's multipliers, xors with the
// other two words and the key, and a Weyl step of the key.
__device__ __forceinline__ uint32_t philox4x32_10_first(uint32_t c0, uint32_t c1, uint32_t k0, uint32_t k1) {
    uint32_t c2 = 0, c3 = 0;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t a = (uint64_t)0xD2511F53u * c0, b = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(b >> 32) ^ c1 ^ k0, n2 = (uint32_t)(a >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c0;
}

constexpr int HALF = WAVE / 2;               // lanes of one of two packed replays
constexpr int SEG_CHUNK = 8;                 // segments of a request whose rows are loaded together

// Orders the LDS accesses of one wavefront's lanes (the hardware executes them in program order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// dynamic LDS of one replay: its queues, then the tuner's TTFT window
__host__ __device__ inline size_t replay_queue_lds_bytes(int R, int B, bool engine, int window) {
    return SlotQueues::bytes(R, B, engine) + (size_t)((window + 7) & ~7) * sizeof(double);
}

// exp(x) for |x| <= 700 from additions and multiplications only, in a fixed order, so that the weights the
// online tuner proposes (Sec. 2.3) have the same bits wherever they are computed: k = floor(x / ln 2 + 1/2),
// r = (x - k LN2_HI) - k LN2_LO with ln 2 split so that k LN2_HI is exact, exp(r) as its Taylor polynomial of
// degree 13 by Horner's rule from the highest term down, times 2^k.
__device__ __forceinline__ double tuner_exp(double x) {
    const double INV_LN2 = 1.44269504088896338700e+00;
    const double LN2_HI = 6.93147180369123816490e-01;
    const double LN2_LO = 1.90821492927058770002e-10;
    const double k = __builtin_floor(x * INV_LN2 + 0.5);
    const double r = (x - k * LN2_HI) - k * LN2_LO;
    double p = 1.0 / 6227020800.0;
    p = p * r + 1.0 / 479001600.0;
    p = p * r + 1.0 / 39916800.0;
    p = p * r + 1.0 / 3628800.0;
    p = p * r + 1.0 / 362880.0;
    p = p * r + 1.0 / 40320.0;
    p = p * r + 1.0 / 5040.0;
    p = p * r + 1.0 / 720.0;
    p = p * r + 1.0 / 120.0;
    p = p * r + 1.0 / 24.0;
    p = p * r + 1.0 / 6.0;
    p = p * r + 1.0 / 2.0;
    p = p * r + 1.0;
    p = p * r + 1.0;
    const unsigned long long bits = (unsigned long long)((long long)k + 1023) << 52;
    return p * __longlong_as_double((long long)bits);
}
__device__ __forceinline__ double clip(double x, double lo, double hi) {
    const double up = x < lo ? lo : x;
    return hi < up ? hi : up;
}

// k-th smallest (1-based) of the W values of `ring` (LDS, W <= 1024), by taking elements out from the nearer end: the
// largest W + 1 - k times, or the smallest k times (the tuner's k is the 95th percentile's: 7 rounds for a window
// of 128, against 128 comparisons for every element when the elements are ranked by counting).  Lane l looks after
// the elements l, l + 64, ...; a round takes this lane's best remaining element, finds the best over the wavefront
// (two 32-bit cross-lane reductions on the order-preserving integer image of the doubles, the second one only when
// the high words tie) and marks it as taken in the lowest lane that holds it.  Equal values are taken one by one, as
// a sorted list would have them.
__device__ __forceinline__ double window_kth(const double* ring, int W, int kth, int lane) {
    const bool from_top = W + 1 - kth <= kth;
    const int rounds = from_top ? W + 1 - kth : kth;
    unsigned taken = 0;                 // bit c: element c * 64 + lane is out
    unsigned last_hi = 0, last_lo = 0;
    // the wanted end is the largest key: the order-preserving integer image of the value, complemented from the bottom
    auto key_of = [&](int e) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(ring[e]);
        const unsigned long long up = (b >> 63) ? ~b : (b | 0x8000000000000000ull);      // increasing with the value
        return from_top ? up : ~up;
    };
    // (this lane's first two elements stay in registers: windows of up to 128 values read LDS once)
    const bool has0 = lane < W, has1 = lane + WAVE < W;
    const unsigned long long key0 = has0 ? key_of(lane) : 0, key1 = has1 ? key_of(lane + WAVE) : 0;
    for (int round = 0; round < rounds; ++round) {
        const bool use0 = has0 && (taken & 1u) == 0;
        unsigned long long best = use0 ? key0 : 0;
        int best_c = use0 ? 0 : -1;
        const bool use1 = has1 && (taken & 2u) == 0 && (best_c < 0 || key1 > best);
        best = use1 ? key1 : best;
        best_c = use1 ? 1 : best_c;
        for (int c = 2, e = lane + 2 * WAVE; e < W; ++c, e += WAVE) {
            const unsigned long long key = key_of(e);
            const bool better = ((taken >> c) & 1u) == 0 && (best_c < 0 || key > best);
            best = better ? key : best;
            best_c = better ? c : best_c;
        }
        const bool have = best_c >= 0;
        const unsigned hi = (unsigned)(best >> 32), lo = (unsigned)best;
        const unsigned top_hi = ~wave_min_u32(~(have ? hi : 0u));
        const bool tie = have && hi == top_hi;
        unsigned long long who = __ballot(tie);
        if (__builtin_popcountll(who) > 1) {
            const unsigned top_lo = ~wave_min_u32(~(tie ? lo : 0u));
            who = __ballot(tie && lo == top_lo);
        }
        const int winner = __ffsll(who) - 1;
        last_hi = (unsigned)__builtin_amdgcn_readlane((int)hi, winner);
        last_lo = (unsigned)__builtin_amdgcn_readlane((int)lo, winner);
        taken |= lane == winner ? 1u << (best_c & 31) : 0u;
    }
    const unsigned long long key = ((unsigned long long)last_hi << 32) | last_lo;
    const unsigned long long up = from_top ? key : ~key;
    const unsigned long long b = (up >> 63) ? (up & 0x7FFFFFFFFFFFFFFFull) : ~up;
    return __longlong_as_double((long long)b);
}

// Cached blocks of one segment [pos, end) whose row cell holds rl, against a cursor (c_r, c_k): all of them
// if a later request than the cursor's touched it last, those below the cursor position if the cursor's
// request did, none otherwise.  (A never-touched cell, -1, can only tie with the initial cursor (-1, 0).)
__device__ __forceinline__ int cached_in(int32_t rl, int pos, int end, int c_r, int c_k) {
    const int len = end - pos;
    int part = c_k - pos;
    part = part < 0 ? 0 : (part > len ? len : part);
    return rl > c_r ? len : (rl == c_r ? part : 0);
}


// ---------------------------------------------------------------------------------------------- hand-over
// Descriptor of one request, written by the front end.
struct __align__(16) SegDesc {
    uint32_t rowoff[SEG_CHUNK];  // first eight segments: byte offset, within the replay's rows, of the row that the match
                         // reads.  Past the last segment: the never-cached row.  Also the never-cached row for a segment whose
                         // row slot starts over with this request (SEG_FRESH: what the slot still holds belongs to a segment of
                         // the past), and for one whose slot started over with one of the three requests before (this request's
                         // rows are loaded before those stores are sure to be there)
    int32_t end[SEG_CHUNK];      // blocks of the request up to and including the segment (past the last one: n)
    int32_t L, n, s;     // input tokens, blocks, segments
    int32_t flags;       // DESC_* | leading segments shared with the request j before, as far as none in between started them
                         // over, << DESC_COMMON[j - 1] | index of the first fresh segment among the first eight (8: none) << 16
    int64_t j0;          // index of the request's first segment reference (for requests of more than 8 segments)
    int32_t target;      // replica dictated by the session-affinity / random policy
    uint32_t tail;       // the row of the request's last segment if DESC_FRESH_TAIL, else the spare row
    uint32_t slot[SEG_CHUNK];   // where the rows of the first eight segments really are (past the last one: the spare row)
    double t2[2];        // arrival of the request after next at the time scale of each replay of the workgroup
    double dec;          // decode time in the linear model
    int32_t O;           // output tokens
    int32_t pad;
};
static_assert(sizeof(SegDesc) == 160, "descriptor layout");
constexpr int DESC_MORE4 = 1;        // more than four segments
constexpr int DESC_DEEP = 2;         // more than eight segments
constexpr int DESC_FRESH_TAIL = 4;   // the last segment is fresh, among the first eight, and lanes 32..63 reset its row
constexpr int DESC_FRESH_MORE = 8;   // further fresh segments among the first eight
constexpr int DESC_SYNC = 16;        // all wavefronts meet once more between this request and the next
constexpr int DESC_SHARED = 0xF0FF00;            // any leading segment shared with the three requests before
constexpr int DESC_RING = 16;        // descriptors in flight (power of two)
constexpr int DESC_GROUP = WAVE / SEG_CHUNK;     // requests whose descriptors are written together
constexpr int DESC_AHEAD = DESC_GROUP;           // how far ahead of the request in hand
static_assert(DESC_AHEAD + DESC_GROUP <= DESC_RING, "the front end overwrites descriptors of requests that are done with");
constexpr int32_t NEVER_CACHED = INT32_MIN;      // cell value of the extra row: below any cursor

constexpr int CELL_SETS = 3;          // requests whose row cells are in LDS: two ahead are loaded while one is at hand
// Log records of look-ahead kept in LDS, of each cursor: eight per replica.  The proxy variants have two cursors and keep
// eight for 32 replicas or fewer, four for more (a cursor among 33 needs one half as often as one among 16); with the
// engine model and the tuner as well, half of that.  Their workgroups then fit a CU as often as the others' do.
__host__ __device__ constexpr int look_words(bool engine, bool online, bool proxy) {
    return proxy ? (engine && online ? 2 * WAVE : 4 * WAVE) : 8 * WAVE;
}
// How often the look-ahead is fed, as a mask: a record per replica every fourth request, or every eighth with 24 replicas
// or more.  The cursors of all replicas together pass about 0.9 log records per request, so the more replicas there are
// the less often each needs one, and taking one costs the deciding wavefront some 500 cycles.  (1,024 replays of 10,000
// requests, every fourth against every eighth: 16 replicas 7.34 / 7.29 ms, with bursts 7.52 / 7.59, proxy variant 9.50 /
// 9.54; 20 replicas 6.93 / 6.84, 7.14 / 7.07, 8.57 / 8.47; 24 replicas 6.69 / 6.57, 6.89 / 6.74, 8.17 / 8.03; 32 replicas
// 6.54 / 6.37, 6.58 / 6.40, 7.92 / 7.74.  All requests sent to one replica, 256 replays: 8.68 / 8.74 whatever their number:
// its cursor then runs past what either brings, and takes most records from memory.)
__host__ __device__ constexpr int look_every(int R) { return R >= 24 ? 7 : 3; }
// What every replica would mean for a request, written by its lane before the minimum is known; the replica with the
// minimum is announced by its number alone.
template <bool PROXY>
struct __align__(16) Choice {
    double prefill;                   // prefill time (linear model) or tokens to prefill
    int owner;                        // request whose owned suffix would start at `end`, -2: none (or dealt with)
    unsigned hit_end;                 // cached blocks | end << 16
};
template <>
struct __align__(16) Choice<true> {
    int prefill;                      // tokens to prefill
    int seen;                         // blocks the proxy believes cached
    int owner;
    unsigned hit_end;
};
// An ownership change: `owner`'s owned suffix now starts at `end`.
struct OwnChange {
    int owner, end;
};
constexpr int OWN_LIST = -3;              // in Choice::owner: the changes are in Handover::changes, as many as its `end` says
// What the deciding and the queue wavefront tell each other, in both formulations.
template <bool PROXY>
struct __align__(16) QueueHandover {
    Choice<PROXY> choice[2][WAVE];        // [request mod 2][replica]
    double gone[2][WAVE];                 // [request mod 2][replica]: minus the tokens (least-request policy: the requests) that
                                          // left the load signal between the previous request's arrival and this one's
    double w[2][3];                       // online tuner: weights in use
    int best[2][2];                       // [request mod 2][replay of the workgroup] the choice: lane of the replica
    double half[PROXY ? 1 : WAVE];        // half the round trip time per replica (proxy variants: kept by the queue wavefront)
    double rtt[PROXY ? 2 : 1][PROXY ? WAVE : 1];   // proxy variants, [request mod 2]: estimated round trip time per replica
};
template <bool PROXY, int PACK, int LOOK>
struct Handover : QueueHandover<PROXY> {
    static constexpr int LOOK_WORDS = LOOK;
    static constexpr bool APART = false;
    int32_t cells[CELL_SETS][SEG_CHUNK][WAVE];    // [request mod 3]: row cells of the request's first eight segments per replica
    // look-ahead of the eviction cursors (the cache's; the proxy's index's): per replica, log records fetched ahead
    // of the cursor (one slot is always free)
    unsigned long long look[PROXY ? 2 : 1][LOOK];
    // the log record that the front end is to fetch, every fourth or eighth request, then what it has fetched
    unsigned long long record[PROXY ? 2 : 1][WAVE];
    SegDesc ring[DESC_RING];
    int first[WAVE];                      // first request routed to each replica (-1: none yet)
    OwnChange changes[2][PACK][SEG_CHUNK];   // [request mod 2][replay]
};

// Workgroup barrier; `after_lds`: this wavefront's LDS accesses have been performed before it arrives (what it wrote is
// there for the others, what it read has been read).  Global memory is not waited for: the wavefronts of a workgroup
// share one CU, whose vector memory accesses are performed in the order they were issued.
__device__ __forceinline__ void meet(bool after_lds) {
    if (after_lds) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_barrier" ::: "memory");
}

// Section clock of the timed instantiation: cycles since the previous call are added to section k.  (Reading the
// clock waits for this wavefront's outstanding LDS and scalar-memory accesses, which the plain kernel does not.)
constexpr int SECTIONS = 12;
template <bool TIMED>
struct SectionClock {
    unsigned long long acc[SECTIONS] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    unsigned long long last = 0;
    __device__ __forceinline__ void start() {
        if (TIMED) last = __builtin_readcyclecounter();
    }
    __device__ __forceinline__ void tick(int k) {
        if (TIMED) {
            const unsigned long long now = __builtin_readcyclecounter();
            acc[k] += now - last;
            last = now;
        }
    }
    __device__ __forceinline__ void write(unsigned long long* out, int lane) {
        if (TIMED && out && lane == 0)
            for (int k = 0; k < SECTIONS; ++k) out[k] = acc[k];
    }
};


// Lowest-index minimum as wave_argmin, with the lane mask given.
__device__ __forceinline__ int argmin_lanes(double v, bool in) {
    const unsigned long long bits = (unsigned long long)__double_as_longlong(v + 0.0);
    const unsigned hi = (unsigned)(bits >> 32), lo = (unsigned)bits;
    const unsigned neg = (unsigned)((int)hi >> 31);
    const unsigned khi = in ? hi ^ (neg | 0x80000000u) : 0xffffffffu;
    const unsigned mhi = wave_min_u32(khi);
    const bool tie = khi == mhi;             // (lanes outside hold the all-ones key, which no score maps to)
    const unsigned long long ties = ballot(tie);
    if (__builtin_popcountll(ties) <= 1) return __builtin_ctzll(ties);      // one lane holds the smallest high word: done
    const unsigned klo = lo ^ neg;
    const unsigned mlo = wave_min_u32(tie ? klo : 0xffffffffu);
    return __builtin_ctzll(ballot(tie && klo == mlo));
}

// Lowest-index minimum over the wavefront or over either half of it (PACK = 2): a mask with one bit per replay.  The
// values are compared as in wave_argmin; none is NaN or -0.0, lanes without a replica hold +inf.
template <int PACK>
__device__ __forceinline__ unsigned long long argmin_mask(double v, bool upper) {
    const unsigned long long bits = (unsigned long long)__double_as_longlong(v);
    const unsigned hi = (unsigned)(bits >> 32), lo = (unsigned)bits;
    const unsigned neg = (unsigned)((int)hi >> 31);
    const unsigned khi = hi ^ (neg | 0x80000000u);
    auto least = [&](unsigned x) {
        x = dpp_min_u32<0x111, 0xf>(x);   // row_shr:1
        x = dpp_min_u32<0x112, 0xf>(x);   // row_shr:2
        x = dpp_min_u32<0x114, 0xf>(x);   // row_shr:4
        x = dpp_min_u32<0x118, 0xf>(x);   // row_shr:8
        x = dpp_min_u32<0x142, 0xa>(x);   // row_bcast:15 into rows 1, 3
        if (PACK == 2) {
            const unsigned m0 = (unsigned)__builtin_amdgcn_readlane((int)x, HALF - 1);
            const unsigned m1 = (unsigned)__builtin_amdgcn_readlane((int)x, WAVE - 1);
            return upper ? m1 : m0;
        }
        x = dpp_min_u32<0x143, 0xc>(x);   // row_bcast:31 into rows 2, 3
        return (unsigned)__builtin_amdgcn_readlane((int)x, WAVE - 1);
    };
    auto lowest = [](unsigned long long m) {
        if (PACK == 1) return m & (0 - m);
        const unsigned a = (unsigned)m, b = (unsigned)(m >> 32);
        return (unsigned long long)(a & (0 - a)) | ((unsigned long long)(b & (0 - b)) << 32);
    };
    const bool tie = khi == least(khi);
    const unsigned long long ties = ballot(tie);
    if (__builtin_popcountll(ties) == PACK) return ties;      // one lane (of each half) holds the smallest high word: done
    const unsigned klo = lo ^ neg;
    const unsigned mlo = least(tie ? klo : 0xffffffffu);
    return lowest(ballot(tie && klo == mlo));
}
__device__ __forceinline__ bool of_mask(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Eviction cursor of one LRU over a replica's log of routed requests, held by lane = replica.
//   cursor: blocks last touched by a request before cur_r, or by cur_r at positions >= cur_k, are evicted;
//   cur_own is where cur_r's owned suffix starts.
//   The log is read ahead of the cursor, a record per visit: last_r is the last record read, fill_r the one after it if
//   its link is known.  Where it is not (the log had not gone on), the next visit reads the link again, so that nothing
//   has to be done for this when a request is added to the log.
//   pend_*: a record being fetched by the front end; ownership changes made to it meanwhile are kept in pend_own and
//   override the loaded field.
//   Records that have arrived wait in a ring in LDS until the cursor reaches them: the log is
//   read as far ahead of the cursor as the ring is long, so that a request which evicts several records' blocks at
//   once rarely has to wait for a record to come from memory.
//   The records in memory are written by the book-keeping wavefront, which is one request behind: the ownership change
//   that the latest decided request makes (Fresh) may not have arrived, and is applied to what is loaded on the spot.
// The same machinery serves the proxy's own index of the replica, an LRU of another capacity over the same log.
struct Fresh {
    int r = -1;               // the latest decided request (its own record cannot be loaded yet)
    int owner = -2, end = 0;  // on the replica it went to: record whose owned suffix now starts at `end`
    int count = 0;            // ... or several such records
    const OwnChange* list = nullptr;
    __device__ __forceinline__ int of(int x) const {
        int own = x == owner ? end : -1;
        for (int i = 0; ballot(i < count) != 0; ++i) {
            const OwnChange c = list[i & (SEG_CHUNK - 1)];
            own = i < count && c.owner == x ? c.end : own;
        }
        return own;
    }
};
template <int WORDS>
struct EvictCursor {
    int cur_r = -1, cur_k = 0, cur_own = 0;
    int last_r = -1, fill_r = -1;
    int pend_r = -1, pend_own = -1;      // pend_r: record asked for (last_r: only its link), -1 none
    unsigned long long* record = nullptr;            // where it will be
    // The look-ahead: a ring of records in LDS (packed r | own << 32 | n << 48), ring_cnt of them from slot ring_head on,
    // the youngest being request ring_hi.
    unsigned long long* ring = nullptr;
    int apart = 0;            // log2 of the distance between a lane's slots
    int ring_head = 0, ring_cnt = 0, ring_hi = -1;
    int over = 0;             // blocks this LRU holds beyond its capacity (below 0: room)
    int n_spot = 0, n_adv = 0, n_dead = 0;       // statistics (only the timed instantiation reads them): records fetched
                                                 // on the spot, cursor advances, records dropped because they own nothing

    // `look`, `record`: the handed-over words of this cursor.  Lanes that no replica can have where the slots are 32 apart use
    // their own word of `record` instead, which nothing else is done with.
    __device__ __forceinline__ void init(unsigned long long* look, unsigned long long* record_, int R, int lane) {
        apart = WORDS < 8 * WAVE && R <= HALF ? 5 : 6;
        const bool there = lane < 1 << apart;
        ring = there ? look + lane : record_ + lane;
        record = record_ + lane;
        *record = ~0ull;
        if (there)
            for (int k = 0; k < slots(); ++k) *at(k) = ~0ull;
    }
    __device__ __forceinline__ int slots() const { return WORDS < 8 * WAVE ? WORDS >> apart : 8; }
    __device__ __forceinline__ unsigned long long* at(int k) const { return ring + ((k & (slots() - 1)) << (WORDS < 8 * WAVE ? apart : 6)); }

    // In the lanes with `who` set, what was asked for has arrived: the link of last_r, or a record, which is dropped if
    // it owns nothing and else joins the ring.  Straight-line code: lanes with nothing pending go through it unchanged
    // (every lane stores to LDS: those with nothing for the ring into its free slot).
    __device__ __forceinline__ void take_pending(unsigned long long raw, bool who = true) {
        const bool have = who && pend_r >= 0;
        const unsigned hi = (unsigned)(raw >> 32);
        const int n = (int)(hi >> 16);
        const int own_mem = (int)(hi & 0xFFFFu);
        const int own = pend_own > own_mem ? pend_own : own_mem;
        const bool record = have && pend_r != last_r;
        const bool alive = record && own < n;
        *at(ring_head + ring_cnt) = (unsigned long long)(unsigned)pend_r | ((unsigned long long)((hi & 0xFFFF0000u) | (unsigned)own) << 32);
        ring_cnt += alive ? 1 : 0;
        ring_hi = alive ? pend_r : ring_hi;
        n_dead += record && !alive ? 1 : 0;
        fill_r = have ? (int)(unsigned)raw : fill_r;
        last_r = have ? pend_r : last_r;
        pend_r = have ? -1 : pend_r;
    }
    // What the next visit has to read: the record after the last one, or that one's link (-1: nothing, the log is empty).
    // A replica's first request is announced in `first`.
    __device__ __forceinline__ int wanted(const Fresh& f, int first) {
        fill_r = last_r < 0 && fill_r < 0 ? first : fill_r;
        return fill_r >= 0 && fill_r != f.r ? fill_r : last_r;
    }
    // Asks for the next record of the log where the ring has room for it (`spare`, the record behind the log, where
    // there is nothing to fetch).  Called right after take_pending: nothing is pending.  The front end loads it after
    // X(r), when everything that r - 1 changes is there; what r changes is kept in pend_own.
    __device__ __forceinline__ int ask(int spare, const Fresh& f, int first) {
        const int x = wanted(f, first);
        const bool want = x >= 0 && ring_cnt < slots() - 1;
        pend_r = want ? x : -1;
        pend_own = -1;
        return want ? x : spare;
    }
    // whether request `owner` may be one of the records in the ring (then disowned_anywhere is the call to make)
    __device__ __forceinline__ bool maybe_in_ring(int owner) const { return ring_cnt > 0 && owner <= ring_hi; }
    // request `owner`'s owned suffix now starts at `end` (owner = -2: nobody's); the owner is not in the ring
    __device__ __forceinline__ void disowned(int owner, int end) {
        cur_own = owner == cur_r ? end : cur_own;
        pend_own = owner == pend_r ? end : pend_own;
    }
    // The owner may be a record in the ring: its copy there (every slot of a trip is looked at before any is written; a number may
    // stand in the free slot as well).  Eight slots a trip to LDS; where there is the index's ring as well four, for with eight
    // the proxy variants took 96 registers and spilled six, 85 so.  (10,000 requests, 1,024 replays, 32 replicas of 700 blocks: one
    // slot a trip 9.0 ms, proxy 14.8; four 6.5 and 8.5; eight 6.4 and 8.5.  All lanes together, a slot each: proxy 8.5.)
    __device__ __forceinline__ void disowned_in_ring(int owner, int end) {
        constexpr int SLOTS = WORDS < 8 * WAVE ? WORDS >> 5 : 8;      // (at most; with fewer some are looked at twice)
        constexpr int TRIP = WORDS < 8 * WAVE ? 4 : 8;
#pragma nounroll
        for (int k0 = 0; k0 < SLOTS; k0 += TRIP) {
            unsigned found = 0;
#pragma unroll
            for (int k = 0; k < TRIP; ++k) found |= (int)(unsigned)*at(k0 + k) == owner ? 1u << k : 0u;
            for (; found != 0; found &= found - 1) {
                unsigned long long* const e = at(k0 + __builtin_ctz(found));
                *e = (*e & ~(0xFFFFull << 32)) | ((unsigned long long)(unsigned)end << 32);
            }
        }
    }
    // the same where that is not known (only called by the lanes it concerns)
    __device__ __forceinline__ void disowned_anywhere(int owner, int end) {
        disowned(owner, end);
        if (maybe_in_ring(owner)) disowned_in_ring(owner, end);
    }
    // takes up to E blocks from the owned suffix of the cursor's record
    __device__ __forceinline__ void take_from_cursor(int& E) {
        int avail = cur_k - cur_own;
        avail = avail > 0 ? avail : 0;
        const int take = avail < E ? avail : E;
        cur_k -= take;
        E -= take;
    }
    // The cursor moves on to further records until E blocks have been given up (all lanes together, those with
    // nothing to evict unchanged): records come from the ring, and from memory on the spot when the ring has run
    // out.  Works on a copy of the state, written back at the end: the request loop's common path, which does not
    // come here, then carries no register copies for this loop's sake.
    __device__ __forceinline__ void advance(int E_in, const unsigned long long* log64, int spare, const Fresh& f, int first) {
        EvictCursor w = *this;
        int E = E_in;
        w.advance_loop(E, log64, spare, f, first);
        *this = w;
    }
    __device__ __forceinline__ void advance_loop(int& E, const unsigned long long* log64, int spare, const Fresh& f, int first) {
        int asked = 0;
        do {
            const bool empty = E > 0 && ring_cnt == 0;
            if (ballot(empty) != 0) {
                // fetch a record, or the link to it, on the spot (what the front end has been asked for, if anything, may
                // not be there yet)
                const bool asked_for = pend_r >= 0;
                const int x = asked_for ? pend_r : wanted(f, first);
                // (no record, or a link that stays open: cannot happen while blocks are to be evicted; bounds the loop)
                const bool stuck = empty && (x < 0 || (x == last_r && asked >= 2));
                const bool fetch = empty && !stuck;
                asked = fetch ? (x == last_r ? asked + 1 : 0) : asked;
                E = stuck ? 0 : E;
                const unsigned long long got = ld(&log64[fetch ? x : spare]);
                pend_own = fetch && !asked_for ? f.of(x) : pend_own;
                pend_r = fetch ? x : pend_r;
                n_spot += fetch ? 1 : 0;
                take_pending(got, fetch);
                continue;
            }
            const bool go = E > 0;
            const unsigned long long e = *at(ring_head);
            const unsigned hi = (unsigned)(e >> 32);
            n_adv += go ? 1 : 0;
            cur_r = go ? (int)(unsigned)e : cur_r;
            cur_k = go ? (int)(hi >> 16) : cur_k;
            cur_own = go ? (int)(hi & 0xFFFFu) : cur_own;
            ring_head += go ? 1 : 0;
            ring_cnt -= go ? 1 : 0;
            take_from_cursor(E);         // (lanes with E = 0 take nothing)
        } while (ballot(E > 0) != 0);
    }
    // `added` blocks have joined the LRU.  First half: what the cursor's own record can give up, straight-line code;
    // returns what is still to be evicted.  Second half (advance), where some lane has any: steps to further records
    // (all lanes together, those with nothing to evict unchanged), taking records from the ring, and from memory on the
    // spot when the ring has run out.
    __device__ __forceinline__ int evict_first(int added) {
        over += added;
        int E = over > 0 ? over : 0;
        over -= E;
        take_from_cursor(E);
        return E;
    }
};

// Loads that only bring what somebody will read to the L2.  Each has a register of its own that nothing is done with until the
// next ones are due: put together, they had to be waited for where they were issued, for a trip to memory.  (2,048 replays of 40,000
// requests on 32 replicas 31.8 -> 30.9 ms; six wavefronts, 64 of 50,000 on eight 27.2 -> 26.8.)
template <int PACK>
struct Touched {
    int first = 0, last = 0, first2 = 0, last2 = 0, also = 0;
    // a row of either replay at `off`; to_end: to its last word, where that may be on another cache line (else 0)
    __device__ __forceinline__ void rows(const char* rows, uint32_t off, uint32_t to_end, uint32_t other_replay) {
        first = ld(reinterpret_cast<const int32_t*>(rows + off));
        if (PACK == 2) first2 = ld(reinterpret_cast<const int32_t*>(rows + (off + other_replay)));
        if (to_end != 0) {
            last = ld(reinterpret_cast<const int32_t*>(rows + (off + to_end)));
            if (PACK == 2) last2 = ld(reinterpret_cast<const int32_t*>(rows + (off + other_replay + to_end)));
        }
    }
    __device__ __forceinline__ void done() const { asm volatile("" ::"v"(first), "v"(last), "v"(first2), "v"(last2), "v"(also)); }
};

// ---------------------------------------------------------------------------------------------- front end
// Front-end wavefront: lane = (request of a group of eight, segment reference).  A group's scalars, references and
// descriptors are requested, requested and written in turn, eight requests apart, so that no load is waited for.
template <int MODE, bool PROXY, int PACK, bool TIMED, class Comm>
__device__ __forceinline__ void front_wave(const SegArgs& a, int lane, Comm* comm) {
    constexpr bool APART = Comm::APART;      // the book-keeping wavefront touches the rows, the evicting one reads the log
    constexpr bool SIGNAL = MODE == MODE_COST_MODEL || MODE == MODE_ONLINE || MODE == MODE_LEAST_REQUEST;
    const int R = a.R, N = (int)a.N;
    const int q = lane / SEG_CHUNK, k = lane % SEG_CHUNK;
    const double least_dec = kept(a.least_dec), a_dec = kept(a.a_dec);
    const size_t p = MODE == MODE_GIVEN ? 0 : (size_t)blockIdx.x * PACK;
    const bool pair = PACK == 2 && (!APART || p + 1 < (size_t)a.P);      // (four wavefronts: an even number of replays)
    const double scale0 = a.scale[p], scale1 = PACK == 2 ? a.scale[p + (pair ? 1 : 0)] : 0.0;
    const uint64_t seed = MODE == MODE_RANDOM ? a.seeds[p] : 0;
    const uint32_t row_bytes = (uint32_t)R * 4u;
    const uint32_t never_off = (uint32_t)(a.nseg - 2) * row_bytes;      // the extra row that no request touches
    const uint32_t spare_off = (uint32_t)(a.nseg - 1) * row_bytes;      // the row that nothing reads
    const char* const rows = reinterpret_cast<const char*>(a.last + p * (size_t)a.nseg * R);
    // lane = replica, for the row cells and the log records that the deciding wavefront gets
    const bool upper = pair && lane >= HALF;
    const int rl = PACK == 2 ? lane & (HALF - 1) : lane;
    const uint32_t lane_off = (upper ? (uint32_t)a.nseg * row_bytes : 0u) + (uint32_t)(rl < R ? rl : 0) * 4u;
    const unsigned long long* const log64 = reinterpret_cast<const unsigned long long*>(a.log + (p + (upper ? 1 : 0)) * ((size_t)N + 1));
    const uint32_t other_replay = PACK == 2 ? (uint32_t)a.nseg * row_bytes : 0u;
    // A request's numbers as they are in memory: nothing is done with them before the group is next, so that no load is
    // waited for where it is issued (low words where only differences count).
    struct Scalars {
        int64_t j0;
        uint32_t j1, j2, b0, b1;
        int64_t ts0, ts1, ts2;
        int L, O;
        uint32_t hash;
    };
    auto load_scalars = [&](int g0, Scalars& c) {
        const int r = g0 + q;
        const int x = r < N ? r : N - 1, x1 = r + 1 < N ? r + 1 : N - 1, x2 = r + 2 < N ? r + 2 : N - 1;
        auto low = [](const int64_t* at) { return *reinterpret_cast<const uint32_t*>(at); };
        c.j0 = a.seg_off[x];
        c.j1 = low(&a.seg_off[x + 1]);
        c.j2 = low(&a.seg_off[x1 + 1]);
        c.b0 = low(&a.blk_off[x]);
        c.b1 = low(&a.blk_off[x + 1]);
        c.ts0 = a.ts[x];
        c.ts1 = a.ts[x1];
        c.ts2 = a.ts[x2];
        c.L = a.in_len[x];
        c.O = a.out_len[x];
        c.hash = MODE == MODE_AFFINITY ? a.first_hash[x] : 0u;
    };
    struct Request {
        int L, s, n;
        int64_t j0;
        uint32_t hash;
        bool sync;
        double t0, t1;       // arrival of the request after next, at the time scale of each replay of the workgroup
        int O;
    };
    auto settle = [&](int g0, const Scalars& c) {
        Request x;
        const int r = g0 + q;
        const bool on = r < N, has1 = r + 1 < N, has2 = r + 2 < N;       // (requests past the end look empty)
        x.j0 = c.j0;
        x.s = on ? (int)(c.j1 - (uint32_t)c.j0) : 0;
        x.n = on ? (int)(c.b1 - c.b0) : 0;
        x.L = on ? c.L : 0;
        x.hash = c.hash;
        x.O = c.O;
        const double t2 = (double)c.ts2;
        // (nothing completes by the arrival of a request that there is not: the queue wavefront need not ask whether there is
        // one; with two replays the test is the cheaper: 2,048 of 20,000 requests 16.0 / 16.25 ms)
        x.t0 = PACK == 2 || has2 ? t2 * scale0 : -INFINITY;
        x.t1 = t2 * scale1;
        // whether all wavefronts meet once more before the next request: if it has more segments than are preloaded ...
        bool sync = has1 && c.j2 - c.j1 > (uint32_t)SEG_CHUNK;
        // ... if this one may have completed by its arrival -- it takes its decode time at least: every further term of its
        // completion time is added to it and none is negative, and rounding keeps the order ...
        if (SIGNAL) {
            const double t = (double)c.ts0, t1 = (double)c.ts1, dec = least_dec * (double)c.O;
            sync = sync || !(t * scale0 + dec > t1 * scale0);
            if (PACK == 2) sync = sync || !(t * scale1 + dec > t1 * scale1);
        }
        // ... and if the tuner changes the weights after this one
        if (MODE == MODE_ONLINE) sync = sync || (r + 1 >= a.window && (unsigned)(r + 1 - a.window) % (unsigned)a.hop == 0u);
        x.sync = has1 && sync;
        return x;
    };
    int ref_id = -1, ref_end = 0;                    // (-1: no such segment)
    SegRef raw_ref{-1, 0};
    auto load_ref = [&](const Request& c) { raw_ref = a.seg[c.j0 + (k < c.s ? k : 0)]; };   // (one behind the last is there to be read)
    auto settle_ref = [&](const Request& c) {
        ref_id = k < c.s ? raw_ref.id : -1;
        ref_end = k < c.s ? raw_ref.end : 0;         // (with the SEG_FRESH mark)
    };
    int old_id = -1, old_end = 0;                    // the references of the group before
    Touched<PACK> touched;
    Request now;
    Scalars next;
    // The descriptors of group g0 (scalars `now`, references in ref_*), in pieces of about equal length; done(k) is
    // called after each.
    auto commit = [&](int g0, auto done) {
        settle_ref(now);
        // the references at the same place of the path in the three requests before: same tree, same path so far
        const int from1 = ((lane - SEG_CHUNK) & (WAVE - 1)) << 2, from2 = ((lane - 2 * SEG_CHUNK) & (WAVE - 1)) << 2,
                  from3 = ((lane - 3 * SEG_CHUNK) & (WAVE - 1)) << 2;
        int p1_id = __builtin_amdgcn_ds_bpermute(from1, q < 7 ? ref_id : old_id);
        int p1_end = __builtin_amdgcn_ds_bpermute(from1, q < 7 ? ref_end : old_end);
        int p2_id = __builtin_amdgcn_ds_bpermute(from2, q < 6 ? ref_id : old_id);
        int p2_end = __builtin_amdgcn_ds_bpermute(from2, q < 6 ? ref_end : old_end);
        int p3_id = __builtin_amdgcn_ds_bpermute(from3, q < 5 ? ref_id : old_id);
        int p3_end = __builtin_amdgcn_ds_bpermute(from3, q < 5 ? ref_end : old_end);
        done(0);
        const bool real = k < now.s, fresh = real && (ref_end & SEG_FRESH) != 0;
        const int my_end = ref_end & SEG_END_MASK;
        // (a fresh segment may sit in the slot that a request before just gave up)
        const bool same1 = real && !fresh && ref_id == p1_id && my_end == (p1_end & SEG_END_MASK);
        const bool new1 = same1 && (p1_end & SEG_FRESH) != 0;
        const bool same2 = real && !fresh && !new1 && ref_id == p2_id && my_end == (p2_end & SEG_END_MASK);
        const bool new2 = same2 && (p2_end & SEG_FRESH) != 0;
        const uint32_t slot_off = (uint32_t)ref_id * row_bytes;
        const bool same3 = real && !fresh && !new1 && !new2 && ref_id == p3_id && my_end == (p3_end & SEG_END_MASK);
        const bool new3 = same3 && (p3_end & SEG_FRESH) != 0;
        const uint32_t off = real && !fresh && !new1 && !new2 && !new3 ? slot_off : never_off;
        const unsigned long long all1 = ballot(same1), all2 = ballot(same2), all3 = ballot(same3), allf = ballot(fresh);
        done(1);
        SegDesc* const d = &comm->ring[(g0 + q) & (DESC_RING - 1)];
        d->rowoff[k] = off;
        d->end[k] = real ? my_end : now.n;
        d->slot[k] = real ? slot_off : spare_off;
        if constexpr (!APART) {
            // The rows that will be read a dozen requests from now are touched once, so that they come from the L2 then and
            // not from memory: one load per 64 rows (both ends of rows that straddle a cache line, or
            // are longer than one).  The values are only used to keep the loads.
            touched.done();
            touched.rows(rows, off, (row_bytes & 127u) != 0 || row_bytes > 128u ? row_bytes - 4u : 0u, other_replay);
        }
        done(2);
        const int byte = q * SEG_CHUNK;
        const unsigned common1 = __builtin_ctz(~(unsigned)(all1 >> byte) | 0x100u);
        const unsigned common2 = __builtin_ctz(~(unsigned)(all2 >> byte) | 0x100u);
        const unsigned common3 = __builtin_ctz(~(unsigned)(all3 >> byte) | 0x100u);
        const unsigned fresh8 = (unsigned)(allf >> byte) & 0xffu;
        // the last segment's row, if it is fresh: with at most 32 replicas the book-keeping wavefront's upper lanes
        // reset it in the same store
        const bool tail_fresh = (PACK == 1 || APART) && R <= 32 && now.s > 0 && now.s <= SEG_CHUNK && ((fresh8 >> ((now.s - 1) & 31)) & 1u) != 0;
        const uint32_t tail = (uint32_t)__builtin_amdgcn_ds_bpermute((byte + ((now.s - 1) & (SEG_CHUNK - 1))) << 2, (int)slot_off);
        const unsigned rest = fresh8 & ~(tail_fresh ? 1u << (now.s - 1) : 0u);
        const int flags = (now.s > 4 ? DESC_MORE4 : 0) | (now.s > SEG_CHUNK ? DESC_DEEP : 0) | (tail_fresh ? DESC_FRESH_TAIL : 0) |
                          (rest != 0 ? DESC_FRESH_MORE : 0) | (now.sync ? DESC_SYNC : 0) | (int)(common1 << 8) | (int)(common2 << 12) |
                          (int)(common3 << 20) | (int)(__builtin_ctz(fresh8 | 0x100u) << 16);
        done(3);
        if (k == 0) *reinterpret_cast<int4*>(&d->L) = int4{now.L, now.n, now.s, flags};
        if (k == 1) {
            d->j0 = now.j0;
            d->tail = tail_fresh ? tail : spare_off;
            if (MODE == MODE_AFFINITY) d->target = now.s > 0 ? spread(now.hash, R) : 0;
            else if (MODE == MODE_RANDOM)
                d->target = spread(philox4x32_10_first((uint32_t)(g0 + q), 0u, (uint32_t)seed, (uint32_t)(seed >> 32)), R);
        }
        if (k == 2) {
            d->t2[0] = now.t0;
            d->t2[1] = now.t1;
        }
        if (k == 3) {
            d->dec = a_dec * (double)now.O;
            d->O = now.O;
        }
        old_id = ref_id;
        old_end = ref_end;
        done(4);
    };
    const auto at_once = [](int) {};
    for (int g0 = 0; g0 < DESC_AHEAD; g0 += DESC_GROUP) {
        load_scalars(g0, next);
        now = settle(g0, next);
        load_ref(now);
        commit(g0, at_once);
    }
    load_scalars(DESC_AHEAD, next);
    now = settle(DESC_AHEAD, next);
    load_ref(now);
    load_scalars(DESC_AHEAD + DESC_GROUP, next);
    // The row cells of request x, for the deciding wavefront, which reads them from LDS after the next meeting.
    int32_t cell[SEG_CHUNK];
    bool more4 = false;
    auto load_cells = [&](int x) {
        const SegDesc& d = comm->ring[x & (DESC_RING - 1)];
        more4 = (__builtin_amdgcn_readfirstlane(d.flags) & DESC_MORE4) != 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) cell[j] = ld(reinterpret_cast<const int32_t*>(rows + (d.rowoff[j] + lane_off)));
        if (more4) {
#pragma unroll
            for (int j = 4; j < 8; ++j) cell[j] = ld(reinterpret_cast<const int32_t*>(rows + (d.rowoff[j] + lane_off)));
        }
    };
    int set = 0;                                     // the set of cells that the next request gets
    auto store_cells = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j) comm->cells[set][j][lane] = cell[j];
        if (more4) {
#pragma unroll
            for (int j = 4; j < 8; ++j) comm->cells[set][j][lane] = cell[j];
        }
        set = set == CELL_SETS - 1 ? 0 : set + 1;
    };
    load_cells(0);
    store_cells();
    load_cells(1);
    store_cells();
    meet(true);         // the first descriptors and cells are there
    meet(false);
    SectionClock<TIMED> clk;
    clk.start();
    const int every = look_every(R);
    // what is done before the meeting X(r): the cells of r + 2 are loaded, and after a piece of the descriptors' work
    // handed over; every fourth or eighth time the log records that were asked for as well
    unsigned long long raw[PROXY ? 2 : 1] = {};
    auto begin = [&](int r) {
        if (r >= N) return;
        load_cells(r + 2);
        if constexpr (!APART) {
            if ((r & every) == 0 && r > 0)
                for (int c = 0; c < (PROXY ? 2 : 1); ++c) raw[c] = ld(&log64[(int)(unsigned)comm->record[c][lane]]);
        }
    };
    auto pass = [&](int r) {
        if (r >= N) return;
        const bool sync = (__builtin_amdgcn_readfirstlane(comm->ring[r & (DESC_RING - 1)].flags) & DESC_SYNC) != 0;
        store_cells();
        if constexpr (!APART) {
            if ((r & every) == 0 && r > 0)
                for (int c = 0; c < (PROXY ? 2 : 1); ++c) comm->record[c][lane] = raw[c];
        }
        clk.tick(0);                                                 // descriptors, cells
        meet(true);                                                  // X(r)
        if (sync) meet(false);                                       // Y(r)
        clk.tick(1);                                                 // waiting
    };
    for (int r = 0; r < N; r += DESC_GROUP) {
        // (a piece between any two meetings: all at once the work would make the meeting late)
        begin(r);
        commit(r + DESC_AHEAD, [&](int i) {
            pass(r + i);
            begin(r + i + 1);
        });
        now = settle(r + DESC_AHEAD + DESC_GROUP, next);
        load_ref(now);
        pass(r + 5);
        begin(r + 6);
        load_scalars(r + DESC_AHEAD + 2 * DESC_GROUP, next);
        pass(r + 6);
        begin(r + 7);
        pass(r + 7);
    }
    touched.done();
    if (TIMED && a.sections && lane == 0)            // (the book-keeping wavefront writes the next two)
        for (int which = 0; which < (pair ? 2 : 1); ++which)
            for (int i = 0; i < 2; ++i) a.sections[((p + which) * 3 + 2) * SECTIONS + i] = clk.acc[i];
}

// ---------------------------------------------------------------------------------------------- tuner, probe epochs
// Online tuner (Sec. 2.3, Sec. 4), run by the wavefront that has the TTFTs: after every hop the p95
// TTFT of the last `window` requests is the fitness of the weights in use; they replace the parent iff they
// beat it; the step size follows the 1/5 rule; the next offspring is a log-space mutation of the parent.
// The three weights are held by lanes 0 to 2 (the other lanes repeat the third), the rest of the state by every lane.
template <bool ONLINE>
struct Tuner {
    const SegArgs& a;
    const size_t p;
    double* const ring;                 // the window (LDS)
    const int lane, W, H, kth;
    const int wk;                       // the weight of this lane
    const bool there;                   // whether the replay reports
    int ring_pos = 0, until_step, accepted = 0;
    int64_t step = 0;
    bool have_parent = false;
    double ln_par = 0.0, ln_cur = 0.0, f_par = 0.0, sigma = 0.0;
    __device__ __forceinline__ Tuner(const SegArgs& a_, size_t p_, double* ring_, int lane_, bool there_ = true)
        : a(a_), p(p_), ring(ring_), lane(lane_), W(ONLINE ? a_.window : 0), H(ONLINE ? a_.hop : 0), kth((95 * W + 99) / 100),
          wk(lane_ < 3 ? lane_ : 2), there(there_), until_step(W) {
        if (ONLINE) {
            ln_par = ln_cur = a.ln_theta0[3 * p + wk];
            sigma = a.tuner[12];
            if (W + lane < ((W + 7) & ~7)) ring[W + lane] = INFINITY;     // padding (entries below W are written before use)
        }
    }
    __device__ __forceinline__ void results() const {
        if (ONLINE && there) {
            const double best = clip(tuner_exp(ln_par), a.tuner[wk], a.tuner[3 + wk]);
            if (a.theta_final && lane < 3) a.theta_final[3 * p + lane] = best;
            if (a.sigma_final && lane == 0) a.sigma_final[p] = sigma;
            if (a.accepted && lane == 0) a.accepted[p] = accepted;
        }
    }
    // the next request's TTFT; weights: where the weights in use are handed over
    __device__ __forceinline__ void sample(double ttft, double* weights) {
        if (lane == 0) ring[ring_pos] = ttft;
        ring_pos = ring_pos + 1 == W ? 0 : ring_pos + 1;
        if (--until_step == 0) {
            until_step = H;
            wave_sync();
            const double f = window_kth(ring, W, kth, lane);
            if (!have_parent) {
                f_par = f;                 // the first window measures the initial weights: the parent
                have_parent = true;
            } else {
                const bool success = f < f_par;
                if (success) {
                    ln_par = ln_cur;
                    f_par = f;
                    ++accepted;
                }
                sigma = sigma * (success ? a.tuner[13] : a.tuner[14]);
            }
            const double moved = ln_par + sigma * a.z[(p * a.steps + step) * 3 + wk];
            ln_cur = clip(moved, a.tuner[6 + wk], a.tuner[9 + wk]);
            const double th = clip(tuner_exp(ln_cur), a.tuner[wk], a.tuner[3 + wk]);
            if (lane < 3) {
                weights[lane] = th;
                if (a.theta_step && there) a.theta_step[(p * a.steps + step) * 3 + lane] = th;
            }
            if (lane == 0 && a.fitness_step && there) a.fitness_step[p * a.steps + step] = f;
            ++step;
            wave_sync();
        }
    }
};

// Imperfect proxy knowledge (Sec. 2.2, Sec. 4 RTT figure): time is cut into probe epochs, the epoch of t being
// the largest e with e * probe_ms <= t (capped at the last one given); a request experiences the true round
// trip time of its epoch, the cost model scores with the proxy's moving average, handed to the deciding wavefront
// two requests ahead.
template <bool PROXY>
struct ProbeEpochs {
    const SegArgs& a;
    const int lane;
    int epoch = 0;
    double next_probe, rtt_now = 0.0, est_now = 0.0;
    __device__ __forceinline__ ProbeEpochs(const SegArgs& a_, int lane_) : a(a_), lane(lane_), next_probe(PROXY ? (double)a_.probe_ms : 0.0) {}
    // request r arrives at t: half the round trip time of replica = lane.  PACK, which: the estimates go to the lanes of one of two
    // replays.
    template <int PACK = 1, class Comm>
    __device__ __forceinline__ double at(double t, int r, Comm* comm, int which = 0) {
        bool moved = r == 0;
        while (epoch + 1 < a.epochs && next_probe <= t) {       // (timestamps do not decrease)
            ++epoch;
            next_probe = (double)(epoch + 1) * (double)a.probe_ms;
            moved = true;
        }
        if (moved) {
            const size_t x = (size_t)epoch * a.R + (lane < a.R ? lane : 0);
            rtt_now = a.rtt_true[x];
            est_now = a.rtt_est[x];
        }
        if constexpr (PROXY) {
            if (PACK == 1 || lane < HALF) comm->rtt[r & 1][which * HALF + lane] = est_now;
        }
        return 0.5 * rtt_now;
    }
};

// ---------------------------------------------------------------------------------------------- queue side
// Queue wavefront of a replay (`which` of the workgroup's).  One request behind the deciding wavefront: after
// X(r) it serves r, then retires what completes by the arrival of r + 2, which the deciding wavefront reads after
// X(r + 1).  BLOCKS: the partner is the block-table formulation's cache wavefront; the two meet twice at every request
// and the route and hit outputs are written here.
template <int MODE, bool ENGINE, bool PROXY, int PACK, bool BLOCKS, bool TIMED, class Comm>
__device__ __forceinline__ void queue_wave(const SegArgs& a, int which, int lane, unsigned char* lds_raw, Comm* comm) {
    constexpr bool ONLINE = MODE == MODE_ONLINE;
    constexpr bool COUNTS = MODE == MODE_LEAST_REQUEST;      // the load signal is the number of requests, not their tokens
    const int R = a.R, N = (int)a.N;
    const size_t p = (size_t)blockIdx.x * PACK + which;
    SlotQueues Q;
    Q.init(lds_raw, R, a.B, ENGINE, lane);
    Tuner<ONLINE> tuner(a, p, reinterpret_cast<double*>(lds_raw + SlotQueues::bytes(R, a.B, ENGINE)), lane);
    if (N == 0) {           // (an empty trace still reports the tuner's initial state)
        tuner.results();
        return;
    }
    if (ONLINE && lane < 3) comm->w[which][lane] = a.params[3 * p + lane];
    const double sc = a.scale[p];
    ProbeEpochs<PROXY> probes(a, lane);
    const double a_pf = PROXY ? kept(a.a_pf) : 0.0, slowdown = ENGINE ? kept(a.eng_slowdown) : 0.0;
    // proxy variants: half the round trip time of replica = lane, the request in hand's and the next two's
    double half0 = 0.0, half1 = 0.0, half2 = 0.0;
    if constexpr (!PROXY) comm->half[lane] = lane < R ? 0.5 * a.rtt[lane] : 0.0;
    // engine model: this lane's replica has its own rates and KV budget
    const double my_a_pf = ENGINE && lane < R ? a.eng_a_pf[lane] : 0.0;
    const double my_a_dec = ENGINE && lane < R ? a.eng_a_dec[lane] : 0.0;
    const double my_budget = ENGINE && lane < R ? a.eng_budget[lane] : 0.0;
    Rec* const rec = a.rec + p * (size_t)N;

    // ---- times and lengths come with the descriptors; block tables have none: 64 requests per lane-held batch (lane =
    // request), two batches deep so that a batch's loads have a whole batch of time to arrive
    struct Batch {
        double t;        // arrival time, scaled
        int L, O;        // input tokens, output tokens
    };
    auto load_batch = [&](int b0, Batch& b) {
        const int x = b0 + lane;
        const int xx = x < N ? x : N - 1;
        b.t = (double)a.ts[xx] * sc;                 // time scale: gaps scale linearly
        b.L = a.in_len[xx];
        b.O = a.out_len[xx];
    };
    Batch cur{0.0, 0, 0}, nxt{0.0, 0, 0};
    if (BLOCKS) {
        load_batch(0, cur);
        load_batch(WAVE, nxt);
    } else {
        meet(true);      // (the first descriptors are there)
    }
    double* const gone0 = &comm->gone[0][which * HALF];
    auto gone = [&](int r) { return gone0 + (r & 1) * WAVE; };
    for (int b = 0; b < 2; ++b)
        if (PACK == 1 || lane < HALF) gone(b)[lane] = 0.0;
    // requests that complete by t leave the load signal between the arrivals of r - 1 and r
    constexpr bool ASK = BLOCKS || PACK == 2;      // whether there is a next request is asked here
    auto retire = [&](unsigned due, double t, int r) { Q.template retire<!PROXY>(due, t, rec, lane, gone(r)); };
    // arrival times of the request in hand and the two after it
    double t0, t1, t2 = 0.0;
    if (BLOCKS) {
        t0 = readlane_f64(cur.t, 0);
        t1 = readlane_f64(cur.t, 1);
    } else {
        t0 = (double)a.ts[0] * sc;
        t1 = (double)a.ts[N > 1 ? 1 : 0] * sc;
    }
    if (PROXY) {
        half0 = probes.at(t0, 0, comm);
        if (N > 1) half1 = probes.at(t1, 1, comm);
    }
    meet(true);        // (nothing has completed yet: the first request can be decided)

    // What the descriptor of the next request says, read (LDS) while this one's completions are retired: a round trip less
    // before the meeting (64 replays of 50,000 requests 35.4 -> 34.9 ms, 1,024 online tuners of 40,000 32.9 -> 32.0; the
    // proxy variants, whose deciding wavefront has the longer chain, lose 1 % and read it when they need it).
    constexpr bool AHEAD = !BLOCKS && !PROXY;
    struct {
        int L, O, flags;
        double t2, dec;
    } coming{0, 0, 0, 0.0, 0.0};
    auto read_desc = [&](int r) {
        if constexpr (!BLOCKS) {
            const SegDesc& d = comm->ring[r & (DESC_RING - 1)];
            const int4 h = *reinterpret_cast<const int4*>(&d.L);
            coming.L = h.x;
            coming.flags = h.w;
            coming.t2 = d.t2[which];
            if (ENGINE) coming.O = d.O;
            else coming.dec = d.dec;
        }
    };
    if (AHEAD) read_desc(0);

    double o_ttft = 0.0, o_e2e = 0.0;
    int o_route = 0, o_hit = 0, o_believed = 0;
    SectionClock<TIMED> clk;
    clk.start();
    for (int b0 = 0; b0 < N; b0 += WAVE) {
        const int in_batch = N - b0 < WAVE ? N - b0 : WAVE;
        for (int i = 0; i < in_batch; ++i) {
            const int r = b0 + i;
            int L, O = 0;
            double dec = 0.0;
            bool sync = true;
            if (BLOCKS) {
                const int i2 = i + 2;
                L = __builtin_amdgcn_readlane(cur.L, i);
                O = __builtin_amdgcn_readlane(cur.O, i);
                t2 = i2 < WAVE ? readlane_f64(cur.t, i2) : readlane_f64(nxt.t, i2 - WAVE);
                dec = a.a_dec * (double)O;
            } else {
                if (!AHEAD) read_desc(r);
                L = coming.L;
                O = coming.O;
                t2 = coming.t2;
                dec = coming.dec;
                sync = (__builtin_amdgcn_readfirstlane(coming.flags) & DESC_SYNC) != 0;
            }
            clk.tick(0);
            meet(true);                                                  // X(r)
            clk.tick(1);                                                 // waiting at X
            const int lane_best = __builtin_amdgcn_readfirstlane(comm->best[r & 1][which]);
            // (what completes by the arrival of the request after next, or of the next one where it is waited for, this request's
            // own completion aside: read now, while the choice is on its way)
            const double until = sync ? t1 : t2;
            unsigned due = Q.due(until, lane);
            const Choice<PROXY>* const ch = &comm->choice[r & 1][lane_best];
            const double prefill = (double)ch->prefill;
            const int best = PACK == 2 ? lane_best & (HALF - 1) : lane_best;
            double half;
            if constexpr (PROXY) half = readlane_f64(half0, best);
            else half = comm->half[best];
            const int weight = COUNTS ? 1 : L;
            double ttft, e2e;
            if constexpr (ENGINE) {
                Q.template serve_engine<PROXY>(r, best, t0, half, readlane_f64(my_a_pf, best) * prefill,
                                               readlane_f64(my_a_dec, best) * (double)O, weight, (unsigned)L + (unsigned)O,
                                               readlane_f64(my_budget, best), slowdown, rec, lane, &ttft, &e2e, until, due);
            } else {
                Q.template serve<PROXY>(r, best, t0, half, PROXY ? a_pf * prefill : prefill, dec, weight, rec, lane, &ttft, &e2e, until, due);
            }
            clk.tick(9);                                                 // service
            if (AHEAD) read_desc(r + 1);
            o_ttft = lane == i ? ttft : o_ttft;
            o_e2e = lane == i ? e2e : o_e2e;
            if (BLOCKS) {
                o_route = lane == i ? best : o_route;
                o_hit = lane == i ? (int)(ch->hit_end & 0xFFFFu) : o_hit;
                if constexpr (PROXY) o_believed = lane == i ? ch->seen : o_believed;
            }
            if constexpr (ONLINE) tuner.sample(ttft, comm->w[which]);        // (in use from the next request on: Y(r) follows)
            clk.tick(5);                                                 // outputs, tuner
            if (sync) {
                // the request may have completed before the next one arrives, or its latency matters to the next one
                if (!ASK || r + 1 < N) retire(due, t1, r + 1);
                meet(true);                                              // Y(r)
                due = Q.due(t2, lane);
            }
            // The completions up to the arrival of the request after next (this request's among them) do not depend on
            // where the next request goes, whose own completion the deciding wavefront has ruled out, or will wait for.
            if (!ASK || r + 2 < N) {
                retire(due, t2, r + 2);
                if (PROXY) half2 = probes.at(t2, r + 2, comm);
            }
            if (PROXY) {
                half0 = half1;
                half1 = half2;
            }
            t0 = t1;
            t1 = t2;
            clk.tick(2);                                                 // retiring
        }
        // the batch is done: its outputs go out
        if (lane < in_batch) {
            const size_t o = p * N + b0 + lane;
            if (a.ttft) a.ttft[o] = o_ttft;
            if (a.e2e) a.e2e[o] = o_e2e;
            if (BLOCKS) {
                if (a.route) a.route[o] = (uint8_t)o_route;
                if (a.hit) a.hit[o] = (uint16_t)o_hit;
                if (PROXY && a.believed) a.believed[o] = (uint16_t)o_believed;
            }
        }
        if (BLOCKS) {
            cur = nxt;
            load_batch(b0 + 2 * WAVE, nxt);
        }
        clk.tick(6);                                                   // batch turnover
    }
    clk.write(a.sections ? a.sections + (p * 3 + 1) * SECTIONS : nullptr, lane);
    tuner.results();
}

// ---------------------------------------------------------------------------------------------- book-keeping
// Book-keeping wavefront: after X(r) it stores what decision r changes in memory -- the cells of the request's segments
// on the chosen replica, the rows that start over, the log record, its link, the previous owner's suffix -- and keeps
// the routes and hit counts.  Stores that only some lanes have use for are issued by every lane, the others aimed at a
// row and a log record that nothing reads: a plain instruction is cheaper than a branch around it.
template <bool PROXY, int PACK, bool TIMED, class Comm>
__device__ __forceinline__ void book_wave(const SegArgs& a, int lane, Comm* comm) {
    const int R = a.R, N = (int)a.N;
    const bool upper = PACK == 2 && lane >= HALF;
    const int rl = PACK == 2 ? lane & (HALF - 1) : lane;
    const size_t p0 = (size_t)blockIdx.x * PACK, p = p0 + (upper ? 1 : 0);
    const bool in = rl < R;
    const unsigned row_bytes = (unsigned)R * 4u;
    const unsigned spare_row = (unsigned)(a.nseg - 1) * row_bytes;
    const unsigned replay_off = upper ? (unsigned)a.nseg * row_bytes : 0u;
    char* const rows = reinterpret_cast<char*>(a.last + p0 * (size_t)a.nseg * R);
    auto cell_of = [&](uint32_t rowoff, int replica) -> int32_t* {
        return reinterpret_cast<int32_t*>(rows + (rowoff + replay_off + (unsigned)replica * 4u));
    };
    auto cell_at = [&](uint32_t rowoff) -> int32_t* { return cell_of(rowoff, in ? rl : 0); };
    LogRec* const log = a.log + p * ((size_t)N + 1);
    unsigned long long* const log64 = reinterpret_cast<unsigned long long*>(log);
    // the lanes that reset the row of a fresh last segment, and the replica of each
    const bool narrow = PACK == 1 && R <= 32;
    const bool reset_lane = narrow && lane >= 32;
    const int reset_rep = lane - 32 < R ? lane - 32 : R - 1;
    int tail_r = -1;                          // youngest request routed to replica = lane
    int o_route = 0, o_hit = 0, o_seen = 0;
    constexpr int BATCH = WAVE / PACK;
    comm->first[lane] = -1;
    meet(true);                               // the first descriptors are there
    meet(false);
    SectionClock<TIMED> clk;
    clk.start();
    for (int r = 0; r < N; ++r) {
        const SegDesc* const d = &comm->ring[r & (DESC_RING - 1)];
        const uint32_t of_seg = d->slot[rl & (SEG_CHUNK - 1)], of_tail = d->tail;
        const int n = d->n, s = __builtin_amdgcn_readfirstlane(d->s), flags = __builtin_amdgcn_readfirstlane(d->flags);
        clk.tick(2);                                                 // stores
        meet(true);                                                  // X(r)
        clk.tick(3);                                                 // waiting at X
        const int lane_best = comm->best[r & 1][upper ? 1 : 0];
        const Choice<PROXY> c = comm->choice[r & 1][lane_best];
        const int best = PACK == 2 ? lane_best & (HALF - 1) : lane_best;
        const bool is_best = rl == best;
        // every segment of the request is now last touched by r on the chosen replica (lanes k, k + 8, ...: segment k).
        // A segment that this request is the first to reference has taken over a row slot from a segment of the past: its
        // row starts over, never cached except on the chosen replica.  Fresh segments are the last ones of the path;
        // mostly there is one, or none.  With at most 32 replicas the upper lanes do that in the same store; further
        // fresh segments, and any with more replicas or two replays, take a loop of their own.
        {
            const int rep = reset_lane ? reset_rep : best;
            const int32_t val = reset_lane && rep != best ? NEVER_CACHED : r;
            const uint32_t off = reset_lane ? (lane - 32 < R ? of_tail : spare_row) : of_seg;
            st(cell_of(off, rep), val);
        }
        if (flags & (DESC_FRESH_MORE | DESC_DEEP)) {      // (one test on the usual path for the two rare cases)
            const int32_t fresh_cell = is_best ? r : NEVER_CACHED;
            if (flags & DESC_FRESH_MORE) {
                const int first_fresh = (flags >> 16) & 15;
                const int stop = (s < SEG_CHUNK ? s : SEG_CHUNK) - ((flags & DESC_FRESH_TAIL) ? 1 : 0);
                for (int k = first_fresh; k < stop; ++k) {
                    const uint32_t off = d->slot[k];
                    st(cell_at(in ? off : spare_row), fresh_cell);
                }
            }
            if (flags & DESC_DEEP) {
                const int64_t j0 = d->j0;
                for (int j = SEG_CHUNK; j < s; ++j) {
                    const SegRef sr = a.seg[j0 + j];
                    const uint32_t off = (uint32_t)sr.id * row_bytes;
                    if (sr.end & SEG_FRESH) st(cell_at(in ? off : spare_row), fresh_cell);
                    else if (is_best) st(cell_at(off), r);
                }
            }
        }
        st(&log64[r], 0xFFFFFFFFull | ((unsigned long long)n << 48));      // next -1, own 0, n
        st(&log[is_best && tail_r >= 0 ? tail_r : N].next, r);
        st(&log[c.owner >= 0 ? c.owner : N].own, (uint16_t)(c.hit_end >> 16));
        if (ballot(c.owner == OWN_LIST) != 0) {
            // (several previous owners: rare)
            const int count = c.owner == OWN_LIST ? (int)(c.hit_end >> 16) : 0;
            for (int i = 0; ballot(i < count) != 0; ++i)
                if (i < count) {
                    const OwnChange x = comm->changes[r & 1][PACK == 2 && upper ? 1 : 0][i];
                    st(&log[x.owner].own, (uint16_t)x.end);
                }
        }
        if (is_best && tail_r < 0) comm->first[lane] = r;
        tail_r = is_best ? r : tail_r;
        const int slot = r & (BATCH - 1);
        const bool mine = rl == slot;
        o_route = mine ? best : o_route;
        o_hit = mine ? (int)(c.hit_end & 0xFFFFu) : o_hit;
        if constexpr (PROXY) o_seen = mine ? c.seen : o_seen;
        if (slot == BATCH - 1 || r == N - 1) {
            const int x = r - slot + rl;
            if (rl <= slot) {
                const size_t o = p * N + x;
                if (a.route) a.route[o] = (uint8_t)o_route;
                if (a.hit) a.hit[o] = (uint16_t)o_hit;
                if (PROXY && a.believed) a.believed[o] = (uint16_t)o_seen;
            }
        }
        if (flags & DESC_SYNC) meet(false);                          // Y(r)
    }
    if (TIMED && a.sections && lane == 0) {
        a.sections[(p0 * 3 + 2) * SECTIONS + 2] = clk.acc[2];
        a.sections[(p0 * 3 + 2) * SECTIONS + 3] = clk.acc[3];
    }
}

// ---------------------------------------------------------------------------------------------- deciding
template <int MODE, bool ENGINE, bool PROXY, int PACK, bool TIMED, class Comm>
__device__ __forceinline__ void decide_wave(const SegArgs& a, int lane, Comm* comm) {
    constexpr bool ONLINE = MODE == MODE_ONLINE;
    constexpr bool SCORED = MODE == MODE_COST_MODEL || MODE == MODE_ONLINE;
    constexpr bool COUNTS = MODE == MODE_LEAST_REQUEST;
    constexpr bool DICTATED = MODE == MODE_AFFINITY || MODE == MODE_RANDOM;
    const int R = a.R, N = (int)a.N;
    const bool upper = PACK == 2 && lane >= HALF;
    const int rl = PACK == 2 ? lane & (HALF - 1) : lane;
    const size_t p0 = (size_t)blockIdx.x * PACK, p = p0 + (upper ? 1 : 0);
    const bool in = rl < R;
    const int block_tokens = kept(a.block_tokens);
    const double a_pf = kept(a.a_pf);
    double w_rtt = a.params[3 * p + 0], w_prefill = a.params[3 * p + 1], w_queue = a.params[3 * p + 2];
    double my_rtt = !PROXY && in ? a.rtt[rl] : 0.0;              // (proxy variants: comes from the queue wavefront)
    // first product of Eq. 3 (lanes without a replica: a score above any)
    double rtt_term = in ? w_rtt * my_rtt : INFINITY;
    double q = COUNTS && !in ? INFINITY : 0.0;       // load signal of replica = lane (an integer below 2^53, exact in fp64)
    // Proxy variants (Sec. 7: the proxy does not see replica-side eviction): the proxy keeps an index of its own
    // of what it dispatched to each replica, an LRU like the replica's cache but at least as large (or unbounded).
    // It sees the same touches, so it is the same rows read against a second eviction cursor (c2), which lags
    // the replica's; the match yields both prefixes, Eq. 3 scores with the index's.  Ownership is kept for
    // what the index holds, a superset of what is cached, which the replica's eviction walk does not mind:
    // records behind its cursor are never looked at again.  While the index never forgets (or is not used) its
    // cursor stays at the replica's first record and "in the index" means "ever dispatched here".
    const bool own_index = PROXY && a.index_blocks >= 0;
    const int index_cap = PROXY && a.index_blocks > 0 ? (int)a.index_blocks : 0;
    EvictCursor<Comm::LOOK_WORDS> c1, c2;                 // the cache's cursor, the index's cursor
    c1.init(comm->look[0], comm->record[0], R, lane);
    if (PROXY) c2.init(comm->look[PROXY ? 1 : 0], comm->record[PROXY ? 1 : 0], R, lane);
    c1.over = a.C > 0 ? -(int)a.C : INT32_MIN;         // (unbounded)
    c2.over = -index_cap;
    Fresh latest;                             // what the latest decision changes in the log
    unsigned long long went1 = 0, went2 = 0, went3 = 0;  // where the three requests before went (a lane of each replay)

    const char* const rows = reinterpret_cast<const char*>(a.last + p0 * (size_t)a.nseg * R);
    const unsigned row_bytes = (unsigned)R * 4u;
    // this lane's cell of a row; the rows of a workgroup span less than 4 GiB (checked by the host)
    const unsigned lane_off = (upper ? (unsigned)a.nseg * row_bytes : 0u) + (unsigned)(in ? rl : 0) * 4u;
    auto cell_at = [&](uint32_t rowoff) { return reinterpret_cast<const int32_t*>(rows + (rowoff + lane_off)); };
    const int spare = N;                      // the log record behind the last request's
    LogRec* const log = a.log + p * ((size_t)N + 1);
    const unsigned long long* const log64 = reinterpret_cast<const unsigned long long*>(log);

    const int every = look_every(R);
    // the request in hand: row cells of its first eight segments as seen by this lane (= replica), where they end, tokens,
    // blocks, flags; read (LDS) while the minimum of the one before is being found
    int32_t cell[SEG_CHUNK];
    int end[SEG_CHUNK];
    int L = 0, n = 0, word = 0, set = 0;
    auto take = [&](int r, int set) {
        const SegDesc& d = comm->ring[r & (DESC_RING - 1)];
        const int4 h = *reinterpret_cast<const int4*>(&d.L);
#pragma unroll
        for (int k = 0; k < SEG_CHUNK; ++k) cell[k] = comm->cells[set][k][lane];
        const int4 lo = reinterpret_cast<const int4*>(d.end)[0], hi = reinterpret_cast<const int4*>(d.end)[1];
        end[0] = lo.x, end[1] = lo.y, end[2] = lo.z, end[3] = lo.w;
        end[4] = hi.x, end[5] = hi.y, end[6] = hi.z, end[7] = hi.w;
        L = h.x;
        n = h.y;
        word = h.w;       // (the same in every lane; made scalar behind the meeting, where it has arrived)
    };

    SectionClock<TIMED> clk;
    int n_walks = 0;          // statistics: ownership walks
    int before = 0;           // flags of the request before
    meet(true);                               // the first descriptors and cells are there
    take(0, 0);
    meet(true);                               // the queue wavefronts have set themselves up
    clk.start();
    for (int r = 0; r < N; ++r) {
        const SegDesc* const dr = &comm->ring[r & (DESC_RING - 1)];
        const int target = DICTATED ? dr->target : 0;
        const int flags = __builtin_amdgcn_readfirstlane(word);
        double left = DICTATED ? 0.0 : comm->gone[r & 1][lane];      // (read again behind Y(r - 1))
        if constexpr (PROXY) my_rtt = comm->rtt[r & 1][lane];

        // Y(r - 1), as late as this request allows: the match needs only rows that are in hand
        bool behind = (before & DESC_SYNC) != 0;
        auto caught_up = [&]() {
            meet(false);
            behind = false;
            if (!DICTATED) left = comm->gone[r & 1][lane];
            if (ONLINE) {
                w_rtt = comm->w[upper ? 1 : 0][0];
                w_prefill = comm->w[upper ? 1 : 0][1];
                w_queue = comm->w[upper ? 1 : 0][2];
                rtt_term = in ? w_rtt * my_rtt : INFINITY;
            }
        };

        // ---- the rows were loaded before the stores of the three requests before were sure to be there: the leading
        // segments that the paths share get the cells that those requests wrote on their replicas
        auto patch = [&](int32_t& c, int k, int f) {
            c = of_mask(went3) && k < ((f >> 20) & 15) ? r - 3 : c;
            c = of_mask(went2) && k < ((f >> 12) & 15) ? r - 2 : c;
            c = of_mask(went1) && k < ((f >> 8) & 15) ? r - 1 : c;
        };
        if (flags & DESC_SHARED) {
#pragma unroll
            for (int k = 0; k < SEG_CHUNK; ++k) patch(cell[k], k, flags);
        }

        // ---- prefix match: lane = replica.  A request that touches a segment touches all its ancestors,
        // so along the path the cells never increase: first the segments touched after the cursor's
        // request (cached), then those it touched last itself (cached below the cursor position), then
        // older ones (evicted).  The match is max(e_gt, min(cur_k, e_ge)) with e_gt, e_ge the ends of the
        // last segment whose cell is above, respectively not below, the cursor's request.  (Entries past the
        // request's last segment hold the never-cached cell: they change nothing.)
        int e_gt = 0, e_ge = 0;
        int32_t own_gt = -1;        // previous owner of the last segment counted in e_gt
        int e_gt2 = 0, e_ge2 = 0;   // proxy variants: the same against the index's cursor
        int32_t own_gt2 = -1;
        auto compare = [&](int k) {
            const bool gt = cell[k] > c1.cur_r;
            const bool ge = cell[k] >= c1.cur_r;
            e_gt = gt ? end[k] : e_gt;
            own_gt = gt ? cell[k] : own_gt;
            e_ge = ge ? end[k] : e_ge;
            if (PROXY) {
                const bool gt2 = cell[k] > c2.cur_r;
                const bool ge2 = cell[k] >= c2.cur_r;
                e_gt2 = gt2 ? end[k] : e_gt2;
                own_gt2 = gt2 ? cell[k] : own_gt2;
                e_ge2 = ge2 ? end[k] : e_ge2;
            }
        };
        compare(0);
        compare(1);
        compare(2);
        compare(3);
        if (flags & DESC_MORE4) {
            compare(4);
            compare(5);
            compare(6);
            compare(7);
        }
        const int below_cursor = c1.cur_k < e_ge ? c1.cur_k : e_ge;
        const bool some_eq = below_cursor > e_gt;       // blocks of the cursor's own request are matched
        int my_m = some_eq ? below_cursor : e_gt;
        const int below_cursor2 = c2.cur_k < e_ge2 ? c2.cur_k : e_ge2;
        const bool some_eq2 = below_cursor2 > e_gt2;
        int my_seen = PROXY ? (some_eq2 ? below_cursor2 : e_gt2) : 0;       // blocks in the proxy's index (>= my_m)
        // For the ownership update below: where the cached prefix ends on this replica (rounded up to the
        // end of a segment that the cursor's request owns: what lies beyond the cursor is evicted anyway)
        // and whether all cached segments had the same previous owner.  (Proxy variants: the same for the
        // prefix in the index.)
        const int k_end = PROXY ? (some_eq2 ? e_ge2 : e_gt2) : (some_eq ? e_ge : e_gt);
        // (masks over the lanes, put together with scalar instructions: nothing of it is on the chain)
        const unsigned long long by_cursor = PROXY ? ballot(below_cursor2 > e_gt2) : ballot(below_cursor > e_gt);
        const unsigned long long one_owner = (by_cursor & ballot((PROXY ? e_gt2 : e_gt) == 0)) |
                                             (~by_cursor & ballot((PROXY ? own_gt2 : own_gt) == cell[0]));
        clk.tick(1);                                                 // patch, match (and the wait for the rows)
        if (__builtin_expect(behind, 0)) caught_up();
        if (!DICTATED) comm->gone[r & 1][lane] = 0.0;
        clk.tick(4);                                                 // waiting at Y
        unsigned long long in_reach = ~0ull;     // 0: the match went past the preloaded segments
        if (flags & DESC_DEEP) {
            // more than eight segments (rare; memory is up to date behind Y(r - 1)): the rest of the path is read from the
            // trace, eight references at a time, as long as some replica's prefix is still open
            const int64_t j0 = dr->j0;
            const int s = __builtin_amdgcn_readfirstlane(dr->s);
            int pos = end[7];
            bool open = my_m == pos;
            bool open_seen = PROXY && my_seen == pos;
            if (ballot((PROXY ? open_seen : open) && in) != 0) {
                in_reach = 0;
                for (int c0 = 8; c0 < s; c0 += 8) {
                    int32_t more[8];
                    int send[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        more[k] = NEVER_CACHED;
                        send[k] = pos;
                        if (c0 + k < s) {
                            const SegRef sr = a.seg[j0 + c0 + k];
                            send[k] = sr.end & SEG_END_MASK;
                            // (a fresh segment's row still holds what a segment of the past left there)
                            if ((PROXY ? open_seen : open) && in && !(sr.end & SEG_FRESH))
                                more[k] = ld(cell_at((uint32_t)sr.id * row_bytes));
                        }
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        if (c0 + k < s) {
                            const int cnt = cached_in(more[k], pos, send[k], c1.cur_r, c1.cur_k);
                            my_m += open ? cnt : 0;
                            open = open && cnt == send[k] - pos;
                            if (PROXY) {
                                const int cnt_seen = cached_in(more[k], pos, send[k], c2.cur_r, c2.cur_k);
                                my_seen += open_seen ? cnt_seen : 0;
                                open_seen = open_seen && cnt_seen == send[k] - pos;
                            }
                            pos = send[k];
                        }
                    }
                    if (ballot((PROXY ? open_seen : open) && in) == 0) break;
                }
            }
        }
        clk.tick(1);                                                 // a longer path's rows

        // (every fourth or eighth request: the log record asked for the time before has arrived and becomes usable, and the
        // next one is asked for)
        if ((r & every) == every) {
            const int first = comm->first[lane];
            c1.take_pending(*c1.record);
            *c1.record = (unsigned)c1.ask(spare, latest, first);
            if (PROXY) {
                int also = spare;
                if (index_cap > 0) {
                    c2.take_pending(*c2.record);
                    also = c2.ask(spare, latest, first);
                }
                *c2.record = (unsigned)also;
            }
        }
        clk.tick(2);                                                 // log records

        // ---- score (Eq. 3) and lowest-index minimum.  block_tokens * blocks fits: below 2^15 and 2^16.
        int hit_tok = __mul24(block_tokens, my_m);
        hit_tok = hit_tok > L ? L : hit_tok;
        const int my_u = L - hit_tok;
        int my_u_seen = my_u;       // uncached tokens as Eq. 3 sees them
        if (PROXY) {
            int seen_tok = __mul24(block_tokens, own_index ? my_seen : my_m);
            seen_tok = seen_tok > L ? L : seen_tok;
            my_u_seen = L - seen_tok;
        }
        q += left;
        double my_score, my_prefill = (double)my_u;
        if (!ENGINE && !PROXY) my_prefill = a_pf * my_prefill;
        if (SCORED) {
            const double pf = PROXY || ENGINE ? a_pf * (double)my_u_seen : my_prefill;
            const double s_rtt = PROXY ? (in ? w_rtt * my_rtt : INFINITY) : rtt_term;
            const double s_pf = w_prefill * pf;
            const double rtt_and_prefill = s_rtt + s_pf;
            const double qd = a_pf * q;
            const double s_q = w_queue * qd + 0.0;       // (not -0.0: nor is the score then)
            my_score = rtt_and_prefill + s_q;
        } else if (COUNTS) {
            my_score = q;                       // requests in flight
        } else {
            my_score = rl == target ? 0.0 : 1.0;        // the replica is dictated
        }
        // ---- ownership, whatever the choice: the segments this request takes over on the chosen replica stop belonging
        // to their previous requests.  Along the path the previous owners form runs; each run moves its owner's `own` to
        // the end of the run.  Only cached segments matter (evicted ones belong to requests the cursor has passed, or to
        // the cursor request beyond its position).  One previous owner (the usual case) needs no walk.  Its record may wait in a
        // cursor's look-ahead ring: rare where a replica's log is long (the ring holds its oldest records and previous owners are
        // mostly young), usual where a cache holds a dozen requests.  (10,000 requests, 1,024
        // replays, 32 replicas of 700 blocks: 9.0 ms where the walk looked for it, slot after slot, 6.6 so; proxy 14.8, 9.2.)
        const int held = PROXY ? my_seen : my_m;
        const unsigned long long holders = ballot(held > 0);
        const unsigned long long plain = one_owner & in_reach;
        unsigned long long in_ring = ballot(c1.maybe_in_ring(cell[0]));
        if (PROXY) in_ring |= ballot(c2.maybe_in_ring(cell[0]));
        in_ring &= holders & plain;
        const unsigned long long walkers = holders & ~plain;
        const int owner = of_mask(holders & plain) ? cell[0] : -2;
        const unsigned hit_end = (unsigned)my_m | ((unsigned)k_end << 16);
        if constexpr (PROXY) comm->choice[r & 1][lane] = Choice<true>{my_u, own_index ? my_seen : my_m, owner, hit_end};
        else comm->choice[r & 1][lane] = Choice<false>{my_prefill, owner, hit_end};

        // (what is still needed of this request's numbers, and the next one's: its reads are under way during the minimum)
        const int added = n - my_m, also_added = n - my_seen, set_now = set;
        const double tokens = (double)L;
        set = set == CELL_SETS - 1 ? 0 : set + 1;
        take(r + 1, set);

        const unsigned long long bests = argmin_mask<PACK>(my_score, upper);
        if (PACK == 1) comm->best[r & 1][0] = __builtin_ctzll(bests);
        else comm->best[r & 1][upper ? 1 : 0] = upper ? HALF + __builtin_ctz((unsigned)(bests >> 32)) : __builtin_ctz((unsigned)bests);
        const bool is_best = of_mask(bests);
        clk.tick(3);                                                 // score, minimum, announcement
        // (the announcement is on its way through LDS; what follows needs nobody else and gives it the time to arrive)
        latest.r = r;
        latest.owner = is_best ? owner : -2;
        latest.end = k_end;
        latest.count = 0;
        c1.disowned(latest.owner, k_end);
        if (PROXY) c2.disowned(latest.owner, k_end);
        if (__builtin_expect((in_ring & bests) != 0, 0)) {
            if (of_mask(in_ring & bests)) {
                c1.disowned_in_ring(latest.owner, k_end);
                if (PROXY) c2.disowned_in_ring(latest.owner, k_end);
            }
        }
        if (__builtin_expect((walkers & bests) != 0, 0)) {
            // several previous owners, or a prefix longer than the preloaded rows
            ++n_walks;
            bool walking = of_mask(walkers & bests);
            const int cb_r = PROXY ? c2.cur_r : c1.cur_r, cb_k = PROXY ? c2.cur_k : c1.cur_k;
            int run_owner = -1, run_end = 0, vpos = 0;
            // takes one more segment of the path; changed(owner, end) is told of every run that is complete
            auto walk = [&](int32_t at, int to, auto changed) {
                const int cnt = walking ? cached_in(at, vpos, to, cb_r, cb_k) : 0;
                if (cnt > 0) {
                    if (at != run_owner && run_owner >= 0) changed(run_owner, run_end);
                    run_owner = at;
                    run_end = to;
                }
                walking = walking && cnt == to - vpos;
                vpos = to;
            };
            if (in_reach == 0) {
                // from memory, which nobody else writes before X(r) (Y(r - 1))
                auto changed = [&](int of, int to) {
                    st(&log[of].own, (uint16_t)to);
                    c1.disowned_anywhere(of, to);
                    if (PROXY) c2.disowned_anywhere(of, to);
                };
                const int64_t j0 = dr->j0;
                const int s = __builtin_amdgcn_readfirstlane(dr->s);
                for (int j = 0; j < s && ballot(walking) != 0; ++j) {
                    const SegRef sr = a.seg[j0 + j];
                    const int32_t at = walking && !(sr.end & SEG_FRESH) ? ld(cell_at((uint32_t)sr.id * row_bytes)) : NEVER_CACHED;
                    walk(at, sr.end & SEG_END_MASK, changed);
                }
                if (run_owner >= 0) changed(run_owner, run_end);
            } else {
                // from the preloaded rows.  The book-keeping wavefront stores the changes: it may still be at work on the
                // previous request's, which may concern one of these owners.
                OwnChange* const list = comm->changes[r & 1][PACK == 2 && upper ? 1 : 0];
                int count = 0;
                auto changed = [&](int of, int to) { list[count++] = OwnChange{of, to}; };
                const int most = flags & DESC_MORE4 ? SEG_CHUNK : 4;
                for (int k = 0; k < most && ballot(walking) != 0; ++k) {
                    int32_t at = comm->cells[set_now][k][lane];
                    patch(at, k, flags);
                    walk(at, dr->end[k], changed);
                }
                if (run_owner >= 0) changed(run_owner, run_end);
                latest.count = count;
                latest.list = list;
                if (count > 0) {
                    Choice<PROXY>* const mine = &comm->choice[r & 1][lane];
                    mine->owner = OWN_LIST;
                    mine->hit_end = (unsigned)my_m | ((unsigned)count << 16);
                }
                for (int i = 0; ballot(i < count) != 0; ++i)
                    if (i < count) {
                        const OwnChange x = list[i];
                        c1.disowned_anywhere(x.owner, x.end);
                        if (PROXY) c2.disowned_anywhere(x.owner, x.end);
                    }
            }
        }
        const int E = c1.evict_first(is_best ? added : 0);
        // the proxy's index evicts under its own capacity: its cursor walks the same log
        const int E2 = PROXY && index_cap > 0 ? c2.evict_first(is_best ? also_added : 0) : 0;
        unsigned long long more = ballot(E > 0), more2 = PROXY ? ballot(E2 > 0) : 0;
        if (COUNTS) q += is_best ? 1.0 : 0.0;
        else if (!DICTATED) q += is_best ? tokens : 0.0;
        asm volatile("" : "+s"(more), "+v"(q));       // (before the meeting, not after it)
        went3 = went2;
        went2 = went1;
        went1 = bests;
        clk.tick(5);                                                 // ownership, cursor, the next request
        meet(true);                                                  // X(r)
        clk.tick(0);                                                 // waiting at X
        if (more != 0) c1.advance(E, log64, spare, latest, comm->first[lane]);
        if (PROXY && more2 != 0) c2.advance(E2, log64, spare, latest, comm->first[lane]);
        clk.tick(6);                                                 // eviction past the cursor's record
        before = flags;
    }
    if (TIMED) {
        // statistics of the eviction walk, summed over the replicas
        clk.acc[8] = wave_sum_u32((unsigned)c1.n_spot);
        clk.acc[9] = wave_sum_u32((unsigned)c1.n_adv);
        clk.acc[10] = wave_sum_u32((unsigned)c1.n_dead);
        clk.acc[11] = (unsigned)__builtin_amdgcn_readfirstlane(n_walks);
    }
    clk.write(a.sections ? a.sections + p0 * 3 * SECTIONS : nullptr, lane);
}

// One workgroup = one replay, or two neighbouring ones (PACK = 2: at most 32 replicas, one lane per service slot).
// A replay takes its time however few run beside it, so a population that needs a second round takes twice as long.  At most
// 96 vector registers (five wavefronts per SIMD) and what is in LDS hold five workgroups on a CU with 256 slots, 1,280
// replays, and four with 512: every variant, with a tuner window of 128.  (10,000 requests, 1,024 replays of 32 replicas with
// 16 slots, three workgroups on a CU before: engine 15.1 -> 8.0 ms, tuner 15.0 -> 8.1, proxy 14.1 -> 7.8.)
template <int PACK>
constexpr int seg_threads() { return (3 + PACK) * WAVE; }

template <int MODE, bool ENGINE, bool PROXY, int PACK = 1, bool TIMED = false>
__global__ void __launch_bounds__(seg_threads<PACK>(), PACK == 2 ? 6 : 5) replay_segments_kernel(SegArgs a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ Handover<PROXY, PACK, look_words(ENGINE, MODE == MODE_ONLINE, PROXY)> comm;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    unsigned char* const mine = lds_raw + (wave - 1) * replay_queue_lds_bytes(a.R, a.B, ENGINE, MODE == MODE_ONLINE ? a.window : 0);
    if (a.N == 0) {
        if (wave >= 1 && wave <= PACK) queue_wave<MODE, ENGINE, PROXY, PACK, false, TIMED>(a, wave - 1, lane, mine, &comm);
        return;
    }
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);      // the wavefront on the chain goes first at issue
        decide_wave<MODE, ENGINE, PROXY, PACK, TIMED>(a, lane, &comm);
    } else if (wave <= PACK) {
        __builtin_amdgcn_s_setprio(2);
        queue_wave<MODE, ENGINE, PROXY, PACK, false, TIMED>(a, wave - 1, lane, mine, &comm);
    } else if (wave == PACK + 1) {
        __builtin_amdgcn_s_setprio(1);
        book_wave<PROXY, PACK, TIMED>(a, lane, &comm);
    } else {
        front_wave<MODE, PROXY, PACK, TIMED>(a, lane, &comm);
    }
}

}  // namespace gorgo
