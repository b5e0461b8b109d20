// Replay kernel, block formulation over rows of stamps (any trace; where it is taken: make_plan).
//
// As in replay_blocks.h the cache of a replica knows the stamp of the last touch of every block (stamp = request * stride
// + (stride - 1 - position)), a block is cached iff its stamp is not below the replica's threshold, and eviction only raises
// the threshold.  What is looked up differently: between the first and the last request that reference it a block has a row
// slot of its own, the same for every candidate (the loader hands slots on as it does for segments), and a replay keeps a row
// of R stamps per slot.  A stamp is one load, and a request's stamps on a replica are one load instruction per 64
// blocks; no keys, no probes.  A block's first reference (ROW_FRESH) starts its row over; until then its stamps are not
// read, nor on other replicas at the request after it (ROW_NEW_BEFORE), whose match may run beside the reset.
//
// Rows of blocks of the past are gone, so what a logged request still owns is kept with the request: its record has a bit
// per block, cleared when a later request on the replica touches the block.  The eviction cursor takes set bits from the
// record's end and goes on to the next record of the replica that owns anything; records are linked in the order of the
// requests and read ahead, a record per request and replica.
//
// Four wavefronts and two meetings per request: deciding, updating and queue wavefront as in replay_blocks.h, and a
// book-keeping one that writes the records, starts rows over and reads ahead.  A request is one trip to memory: after
// X(r) the updating wavefront reads the chosen replica's stamps and cursor records while the deciding one reads the next
// request's stamps.  What r changes of those is known beforehand: blocks that r has as well (ROW_IN_BEFORE) are cached where r
// went, the others' stamps stay, and the threshold is there at Y(r).
// Bound by the chain of a request, about 1.8 us: the trip to memory, the eviction behind it, the scores and two meetings.
// 65 replays of 3,001 requests on 7 replicas: 23.6 ms with tables, 8.1 with the updating wavefront as the book-keeper, each
// dead record a trip to memory and the chosen replica's stamps read behind Y(r), 6.4 with the eviction record by record and word by
// word and loads waited for between Y(r) and X(r + 1), 5.4 so.  1,024 of 1,000 on 8: 3.2, so 2.7; on 64: 17.9 with tables, 7.5 now.
#pragma once
#include "device_common.h"
#include "internal.h"
#include "replay_blocks.h"
#include "replay_segments.h"

namespace gorgo {

struct RowArgs {
    SegArgs q;               // what the queue wavefront reads, and the model, weights and policy inputs
    const int64_t* blk_off;  // [N+1]
    const uint32_t* ref;     // [T] row slot | ROW_* marks
    int64_t* cells;          // [P][slots][R] stamps
    uint32_t* log;           // [P][N][words]: next request on the replica, blocks | blocks owned << 16, a bit per block
    int64_t slots;
    int32_t words;           // of a record: 2 + one per 32 blocks of the longest request (at most 64)
};

constexpr int ROW_WAVES = 4;
constexpr int ROW_LOOK = 8;          // records read ahead per replica and LRU

// The replicas' LRU state (LDS): the cache's, and the proxy's index's.
//   tau[lru][replica]: eviction threshold.
//   word(replica, lru, ...): cursor request and position (its blocks at that position and beyond are gone), blocks held, and the
// records read ahead that owned something: their number and the records, oldest first.  The updating wavefront takes them out
// before Y(r), the book-keeping one adds them behind it.
constexpr int LRU_CUR_R = 0, LRU_CUR_K = 1, LRU_LIVE = 2, LRU_COUNT = 3, LRU_RING = 4, LRU_WORDS = LRU_RING + ROW_LOOK;
constexpr int LRU_STRIDE = 2 * LRU_WORDS + 1;        // words of a replica (odd: lane = replica meets no bank twice)
struct RowState {
    int64_t* tau;
    int32_t* words;
    int R;
    static __host__ __device__ constexpr size_t bytes(int R) { return (size_t)R * (2 * 8 + LRU_STRIDE * 4) + 4; }
    __device__ __forceinline__ RowState(unsigned char* lds, int R_)
        : tau(reinterpret_cast<int64_t*>(lds)), words(reinterpret_cast<int32_t*>(tau + 2 * R_)), R(R_) {}
    __device__ __forceinline__ int32_t* word(int replica, int lru, int w) const { return words + replica * LRU_STRIDE + lru * LRU_WORDS + w; }
    __device__ __forceinline__ void init(int lane) const {
        for (int i = lane; i < R; i += WAVE)
            for (int j = 0; j < 2; ++j) {
                tau[j * R + i] = 0;
                for (int w = 0; w < LRU_WORDS; ++w) *word(i, j, w) = w == LRU_CUR_R ? -1 : 0;
            }
    }
};
__host__ __device__ inline size_t replay_rows_lds_bytes(int R, int B, bool engine, int window) {
    return ((replay_queue_lds_bytes(R, B, engine, window) + 15) & ~(size_t)15) + RowState::bytes(R);
}

template <bool PROXY>
struct RowHandover : QueueHandover<PROXY> {
    int32_t first_on[WAVE];               // first request on each replica (-1: none yet)
};

// Where a request's blocks are, how many, input tokens, and its first 128 references (lane = block).  Read ahead, the numbers as
// vector loads of the same word by every lane: a scalar load is waited for at the next meeting, as LDS accesses are, and there
// took some 400 cycles of each of the wavefronts' chains.  (Every word that is loaded is used, and no load is under a condition: for
// the register of an unused word, or to merge what is loaded with what is there otherwise, the compiler waits on the spot.)
struct RowRequest {
    int64_t off;
    int n, L;
    uint32_t ref[2];
    int64_t from;                         // as they come from memory
    int to, tokens;                       // (to: its low word)
    __device__ __forceinline__ void ask(const RowArgs& b, int64_t r) {
        uint64_t x = (uint64_t)(r < b.q.N ? r : b.q.N - 1);
        asm("" : "+v"(x));
        from = b.blk_off[x];
        to = reinterpret_cast<const int32_t*>(b.blk_off)[2 * (x + 1)];
        tokens = b.q.in_len[x];
    }
    __device__ __forceinline__ void arrive() {
        off = readlane_i64(from, 0);
        n = __builtin_amdgcn_readfirstlane(to) - (int)off;
        L = __builtin_amdgcn_readfirstlane(tokens);
    }
    __device__ __forceinline__ void read_scalars(const RowArgs& b, int64_t r) {
        ask(b, r);
        arrive();
    }
    // (beyond the request's blocks: the trace's first reference, whose row there is)
    __device__ __forceinline__ void read_refs(const RowArgs& b, int lane) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int k = g * WAVE + lane;
            ref[g] = b.ref[k < n ? off + k : 0];
        }
    }
    // reference k = base + lane (any one for k >= n)
    __device__ __forceinline__ uint32_t at(const RowArgs& b, int base, int lane) const {
        if (base == 0) return ref[0];
        if (base == WAVE) return ref[1];
        return base + lane < n ? b.ref[off + base + lane] : 0u;
    }
};

__device__ __forceinline__ int64_t ld_cell(const int64_t* cells, uint32_t ref, int R, int replica) {
    return ld(reinterpret_cast<const int64_t*>(reinterpret_cast<const char*>(cells) + ((ref & ROW_SLOT) * (uint32_t)R + (uint32_t)replica) * 8u));
}

// Deciding wavefront.  Lane = replica for the first block, the scores and the minimum; lane = block for the match.
template <int MODE, bool ENGINE, bool PROXY>
__device__ __forceinline__ void rows_decide_wave(const RowArgs& b, int p, int lane, const RowState& state, QueueHandover<PROXY>* comm) {
    constexpr bool ONLINE = MODE == MODE_ONLINE;
    constexpr bool SCORED = MODE == MODE_COST_MODEL || MODE == MODE_ONLINE;
    const SegArgs& a = b.q;
    const int R = a.R;
    const int64_t N = a.N;
    const bool in = lane < R;
    const bool two = PROXY && a.index_blocks >= 0;      // the proxy has an index of its own
    const int64_t *const tau1 = state.tau, *const tau2 = state.tau + R;
    state.init(lane);
    double w_rtt = a.params[3 * (size_t)p + 0];
    double w_prefill = a.params[3 * (size_t)p + 1];
    double w_queue = a.params[3 * (size_t)p + 2];
    double q = 0.0;                                               // load signal of replica = lane
    double my_rtt = !PROXY && in ? a.rtt[lane] : 0.0;             // (proxy variants: comes from the queue wavefront)
    const uint64_t seed = MODE == MODE_RANDOM ? a.seeds[p] : 0;
    const int64_t* const cells = b.cells + (size_t)p * (size_t)b.slots * R;

    RowRequest now, next, after;
    now.read_scalars(b, 0);
    now.read_refs(b, lane);
    next.read_scalars(b, 1);
    next.read_refs(b, lane);
    after.ask(b, 2);

    // ---- prefix match of a request on the replicas in `holders`, four at a time.  unread: marks of blocks whose stamps are not
    // there to be read, which are not cached.
    int my_m = 0, my_seen = 0;
    auto match_on = [&](const RowRequest& of, unsigned long long holders, uint32_t unread) {
        const int n = of.n;
        auto match = [&](auto count) {          // the next `count` holders
            constexpr int G = decltype(count)::value;
            int id[G], m1[G], m2[G];
            int64_t t1[G], t2[G];
            bool open1[G], open2[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const bool there = holders != 0;
                id[g] = there ? __builtin_ctzll(holders) : id[0];
                holders &= holders - (there ? 1 : 0);
                t1[g] = tau1[id[g]];
                t2[g] = two ? tau2[id[g]] : t1[g];
                m1[g] = m2[g] = 0;
                open1[g] = there;
                open2[g] = there && two;
            }
            for (int base = 0; base < n; base += 2 * WAVE) {
                // (128 blocks of every replica are asked for before any is looked at)
                int64_t stamp[G][2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t ref = of.at(b, base + h * WAVE, lane);
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        stamp[g][h] = base + h * WAVE < n ? ld_cell(cells, ref, R, id[g]) : -1;
                        stamp[g][h] = (ref & unread) != 0 || base + h * WAVE + lane >= n ? -1 : stamp[g][h];
                    }
                }
                bool more = false;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int left = n - base - h * WAVE;
                    if (left <= 0) break;
                    const int width = left < WAVE ? left : WAVE;
                    const unsigned long long want = width == WAVE ? ~0ull : ((1ull << width) - 1);
                    more = false;
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const unsigned long long got1 = ballot(stamp[g][h] >= t1[g]);
                        const unsigned long long got2 = ballot(stamp[g][h] >= t2[g]);
                        if (open1[g]) {
                            m1[g] += got1 == want ? width : __builtin_ctzll(~got1);
                            open1[g] = got1 == want;
                        }
                        if (open2[g]) {
                            m2[g] += got2 == want ? width : __builtin_ctzll(~got2);
                            open2[g] = got2 == want;
                        }
                        more = more || open1[g] || open2[g];
                    }
                }
                if (!more) break;
            }
#pragma unroll
            for (int g = G - 1; g >= 0; --g) {      // (a repeated first holder is written last)
                my_m = lane == id[g] ? m1[g] : my_m;
                my_seen = lane == id[g] ? m2[g] : my_seen;
            }
        };
        while (holders != 0) {
            const int count = __builtin_popcountll(holders);
            if (count == 1) match(std::integral_constant<int, 1>());
            else if (count == 2) match(std::integral_constant<int, 2>());
            else match(std::integral_constant<int, 4>());
        }
    };
    const unsigned long long all = R >= WAVE ? ~0ull : (1ull << R) - 1;

    meet(true);         // (the queue wavefront has set itself up)
    // (nothing is cached yet: the first request matches nowhere)
    int previous = -1;
    int64_t before[2] = {-1, -1};        // stamps of the first 128 blocks there, from before it was updated
    for (int64_t r = 0; r < N; ++r) {
        const int n = now.n, L = now.L;
        // the replica that the previous request went to was still being updated: its turn now.  The stamps of before serve:
        // what that request touched is cached.
        if (previous >= 0 && n > 0) {
            const int64_t t1 = tau1[previous], t2 = two ? tau2[previous] : t1;
            int m1 = 0, m2 = 0;
            bool open1 = true, open2 = two;
            auto compare = [&](int base, uint32_t ref, int64_t stamp) {
                const bool there = base + lane < n && (ref & ROW_FRESH) == 0, touched = (ref & ROW_IN_BEFORE) != 0;
                const unsigned long long got1 = ballot(there && (touched || stamp >= t1));
                const unsigned long long got2 = ballot(there && (touched || stamp >= t2));
                const int width = n - base < WAVE ? n - base : WAVE;
                const unsigned long long want = width == WAVE ? ~0ull : ((1ull << width) - 1);
                if (open1) m1 += got1 == want ? width : __builtin_ctzll(~got1);
                if (open2) m2 += got2 == want ? width : __builtin_ctzll(~got2);
                open1 = open1 && got1 == want;
                open2 = open2 && got2 == want;
            };
            compare(0, now.ref[0], before[0]);
            if (n > WAVE) compare(WAVE, now.ref[1], before[1]);
            for (int base = 2 * WAVE; base < n && (open1 || open2); base += WAVE) {
                const uint32_t ref = now.at(b, base, lane);
                compare(base, ref, ld_cell(cells, ref, R, previous));
            }
            my_m = lane == previous ? m1 : my_m;
            my_seen = lane == previous ? m2 : my_seen;
        }
        // the next request's first block on every replica, for those that this request does not go to (asked for here: what a path of
        // more than 128 blocks reads above would be waited for together with it)
        const uint32_t ref0 = (uint32_t)__builtin_amdgcn_readlane((int)next.ref[0], 0);
        const int64_t stamp0 = ld_cell(cells, ref0, R, in ? lane : 0);
        // uncached tokens, really and as Eq. 3 sees them (block_tokens * blocks fits: below 2^15 and 2^16)
        int hit_tok = a.block_tokens * my_m;
        hit_tok = hit_tok > L ? L : hit_tok;
        const int my_u = L - hit_tok;
        int seen_tok = a.block_tokens * (two ? my_seen : my_m);
        seen_tok = seen_tok > L ? L : seen_tok;
        const int my_u_seen = L - seen_tok;
        // the replica a baseline policy dictates (Sec. 4): hash of the first block, or a counter-based draw
        int target = 0;
        if (MODE == MODE_AFFINITY) target = n > 0 ? spread(a.first_hash[r], R) : 0;
        else if (MODE == MODE_RANDOM)
            target = spread(philox4x32_10_first((uint32_t)r, (uint32_t)((uint64_t)r >> 32), (uint32_t)seed,
                                                (uint32_t)(seed >> 32)), R);

        // ---- score (Eq. 3), lowest-index minimum; the load signal is kept here, what left it comes from the queue wavefront
        q += comm->gone[r & 1][lane];
        comm->gone[r & 1][lane] = 0.0;
        if constexpr (PROXY) my_rtt = comm->rtt[r & 1][lane];
        double my_score;
        if (SCORED) {
            const double pf = a.a_pf * (double)my_u_seen;
            const double s_rtt = w_rtt * my_rtt;
            const double s_pf = w_prefill * pf;
            const double rtt_and_prefill = s_rtt + s_pf;
            const double qd = a.a_pf * q;
            const double s_q = w_queue * qd;
            my_score = rtt_and_prefill + s_q;
        } else if (MODE == MODE_LEAST_REQUEST) {
            my_score = q;                       // requests in flight
        } else {
            my_score = lane == target ? 0.0 : 1.0;
        }
        const int best = argmin_lanes(my_score, in);
        const int m_best = __builtin_amdgcn_readlane(my_m, best);
        const int seen_best = two ? __builtin_amdgcn_readlane(my_seen, best) : m_best;
        const unsigned u_best = (unsigned)__builtin_amdgcn_readlane(my_u, best);
        q += lane == best ? (MODE == MODE_LEAST_REQUEST ? 1.0 : (double)L) : 0.0;
        if (lane == 0) {
            if constexpr (PROXY) comm->choice[r & 1][best] = Choice<true>{(int)u_best, seen_best, -2, (unsigned)m_best};
            else comm->choice[r & 1][best] = Choice<false>{ENGINE ? (double)(int)u_best : a.a_pf * (double)(int)u_best, -2, (unsigned)m_best};
            comm->best[r & 1][0] = best;
        }
        meet(true);                                                  // X(r): the choice is there

        // ---- the next request, on the replicas that this one does not change
#pragma unroll
        for (int h = 0; h < 2; ++h) before[h] = h * WAVE < next.n ? ld_cell(cells, next.ref[h], R, best) : -1;
        after.arrive();
        after.read_refs(b, lane);
        my_m = my_seen = 0;
        if (r + 1 < N && next.n > 0 && (ref0 & (ROW_FRESH | ROW_NEW_BEFORE)) == 0) {
            const int64_t t1 = in ? tau1[lane] : 0, t2 = two && in ? tau2[lane] : t1;
            unsigned long long holders = ballot(in && stamp0 >= (t2 < t1 ? t2 : t1)) & all;
            match_on(next, holders & ~(1ull << best), ROW_FRESH | ROW_NEW_BEFORE);
        }
        now = next;
        next = after;
        after.ask(b, r + 3);
        previous = best;
        meet(true);                                                  // Y(r): what completes by the next arrival is known
        if (ONLINE) {
            w_rtt = comm->w[0][0];
            w_prefill = comm->w[0][1];
            w_queue = comm->w[0][2];
        }
    }
}

// Updating wavefront: between X(r) and Y(r) it brings the chosen replica up to date.  Lane = block, or word of a record.
template <bool PROXY>
__device__ __forceinline__ void rows_update_wave(const RowArgs& b, int p, int lane, const RowState& state, RowHandover<PROXY>* comm) {
    const SegArgs& a = b.q;
    const int64_t N = a.N;
    const int R = a.R, words = b.words;
    const bool two = PROXY && a.index_blocks >= 0;      // the proxy's own index: a second LRU over the same touches
    const int C1 = (int)a.C, C2 = two ? (int)a.index_blocks : 0;          // (0: it never forgets)
    int64_t* const cells = b.cells + (size_t)p * (size_t)b.slots * R;
    uint32_t* const log = b.log + (size_t)p * (size_t)N * words;
    auto record = [&](int x) { return log + (size_t)((uint64_t)(uint32_t)x * (uint32_t)words); };
    // Records' words, a lane each, the last one first, two loads of as many records as fit a wavefront (8, 4 or 2): blocks are
    // evicted in the order of the lanes.  Past the CU's own cache: bits are cleared by atomics, which are performed behind it.
    const int shift = words <= 16 ? 4 : words <= 32 ? 5 : 6, each = WAVE >> shift, group = (1 << shift) - 1;
    const int place_of = group - (lane & group);      // (beyond the record: reads its last word, which then counts for nothing)
    const int word = place_of < words ? place_of : words - 1;
    auto load_record = [&](int x) { return __hip_atomic_load(record(x >= 0 ? x : 0) + word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    RowRequest now, next;
    now.read_scalars(b, 0);
    now.read_refs(b, lane);
    next.read_scalars(b, 1);
    meet(true);
    for (int64_t r64 = 0; r64 < N; ++r64) {
        const int r = __builtin_amdgcn_readfirstlane((int)r64), n = now.n;
        next.read_refs(b, lane);
        RowRequest after;
        after.ask(b, r64 + 2);
        meet(true);                                                  // X(r): the choice is there
        const int best = __builtin_amdgcn_readfirstlane(comm->best[r & 1][0]);
        auto cell = [&](uint32_t ref) {
            return reinterpret_cast<int64_t*>(reinterpret_cast<char*>(cells) + ((ref & ROW_SLOT) * (uint32_t)R + (uint32_t)best) * 8u);
        };
        auto mine = [&](uint32_t ref, int k) { return k < n && (ref & ROW_FIRST) != 0; };
        // ---- every block of the request becomes (or stays) held, with this request's stamp; the cursors' records are asked
        // for beside the stamps of before
        int64_t old[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) old[h] = h * WAVE < n ? ld(cell(now.ref[h])) : -1;
        struct Cursor {
            int id[2];                       // the cursor's record and those read ahead, by lane
            uint32_t rec[2];
            int r, k, live, count;
            __device__ __forceinline__ int youngest(int each, int shift) const {
                const int j = count < 2 * each - 1 ? count : 2 * each - 1;
                return __builtin_amdgcn_readlane(j < each ? id[0] : id[1], (j & (each - 1)) << shift);
            }
        } c[PROXY ? 2 : 1];
        const bool evicts[2] = {C1 > 0, PROXY && C2 > 0};
        const int mine_of = *state.word(best, 0, lane < 2 * LRU_WORDS ? lane : 0);        // (all the words in one trip to LDS)
#pragma unroll
        for (int i = 0; i < (PROXY ? 2 : 1); ++i)
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                const int j = l * each + (lane >> shift);
                c[i].id[l] = *state.word(best, i, j == 0 ? LRU_CUR_R : LRU_RING + j - 1);
            }
#pragma unroll
        for (int i = 0; i < (PROXY ? 2 : 1); ++i) {
            auto of = [&](int w) { return __builtin_amdgcn_readlane(mine_of, i * LRU_WORDS + w); };
            c[i].r = of(LRU_CUR_R);
            c[i].k = of(LRU_CUR_K);
            c[i].live = of(LRU_LIVE);
            c[i].count = of(LRU_COUNT);
            if (evicts[i])
#pragma unroll
                for (int l = 0; l < 2; ++l) {
                    const int j = l * each + (lane >> shift);
                    c[i].id[l] = j <= c[i].count ? c[i].id[l] : -1;
                    c[i].rec[l] = load_record(c[i].id[l]);
                }
        }
        auto tau_of = [](int x, int k) { return x < 0 ? (int64_t)0 : (int64_t)x * STAMP_STRIDE + (STAMP_STRIDE - k); };
        const int64_t t1 = tau_of(c[0].r, c[0].k), t2 = two ? tau_of(c[PROXY ? 1 : 0].r, c[PROXY ? 1 : 0].k) : t1;
        auto stamp_of = [&](int k) { return (int64_t)r * STAMP_STRIDE + (STAMP_STRIDE - 1 - k); };
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (mine(now.ref[h], h * WAVE + lane)) st(cell(now.ref[h]), stamp_of(h * WAVE + lane));
        // the request that owned a block until now (whether it is still held or not), -2: none
        auto was = [&](uint32_t ref, int k, int64_t stamp) { return mine(ref, k) && (ref & ROW_FRESH) == 0 ? stamp : -1; };
        auto place = [](int64_t stamp) { return (int)(STAMP_STRIDE - 1 - (stamp & (STAMP_STRIDE - 1))); };
        int add1 = 0, add2 = 0;
        auto count = [&](int64_t stamp, bool is_mine, int base) {
            add1 += __builtin_popcountll(ballot(is_mine && stamp < t1));
            if (PROXY) add2 += __builtin_popcountll(ballot(is_mine && stamp < t2));
            // Blocks that the records in hand lose: at the same places of the prompt word by word, else one by one.
            const int x = stamp >= 0 ? (int)(stamp >> 16) : -2, k = place(stamp);
#pragma unroll
            for (int i = 0; i < (PROXY ? 2 : 1); ++i) {
                if (!evicts[i]) continue;
                // (none is younger than the last one read ahead; the cursor may have passed that)
                const int last = c[i].count > 0 ? c[i].youngest(each, shift) : -1, most = last > c[i].r ? last : c[i].r;
                unsigned long long lost = ballot(x <= most && x >= c[i].r && x >= 0);
                while (__builtin_expect(lost != 0, 0)) {
                    const int lead = __builtin_ctzll(lost), of = __builtin_amdgcn_readlane(x, lead);
                    const unsigned long long its = lost & ballot(x == of), even = its & ballot(k == base + lane);
                    const int w = 2 + base / 32, at = place_of;
#pragma unroll
                    for (int l = 0; l < 2; ++l)
                        if (c[i].id[l] == of) c[i].rec[l] &= at == w ? ~(uint32_t)even : at == w + 1 ? ~(uint32_t)(even >> 32) : ~0u;
                    for (unsigned long long odd = its & ~even; odd != 0; odd &= odd - 1) {
                        const int bit = __builtin_amdgcn_readlane(k, __builtin_ctzll(odd));
#pragma unroll
                        for (int l = 0; l < 2; ++l)
                            if (c[i].id[l] == of) c[i].rec[l] &= at == 2 + bit / 32 ? ~(1u << (bit & 31)) : ~0u;
                    }
                    lost &= ~its;
                }
            }
        };
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = h * WAVE + lane;
            old[h] = was(now.ref[h], k, old[h]);
            count(old[h], mine(now.ref[h], k), h * WAVE);
        }
        after.arrive();
        // Blocks that change hands, in the records of their owners: a bit each, and their number.  Mostly the turn of the
        // conversation before owned them, at the same places of its prompt.
        auto disown = [&](int64_t stamp, int base) {
            const int x = (int)(stamp >> 16), k = place(stamp);
            unsigned long long lost = ballot(stamp >= 0 && x < r && k < 32 * (words - 2));
            if (lost == 0) return;
            const int of = __builtin_amdgcn_readlane(x, __builtin_ctzll(lost));
            const unsigned long long even = lost & ballot(x == of && k == base + lane);
            if (lane < 3) {
                // (lanes 0 and 1: two words of bits; lane 2: the number)
                uint32_t* const at = record(of) + (lane == 2 ? 1 : 2 + base / 32 + lane);
                if (lane == 2) __hip_atomic_fetch_sub(at, (uint32_t)__builtin_popcountll(even) << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else if (2 + base / 32 + lane < words)
                    __hip_atomic_fetch_and(at, ~(uint32_t)(even >> (32 * lane)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (of_mask(lost & ~even)) {
                __hip_atomic_fetch_and(record(x) + 2 + k / 32, ~(1u << (k & 31)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_fetch_sub(record(x) + 1, 1u << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        };
        bool disowned = false;
        auto disown_all = [&]() {
            disown(old[0], 0);
            disown(old[1], WAVE);
            disowned = true;
        };
        // (a longer request's other blocks: read, entered and disowned at once)
        for (int base = 2 * WAVE; base < n; base += WAVE) {
            const int k = base + lane;
            const uint32_t ref = now.at(b, base, lane);
            const int64_t stamp = was(ref, k, ld(cell(ref)));
            if (mine(ref, k)) st(cell(ref), stamp_of(k));
            count(stamp, mine(ref, k), base);
            disown(stamp, base);
        }

        // ---- eviction: the cursor takes blocks from the end of its record, then from the records after it, until the LRU fits
        auto evict = [&](auto which, int add, int C) {
            constexpr int i = decltype(which)::value;
            auto& u = c[i];
            const int held = u.live + add;
            int E = C > 0 && held > C ? held - C : 0;
            if (lane == 0) *state.word(best, i, LRU_LIVE) = held - E;
            if (E == 0) return;
            // Blocks are taken lane by lane: a sum over the lanes before says in which the last one is, and lane = bit which bit of that
            // it is.  (Record after record and word after word, on scalars, took 1,700 of the 5,000 cycles of a request.)
            int x = u.r, k = u.k, to = -1, used = 0;       // used: records read ahead that the cursor has come to
            // from the records in `there`; lane of the last block taken, -1: they do not hold E
            auto take = [&](uint32_t rec, int id, bool there, int below) {
                const int have = below < 0 ? 0 : below > 32 ? 32 : below;
                uint32_t bits = there && place_of >= 2 && place_of < words ? rec : 0u;
                bits = have < 32 ? bits & ((1u << have) - 1) : bits;
                const unsigned sum = wave_scan_u32((unsigned)__builtin_popcount(bits));
                const unsigned long long enough = ballot((int)sum >= E), any = ballot(there);
                if (enough != 0) {
                    const int lead = __builtin_ctzll(enough);
                    const uint32_t its = (uint32_t)__builtin_amdgcn_readlane((int)bits, lead);
                    const int left = E - (__builtin_amdgcn_readlane((int)sum, lead) - __builtin_popcount(its));
                    const unsigned long long bit = ballot(lane < 32 && __builtin_popcount(its >> (lane & 31)) >= left);
                    x = __builtin_amdgcn_readlane(id, lead);
                    k = 32 * (group - (lead & group) - 2) + (63 - __builtin_clzll(bit));
                    E = 0;
                    return lead;
                }
                E -= __builtin_amdgcn_readlane((int)sum, WAVE - 1);
                if (any != 0) {
                    const int lead = 63 - __builtin_clzll(any);
                    x = __builtin_amdgcn_readlane(id, lead);
                    k = 0;
                    to = __builtin_amdgcn_readlane((int)rec, lead | group);
                }
                return -1;
            };
#pragma unroll
            for (int l = 0; l < 2; ++l) {
                if (l > 0 && (E == 0 || u.count < each)) break;
                const int j = l * each + (lane >> shift);
                // (the cursor may have passed a record while it was being read)
                const bool there = u.id[l] >= 0 && (j == 0 || u.id[l] > u.r);
                const int lead = take(u.rec[l], u.id[l], there, j == 0 ? u.k - 32 * (place_of - 2) : 32);
                const int last = (l + 1) * each - 1;
                used = lead >= 0 ? l * each + (lead >> shift) : u.count < last ? u.count : last;
            }
            if (__builtin_expect(E > 0, 0)) {
                // further records, one after the other
                if (!disowned) disown_all();
                while (E > 0) {
                    if (used < u.count) {
                        const int id = __builtin_amdgcn_readfirstlane(*state.word(best, i, LRU_RING + used));
                        ++used;
                        if (id <= x) continue;
                        to = id;
                    } else if (x < 0) {
                        to = __builtin_amdgcn_readfirstlane(comm->first_on[best]);
                    }
                    if (to < 0 || to >= r) break;             // cannot happen while E > 0; bounds the loop
                    take(load_record(to), to, lane <= group, 32);
                }
            }
            if (used > 0) {
                const int left = *state.word(best, i, LRU_RING + (lane + used < ROW_LOOK ? lane + used : ROW_LOOK - 1));
                if (lane < ROW_LOOK) *state.word(best, i, LRU_RING + lane) = left;
            }
            if (lane == 0) {
                *state.word(best, i, LRU_CUR_R) = x;
                *state.word(best, i, LRU_CUR_K) = k;
                *state.word(best, i, LRU_COUNT) = u.count - used;
                state.tau[i * R + best] = tau_of(x, k);
            }
        };
        evict(std::integral_constant<int, 0>(), add1, C1);
        if constexpr (PROXY) {
            if (two) evict(std::integral_constant<int, 1>(), add2, C2);
        }
        meet(true);                                                  // Y(r)
        if (!disowned) disown_all();
        now = next;
        next = after;
    }
}

// Book-keeping wavefront: behind X(r) it writes the record of r and its link and starts the rows of r's new blocks over on the
// replicas that r did not go to; behind Y(r) it reads the logs ahead.  Lane = block, or replica.
template <bool PROXY>
__device__ __forceinline__ void rows_book_wave(const RowArgs& b, int p, int lane, const RowState& state, RowHandover<PROXY>* comm) {
    const SegArgs& a = b.q;
    const int64_t N = a.N;
    const int R = a.R, words = b.words;
    const bool evicts[2] = {a.C > 0, PROXY && a.index_blocks > 0};
    int64_t* const cells = b.cells + (size_t)p * (size_t)b.slots * R;
    uint32_t* const log = b.log + (size_t)p * (size_t)N * words;
    auto record = [&](int x) { return log + (size_t)x * words; };
    // lane = replica: the log's latest request; and for either LRU the record to be read next (-1: read to its end), the one
    // being fetched, and what has been added behind it meanwhile
    struct Ahead {
        int fill = -1, pend = -1, link = -1;
        uint32_t raw0 = 0, raw1 = 0;
    } ahead[PROXY ? 2 : 1];
    int tail = -1;
    comm->first_on[lane] = -1;
    RowRequest now, next;
    now.read_scalars(b, 0);
    now.read_refs(b, lane);
    next.read_scalars(b, 1);
    meet(true);
    for (int64_t r64 = 0; r64 < N; ++r64) {
        const int r = __builtin_amdgcn_readfirstlane((int)r64), n = now.n;
        next.read_refs(b, lane);
        RowRequest after;
        after.ask(b, r64 + 2);
        meet(true);                                                  // X(r)
        const int best = __builtin_amdgcn_readfirstlane(comm->best[r & 1][0]);
        int owned = 0;
        for (int base = 0; base < n; base += WAVE) {
            const uint32_t ref = now.at(b, base, lane);
            const unsigned long long bits = ballot(base + lane < n && (ref & ROW_FIRST) != 0);
            owned += __builtin_popcountll(bits);
            if (lane < 2 && 2 + base / 32 + lane < words) st(record(r) + 2 + base / 32 + lane, (uint32_t)(bits >> (32 * lane)));
            // rows that start over: replica by replica, or row by row, whichever is fewer stores
            const bool fresh = base + lane < n && (ref & ROW_FRESH) != 0 && (ref & ROW_FIRST) != 0;
            unsigned long long who = ballot(fresh);
            const uint32_t row = (ref & ROW_SLOT) * (uint32_t)R * 8u;
            auto cell_at = [&](uint32_t off) { return reinterpret_cast<int64_t*>(reinterpret_cast<char*>(cells) + off); };
            if (R <= __builtin_popcountll(who)) {
                if (fresh)
                    for (int i = 0; i < R; ++i)
                        if (i != best) st(cell_at(row + (uint32_t)i * 8u), (int64_t)-1);
            } else {
                for (; who != 0; who &= who - 1) {
                    const uint32_t its = (uint32_t)__builtin_amdgcn_readlane((int)row, __builtin_ctzll(who));
                    if (lane < R && lane != best) st(cell_at(its + (uint32_t)lane * 8u), (int64_t)-1);
                }
            }
        }
        // (with zeros for what is beyond its blocks: the eviction reads whole records)
        if (lane < 2 || (lane >= 2 + (n + WAVE - 1) / WAVE * 2 && lane < words))
            st(record(r) + lane, lane == 0 ? ~0u : lane == 1 ? (uint32_t)n | (uint32_t)owned << 16 : 0u);
        if (lane == best) {
            if (tail >= 0) st(record(tail), (uint32_t)r);
            else comm->first_on[lane] = r;
        }
        after.arrive();
        meet(true);                                                  // Y(r)
#pragma unroll
        for (int i = 0; i < (PROXY ? 2 : 1); ++i) {
            if (!evicts[i]) continue;
            Ahead& u = ahead[i];
            int32_t* const mine = state.word(lane < R ? lane : 0, i, 0);
            const int count = mine[LRU_COUNT];
            u.link = lane == best && u.pend >= 0 && u.pend == tail ? r : u.link;
            u.fill = lane == best && u.fill < 0 ? r : u.fill;
            // the record asked for at the request before has arrived: into the ring if it owns anything and there is room
            const bool space = count < ROW_LOOK;
            const bool have = u.pend >= 0 && lane < R, owns = (u.raw1 >> 16) != 0;
            const bool taken = have && (space || !owns);
            if (have && owns && space) {
                mine[LRU_RING + count] = u.pend;
                mine[LRU_COUNT] = count + 1;
            }
            const int link = u.link > (int)u.raw0 ? u.link : (int)u.raw0;
            u.fill = taken ? link : u.fill;
            u.pend = taken ? -1 : u.pend;
            const bool ask = lane < R && u.pend < 0 && u.fill >= 0;
            if (ask) {
                u.pend = u.fill;
                u.link = -1;
                u.raw0 = __hip_atomic_load(record(u.fill), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                u.raw1 = __hip_atomic_load(record(u.fill) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        tail = lane == best ? r : tail;
        now = next;
        next = after;
    }
}

template <int MODE, bool ENGINE, bool PROXY>
__global__ void __launch_bounds__(ROW_WAVES * WAVE, 4) replay_rows_kernel(RowArgs b) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ RowHandover<PROXY> comm;
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const int p = blockIdx.x;
    if (wave == 2) {
        queue_wave<MODE, ENGINE, PROXY, 1, true, false>(kernel_args<RowArgs>().q, 0, lane, lds_raw, &comm);
    } else if (b.q.N > 0) {
        const RowState state(lds_raw + ((replay_queue_lds_bytes(b.q.R, b.q.B, ENGINE, MODE == MODE_ONLINE ? b.q.window : 0) + 15) & ~(size_t)15),
                             b.q.R);
        if (wave == 0) rows_decide_wave<MODE, ENGINE, PROXY>(kernel_args<RowArgs>(), p, lane, state, &comm);
        else if (wave == 1) rows_update_wave<PROXY>(kernel_args<RowArgs>(), p, lane, state, &comm);
        else rows_book_wave<PROXY>(kernel_args<RowArgs>(), p, lane, state, &comm);
    }
}

}  // namespace gorgo
