// Replay kernels, segment formulation, for launches that leave most of the chip idle: six wavefronts per replay, or eight for two.
//
// A replay is one dependent chain of requests, so a launch of few replays takes as long as one of them.  What
// replay_segments.h does in four wavefronts is here spread over six, which costs a quarter more vector instructions per
// request (the wavefronts read the announcement and the descriptors each for themselves) and shortens the longest of
// the chains: with a replay per SIMD the instructions are what counts, with two per CU or fewer the chain is.  With up to 32 replicas
// half of a wavefront's lanes idle where a lane is a replica: two replays share such wavefronts, in halves, and have a
// serving and a retiring one each (PACK = 2), so that four per CU are resident with the chain little longer.  The state, the
// descriptors and the results are the same.
//   The deciding wavefront only matches, scores, takes the minimum and announces.  Meeting X(r).
//   The evicting wavefront holds the eviction cursors.  After X(r) it moves the one of the replica that r went to, while r + 1
// is being decided against the cursors as they stand in LDS.  That makes no difference to r + 1 unless it matches blocks on
// that replica whose last request is among the oldest the cursor has in hand; then the deciding wavefront waits for it.
//   The serving wavefront serves r (which slot, from when, until when) and has the latencies, hence the tuner.
//   The retiring wavefront keeps the requests in flight: it enters r - 1, and takes from the load signals what completes by
// the arrival of r + 2.  That r itself completes by then is the serving wavefront's business.
//   The book-keeping wavefront stores, and touches what the front end is about to read, so that it comes from the L2: vector
// memory accesses of a wavefront complete in order, and in the front end a row's way from memory would hold up the cells.
//   The front end is the one of replay_segments.h.
// (A fifth wavefront for the cursors alone left the queue wavefront as the longest chain: 64 replays of 20,000 requests on 8
// replicas 14.2 -> 12.7 ms, with its two halves apart 12.0.)
// Meetings as there: X(r) at every request, Y(r) where the descriptor of r says so.
#pragma once
#include "device_common.h"
#include "internal.h"
#include "replay_segments.h"

namespace gorgo {

constexpr int APART_WAVES = 6;
constexpr int APART_LOOK = 16;       // log records of look-ahead kept in LDS per replica and cursor
constexpr int OWN_WALK = -4;         // in Choice::owner: several previous owners, or a path that goes past the preloaded rows

// A request on its way from the serving to the retiring wavefront.
struct Served {
    double done;         // time its completion event reaches the proxy
    int32_t at;          // service slot, -1: it has completed already
    int32_t weight;      // what it takes from the load signal
};
template <bool PROXY, int PACK = 1>
struct ApartHandover : QueueHandover<PROXY> {
    static constexpr bool APART = true;
    int32_t cells[CELL_SETS][SEG_CHUNK][WAVE];    // [request mod 3]: row cells of the request's first eight segments per replica
    unsigned long long look[PROXY ? 2 : 1][APART_LOOK * WAVE];       // rings of the cursors (one slot is always free)
    SegDesc ring[DESC_RING];
    Served served[PACK][2];               // [replay of the workgroup][request mod 2]
    // Where the eviction cursors are, per replica.
    int32_t cur_r[PROXY ? 2 : 1][WAVE];   // request
    uint32_t k_room[WAVE];                // the cache's cursor's position | room << 16
    int32_t cur_k2[PROXY ? WAVE : 1];     // the index's cursor's position
    int32_t hi[WAVE];                     // youngest record in the ring (of either cursor): a request that adds no more than `room`
                                          // blocks, none of them taken from records up to this one, moves no cursor past it
    // Two words that are polled; their waits end.  Both are written by the evicting wavefront between meetings that it comes to by
    // itself: it waits for nobody but at the meetings, and between X(r) and the next one (Y(r), X(r + 1)) it writes `walked` = r, if r
    // has several previous owners, and `evicted` = r at every request.  Who polls for r has passed X(r), which the evicting
    // wavefront has passed then too, and the next meeting cannot be over before the poller has come to it: so the writer is on
    // its way between the two or done.  All wavefronts of a workgroup are resident, and a poller sleeps between two looks.
    int32_t evicted;                      // the cursors are up to date with the requests up to this one
    int32_t walked;                       // a request whose previous owners have been looked up
};

// The replays of a workgroup: one, or two neighbouring ones, lanes 0..31 and 32..63 of the wavefronts that they share.  The last
// workgroup of an odd number has nothing for its upper half: a replay that is not there reads what belongs to the lower one,
// writes nothing but the spare row and log record, and goes nowhere.
template <int PACK>
struct Pair {
    bool upper;          // this lane's replay is the second one
    bool there;          // ... and there is one
    int rl;              // lane within the replay
    size_t p0, p;        // the workgroup's first replay; this lane's
    __device__ __forceinline__ Pair(const SegArgs& a, size_t first, int lane)
        : upper(PACK == 2 && lane >= HALF), there(!upper || first + 1 < (size_t)a.P), rl(PACK == 2 ? lane & (HALF - 1) : lane), p0(first),
          p(first + (upper && there ? 1 : 0)) {}
};
// Replay `which` of a workgroup whose first is p0, for the wavefronts that have one replay each.
template <int PACK>
__device__ __forceinline__ bool pair_has(const SegArgs& a, size_t p0, int which) {
    return PACK == 1 || which == 0 || p0 + 1 < (size_t)a.P;
}
// The sum over the lanes of replay `which` of a workgroup.
template <int PACK>
__device__ __forceinline__ unsigned replay_sum_u32(unsigned x, int which) {
    const int scan = (int)wave_scan_u32(x), lower = __builtin_amdgcn_readlane(scan, HALF - 1), all = __builtin_amdgcn_readlane(scan, WAVE - 1);
    return (unsigned)(PACK == 1 ? all : which == 0 ? lower : all - lower);
}
// What a wavefront of a timed instantiation writes: sections first .. last of `row` for each of the workgroup's replays (a wavefront
// that has both takes its time for both).
template <int PACK, class Clock>
__device__ __forceinline__ void write_sections(const SegArgs& a, size_t p0, int row, int first, int last, const Clock& clk, int lane) {
    if (!a.sections || lane != 0) return;
    for (int which = 0; which < PACK && pair_has<PACK>(a, p0, which); ++which)
        for (int k = first; k <= last; ++k) a.sections[((p0 + which) * 3 + row) * SECTIONS + k] = clk.acc[k];
}

// The compiler moves no access to memory across this.
__device__ __forceinline__ void in_order() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

// ---------------------------------------------------------------------------------------------- evicting
// What the latest request changes in the log, which the book-keeping wavefront is writing at the same time.
struct LogChange {
    int r;               // the request (its own record cannot be loaded yet)
    int tail;            // on the replica it went to: the request it is linked behind (elsewhere no record's number)
    int owner, end;      // ... and the one whose owned suffix now starts at `end`
};
// Eviction cursor of one LRU over a replica's log of routed requests, held by lane = replica: as EvictCursor, but with the
// log's links followed as requests are added.
struct ApartCursor {
    int cur_r = -1, cur_k = 0, cur_own = 0;
    int fill_r = -1;                     // the record to be read next (-1: the log has been read to its end)
    int pend_r = -1, pend_own = -1, pend_link = -1;      // record being fetched, and what has changed in it meanwhile
    unsigned long long raw = 0;          // the record asked for
    unsigned long long* ring = nullptr;  // records packed as r | own << 32 | n << 48, ring_cnt of them from slot ring_head on
    int ring_head = 0, ring_cnt = 0, ring_hi = -1, stock = 0;        // the youngest; blocks they own
    int most = APART_LOOK - 1;           // records that the ring is filled up to,
    int near = 0;                        // once there is room for no more than this many blocks;
    int low = 0;                         // ... and at once when it holds fewer than this
    unsigned long long next = ~0ull;     // the record at ring_head, read at the end of the request before
    int over = 0;                        // blocks this LRU holds beyond its capacity (below 0: room)
    int n_spot = 0, n_adv = 0, n_dead = 0;       // statistics of the timed instantiation

    __device__ __forceinline__ void init(unsigned long long* look, int lane) {
        ring = look + lane;
        for (int k = 0; k < APART_LOOK; ++k) *at(k) = ~0ull;
    }
    __device__ __forceinline__ unsigned long long* at(int k) const { return ring + ((k & (APART_LOOK - 1)) * WAVE); }

    // In the lanes with `who` set, what was asked for has arrived: a record, which is dropped if it owns nothing and else
    // joins the ring.  Straight-line code: lanes with nothing pending go through it unchanged (every lane stores to LDS:
    // those with nothing for the ring into its free slot).
    __device__ __forceinline__ void take_pending(unsigned long long got, bool who = true) {
        const bool have = who && pend_r >= 0;
        const unsigned hi = (unsigned)(got >> 32);
        const int n = (int)(hi >> 16);
        const int own_mem = (int)(hi & 0xFFFFu);
        const int own = pend_own > own_mem ? pend_own : own_mem;
        const bool alive = have && own < n;
        *at(ring_head + ring_cnt) = (unsigned long long)(unsigned)pend_r | ((unsigned long long)((hi & 0xFFFF0000u) | (unsigned)own) << 32);
        ring_cnt += alive ? 1 : 0;
        ring_hi = alive ? pend_r : ring_hi;
        stock += alive ? n - own : 0;
        n_dead += have && !alive ? 1 : 0;
        const int link = (int)(unsigned)got;
        fill_r = have ? (pend_link > link ? pend_link : link) : fill_r;
        pend_r = have ? -1 : pend_r;
    }
    __device__ __forceinline__ void expect(bool want, const LogChange& f) {
        pend_r = want ? fill_r : -1;
        pend_own = fill_r == f.owner ? f.end : -1;
        pend_link = fill_r == f.tail ? f.r : -1;
    }
    // Asks for the next record of the log where the ring has room for it (`spare`, the record behind the log, where
    // there is nothing to fetch).  Called when nothing is pending.  Nothing is read ahead while the cache is far from full: a
    // short log would all be in the ring, and every match on its replica waited for (150 requests of 1,000 replays on 30 replicas
    // of 1,500 blocks 241 -> 199 us).
    __device__ __forceinline__ void ask(const unsigned long long* log64, int spare, const LogChange& f) {
        const bool filling = over + near >= 0;
        low = filling ? APART_LOOK / 4 : 0;
        const bool want = fill_r >= 0 && fill_r != f.r && ring_cnt < most && filling;
        expect(want, f);
        raw = ld(&log64[want ? fill_r : spare]);
    }
    // request f.r is added to the log behind request f.tail, in the lanes with `here` set
    __device__ __forceinline__ void append(bool here, const LogChange& f) {
        fill_r = here && fill_r < 0 ? f.r : fill_r;
        pend_link = here && pend_r == f.tail ? f.r : pend_link;
    }
    // Request `owner`'s owned suffix now starts at `end`, in the lanes concerned (elsewhere a request that is no record's).
    // Returns whether it may be one of the records in the ring: then disowned_in_ring is the call to make as well.
    __device__ __forceinline__ bool disowned(int owner, int end) {
        cur_own = owner == cur_r ? end : cur_own;
        pend_own = owner == pend_r ? end : pend_own;
        return ring_cnt > 0 && owner <= ring_hi;
    }
    // The same for the records in the ring of replica `best`, a lane per slot (all lanes together).  With few requests in a
    // replica's log this is looked for at nearly every request: slot after slot, a trip to LDS each, it was the longest of the
    // chains.  (19 replays on 29 replicas: 292 requests 305 us, so 184; 4,672 4.40 ms, 2.92.)
    __device__ __forceinline__ void disowned_in_ring(int best, int owner, int end, int lane) {
        const int head = __builtin_amdgcn_readlane(ring_head, best), cnt = __builtin_amdgcn_readlane(ring_cnt, best);
        unsigned long long* const slot = ring - lane + best + (lane & (APART_LOOK - 1)) * WAVE;
        const unsigned long long e = *slot;
        const bool it = lane < APART_LOOK && ((lane - head) & (APART_LOOK - 1)) < cnt && (int)(unsigned)e == owner;
        if (it) *slot = (e & ~(0xFFFFull << 32)) | ((unsigned long long)(unsigned)end << 32);
        asm volatile("" ::: "memory");       // (another lane's slot: nothing read before is to be taken for it)
        const unsigned long long found = ballot(it);
        const int own = __builtin_amdgcn_readlane((int)(e >> 32), found != 0 ? __builtin_ctzll(found) : 0) & 0xFFFF;
        stock -= found != 0 && lane == best ? end - own : 0;
    }
    // takes up to E blocks from the owned suffix of the cursor's record
    __device__ __forceinline__ void take_from_cursor(int& E) {
        int avail = cur_k - cur_own;
        avail = avail > 0 ? avail : 0;
        const int take = avail < E ? avail : E;
        cur_k -= take;
        E -= take;
    }
    // the cursor moves on to record e, the one at ring_head, in the lanes with `go` set
    __device__ __forceinline__ void step_to(unsigned long long e, bool go) {
        const unsigned hi = (unsigned)(e >> 32);
        n_adv += go ? 1 : 0;
        cur_r = go ? (int)(unsigned)e : cur_r;
        cur_k = go ? (int)(hi >> 16) : cur_k;
        cur_own = go ? (int)(hi & 0xFFFFu) : cur_own;
        stock -= go ? (int)(hi >> 16) - (int)(hi & 0xFFFFu) : 0;
        ring_head += go ? 1 : 0;
        ring_cnt -= go ? 1 : 0;
    }
    // `added` blocks have joined the LRU: what the cursor's own record can give up, then the next one (read ahead), then
    // further ones.
    __device__ __forceinline__ void evict(int added, const unsigned long long* log64, int spare, const LogChange& f) {
        over += added;
        int E = over > 0 ? over : 0;
        over -= E;
        take_from_cursor(E);
        if (ballot(E > 0) != 0) {
            step_to(next, E > 0 && ring_cnt > 0);
            take_from_cursor(E);             // (lanes with E = 0 take nothing)
            if (__builtin_expect(ballot(E > 0) != 0, 0)) advance(E, log64, spare, f);
        }
    }
    __device__ __forceinline__ void look_ahead() { next = *at(ring_head); }
    // The cursor moves on to further records until E blocks have been given up (all lanes together, those with
    // nothing to evict unchanged): records come from the ring, and from memory on the spot when the ring has run
    // out.  Works on a copy of the state, written back at the end: the request loop's common path, which does not
    // come here, then carries no register copies for this loop's sake.
    __device__ __forceinline__ void advance(int E_in, const unsigned long long* log64, int spare, const LogChange& f) {
        ApartCursor w = *this;
        int E = E_in;
        w.advance_loop(E, log64, spare, f);
        *this = w;
    }
    __device__ __forceinline__ void advance_loop(int& E, const unsigned long long* log64, int spare, const LogChange& f) {
        do {
            const bool empty = E > 0 && ring_cnt == 0;
            if (ballot(empty) != 0) {
                if (ballot(empty && pend_r >= 0) != 0) {             // what has been asked for is on its way
                    take_pending(raw, empty);
                    continue;
                }
                // (no record, or the latest request's own, whose blocks are the last to go: cannot happen while blocks are
                // to be evicted; bounds the loop)
                const bool stuck = empty && (fill_r < 0 || fill_r == f.r);
                const bool fetch = empty && !stuck;
                E = stuck ? 0 : E;
                const unsigned long long got = ld(&log64[fetch ? fill_r : spare]);
                if (fetch) expect(true, f);
                n_spot += fetch ? 1 : 0;
                take_pending(got, fetch);
                continue;
            }
            step_to(*at(ring_head), E > 0);
            take_from_cursor(E);
        } while (ballot(E > 0) != 0);
    }
    // blocks that may join before the cursor passes the last record of the ring (saturated: a request has fewer than 2^16)
    __device__ __forceinline__ unsigned room() const {
        const int avail = cur_k - cur_own;
        const unsigned x = (unsigned)(stock + (avail > 0 ? avail : 0)) + (unsigned)(0 - over);
        return x < 0xFFFFu ? x : 0xFFFFu;
    }
};

template <bool PROXY, int PACK, bool TIMED, class Comm>
__device__ __forceinline__ void apart_evict_wave(const SegArgs& a, size_t p0, int lane, Comm* comm) {
    const int R = a.R, N = (int)a.N;
    const Pair<PACK> mine(a, p0, lane);
    const unsigned row_bytes = (unsigned)R * 4u;
    const unsigned spare_row = (unsigned)(a.nseg - 1) * row_bytes;
    LogRec* const log = a.log + mine.p * ((size_t)N + 1);
    const unsigned long long* const log64 = reinterpret_cast<const unsigned long long*>(log);
    const int spare = N;                      // the log record behind the last request's
    int tail_r = -1;                          // youngest request routed to replica = lane
    const int index_cap = PROXY && a.index_blocks > 0 ? (int)a.index_blocks : 0;
    const bool bounded = a.C > 0, forgets = PROXY && index_cap > 0;
    ApartCursor c1, c2;                       // the cache's, the index's
    c1.init(comm->look[0], lane);
    c1.over = bounded ? -(int)a.C : -INT32_MAX;
    if (PROXY) {
        c2.init(comm->look[PROXY ? 1 : 0], lane);
        c2.over = forgets ? -index_cap : -INT32_MAX;
    }
    c1.most = c2.most = a.look;
    c1.near = c2.near = a.near;
    const int every = look_every(R);
    int n_walks[PACK] = {};
    // (the deciding wavefront may look in between: `hi` is written first and read last.  LDS performs a wavefront's accesses in their
    // order, so relaxed ones that the compiler keeps in order will do)
    auto publish = [&]() {
        const unsigned room1 = c1.room(), room2 = PROXY ? c2.room() : room1;
        st(&comm->hi[lane], PROXY && c2.ring_hi > c1.ring_hi ? c2.ring_hi : c1.ring_hi);
        in_order();
        st(&comm->cur_r[0][lane], c1.cur_r);
        st(&comm->k_room[lane], (uint32_t)c1.cur_k | (room2 < room1 ? room2 : room1) << 16);
        if constexpr (PROXY) {
            st(&comm->cur_r[1][lane], c2.cur_r);
            st(&comm->cur_k2[lane], c2.cur_k);
        }
        in_order();
    };
    publish();
    st(&comm->evicted, -1);
    st(&comm->walked, -1);
    meet(true);                               // the first descriptors are there
    meet(true);
    SectionClock<TIMED> clk;
    clk.start();
    for (int r = 0; r < N; ++r) {
        const SegDesc* const d = &comm->ring[r & (DESC_RING - 1)];
        const int n = d->n, s = __builtin_amdgcn_readfirstlane(d->s), flags = __builtin_amdgcn_readfirstlane(d->flags);
        clk.tick(4);                                                 // cursors
        meet(true);                                                  // X(r)
        clk.tick(5);                                                 // waiting at X
        const int best = PACK == 1 ? __builtin_amdgcn_readfirstlane(comm->best[r & 1][0]) : comm->best[r & 1][mine.upper ? 1 : 0];
        const Choice<PROXY> c = comm->choice[r & 1][lane];           // (of this lane's replica: no second trip to LDS)
        const bool is_best = lane == best && mine.there;
        int owner = is_best ? c.owner : spare;
        const int end = (int)(c.hit_end >> 16);
        for (unsigned long long walks = ballot(owner == OWN_WALK); __builtin_expect(walks != 0, 0); walks &= walks - 1) {
            // The segments that this request takes over on the chosen replica have several previous owners: along the path
            // these form runs; each run moves its owner's `own` to the end of the run.  Only what is held matters (what is
            // evicted belongs to requests the cursor has passed, or to the cursor's request beyond its position).  The rows are
            // read as they still are: the book-keeping wavefront waits.
            const int of_lane = __builtin_ctzll(walks);                  // (of either replay)
            const bool second = PACK == 2 && of_lane >= HALF;
            n_walks[0] += second ? 0 : 1;
            n_walks[PACK - 1] += second ? 1 : 0;
            const size_t its_p = p0 + (second ? 1 : 0);
            LogRec* const its_log = a.log + its_p * ((size_t)N + 1);
            const char* const cells = reinterpret_cast<const char*>(a.last + its_p * (size_t)a.nseg * R) + (second ? of_lane - HALF : of_lane) * 4;
            const int cb_r = __builtin_amdgcn_readlane(PROXY ? c2.cur_r : c1.cur_r, of_lane);
            const int cb_k = __builtin_amdgcn_readlane(PROXY ? c2.cur_k : c1.cur_k, of_lane);
            int run_owner = -1, run_end = 0, vpos = 0;
            bool walking = true;
            auto changed = [&](int of, int to) {
                st(&its_log[of].own, (uint16_t)to);
                const int its = lane == of_lane ? of : spare;
                if (ballot(c1.disowned(its, to)) != 0) c1.disowned_in_ring(of_lane, of, to, lane);
                if (PROXY) {
                    if (ballot(c2.disowned(its, to)) != 0) c2.disowned_in_ring(of_lane, of, to, lane);
                }
            };
            // (lane = segment: one load for the references, one for the cells)
            const int64_t j0 = d->j0;
            for (int j = 0; j < s && walking; j += WAVE) {
                const SegRef sr = a.seg[j0 + (j + lane < s ? j + lane : s - 1)];
                const bool fresh = (sr.end & SEG_FRESH) != 0;
                const int32_t cell = ld(reinterpret_cast<const int32_t*>(cells + (fresh ? spare_row : (uint32_t)sr.id * row_bytes)));
                const int my_at = fresh ? NEVER_CACHED : cell, my_to = sr.end & SEG_END_MASK;
                for (int k = 0; k < WAVE && j + k < s && walking; ++k) {
                    const int at = __builtin_amdgcn_readlane(my_at, k), to = __builtin_amdgcn_readlane(my_to, k);
                    const int cnt = cached_in(at, vpos, to, cb_r, cb_k);
                    if (cnt > 0) {
                        if (at != run_owner && run_owner >= 0) changed(run_owner, run_end);
                        run_owner = at;
                        run_end = to;
                    }
                    walking = cnt == to - vpos;
                    vpos = to;
                }
            }
            if (run_owner >= 0) changed(run_owner, run_end);
            owner = lane == of_lane ? spare : owner;
            c1.look_ahead();
            if (PROXY) c2.look_ahead();
            if (PACK == 2 && (walks & (walks - 1)) != 0) continue;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            st(&comm->walked, (int32_t)r);
        }
        if (bounded) {
            const LogChange f{r, is_best ? tail_r : N, owner, end};
            c1.append(is_best, f);
            const bool in_ring = c1.disowned(owner, end);
            bool in_ring2 = false;
            if (PROXY) {
                c2.append(is_best, f);
                in_ring2 = c2.disowned(owner, end);
            }
            const unsigned long long rings = ballot(in_ring || in_ring2);
            if (__builtin_expect(rings != 0, 0)) {
                for (unsigned long long left = rings; left != 0; left &= left - 1) {         // (one of either replay)
                    const int x = __builtin_ctzll(left);
                    const int of = __builtin_amdgcn_readlane(owner, x), to = __builtin_amdgcn_readlane(end, x);
                    if ((ballot(in_ring) >> x & 1) != 0) c1.disowned_in_ring(x, of, to, lane);
                    if (PROXY) {
                        if ((ballot(in_ring2) >> x & 1) != 0) c2.disowned_in_ring(x, of, to, lane);
                    }
                }
                c1.look_ahead();
                if (PROXY) c2.look_ahead();
            }
            c1.evict(is_best ? n - (int)(c.hit_end & 0xFFFFu) : 0, log64, spare, f);
            if constexpr (PROXY) {
                if (forgets) c2.evict(is_best ? n - c.seen : 0, log64, spare, f);
            }
            publish();
            st(&comm->evicted, (int32_t)r);
            // (records arrive every so often for all replicas, and whenever a request goes to one whose ring has run low)
            if ((r & every) == every || ballot(is_best && c1.ring_cnt < c1.low) != 0) {
                c1.take_pending(c1.raw);
                c1.ask(log64, spare, f);
                if (PROXY && forgets) {
                    c2.take_pending(c2.raw);
                    c2.ask(log64, spare, f);
                }
            }
            c1.look_ahead();
            if (PROXY) c2.look_ahead();
            tail_r = is_best ? r : tail_r;
        } else {
            st(&comm->evicted, (int32_t)r);
        }
        if (flags & DESC_SYNC) meet(true);                           // Y(r)
    }
    if (TIMED) {
        write_sections<PACK>(a, p0, 2, 4, 5, clk, lane);
        // statistics of the eviction walk, summed over the replicas
        for (int which = 0; which < PACK; ++which) {
            const unsigned spot = replay_sum_u32<PACK>((unsigned)c1.n_spot, which), adv = replay_sum_u32<PACK>((unsigned)c1.n_adv, which),
                           dead = replay_sum_u32<PACK>((unsigned)c1.n_dead, which);
            if (a.sections && lane == 0 && pair_has<PACK>(a, p0, which)) {
                unsigned long long* const out = a.sections + (p0 + which) * 3 * SECTIONS;
                out[8] = spot;
                out[9] = adv;
                out[10] = dead;
                out[11] = (unsigned)n_walks[which];
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------- book-keeping
// As book_wave of replay_segments.h; also touches, eight requests at a time, the rows and the lines of the trace that the front
// end is going to read.  (Loads whose values only keep them: this wavefront waits for none.)
template <bool PROXY, int PACK, bool TIMED, class Comm>
__device__ __forceinline__ void apart_book_wave(const SegArgs& a, size_t p0, int lane, Comm* comm) {
    const int R = a.R, N = (int)a.N;
    const Pair<PACK> pair(a, p0, lane);
    const bool in = pair.rl < R && pair.there;
    const unsigned row_bytes = (unsigned)R * 4u;
    const unsigned spare_row = (unsigned)(a.nseg - 1) * row_bytes;
    const unsigned other_replay = PACK == 2 && pair_has<PACK>(a, p0, 1) ? (unsigned)a.nseg * row_bytes : 0u;
    const unsigned replay_off = pair.upper ? other_replay : 0u;
    char* const rows = reinterpret_cast<char*>(a.last + p0 * (size_t)a.nseg * R);
    auto cell_of = [&](uint32_t rowoff, int replica) -> int32_t* {
        return reinterpret_cast<int32_t*>(rows + (rowoff + replay_off + (unsigned)replica * 4u));
    };
    auto cell_at = [&](uint32_t rowoff) -> int32_t* { return cell_of(rowoff, in ? pair.rl : 0); };
    LogRec* const log = a.log + pair.p * ((size_t)N + 1);
    unsigned long long* const log64 = reinterpret_cast<unsigned long long*>(log);
    // the lanes that reset the row of a fresh last segment, and the replica of each (two replays: a store of its own)
    const bool reset_lane = PACK == 1 && R <= 32 && lane >= 32;
    const int reset_rep = lane - 32 < R ? lane - 32 : R - 1;
    int tail_r = -1;                          // youngest request routed to replica = lane
    int o_route = 0, o_hit = 0, o_seen = 0;
    Touched<PACK> touched;
    constexpr int BATCH = WAVE / PACK;
    const bool wide = (row_bytes & 127u) != 0 || row_bytes > 128u;      // (rows that straddle a cache line, or are longer)
    const int64_t refs = a.seg_off[N];
    // (a lane per array; a group of eight requests is 32 or 64 bytes of each; one reference behind the last is there to be read)
    // (the arrays' addresses by value: a lane would otherwise pick the argument that it loads its address from, and arguments
    // that a workgroup has worked out would have to lie in memory)
    auto value = [](const void* of) {
        uint64_t x = reinterpret_cast<uint64_t>(of);
        asm("" : "+s"(x));
        return x;
    };
    const uint64_t at0 = value(a.ts), at1 = value(a.seg_off), at2 = value(a.blk_off), at3 = value(a.in_len), at4 = value(a.out_len),
                   at5 = value(a.seg);
    const uint64_t my_array = lane >= 5 && lane < 21 ? at5 : lane == 4 ? at4 : lane == 3 ? at3 : lane == 2 ? at2 : lane == 1 ? at1 : at0;
    const int log_size = lane == 3 || lane == 4 ? 2 : 3;
    static_assert(sizeof(SegRef) == 8);
    auto touch_trace = [&](int x, int64_t j0) {
        const int64_t j = j0 + (lane - 4) * 16, k = lane >= 5 && lane < 21 ? (j < refs ? j : refs) : x < N ? x : N - 1;
        // (a load from global memory: a flat one counts as an access to LDS as well, and the next meeting would wait for it)
        return ld(reinterpret_cast<const __attribute__((address_space(1))) int32_t*>(my_array + ((uint64_t)k << log_size)));
    };
    meet(true);                               // the first descriptors are there
    meet(true);
    SectionClock<TIMED> clk;
    clk.start();
    for (int r = 0; r < N; ++r) {
        const SegDesc* const d = &comm->ring[r & (DESC_RING - 1)];
        const uint32_t of_seg = PACK == 1 || pair.there ? d->slot[lane & (SEG_CHUNK - 1)] : spare_row, of_tail = d->tail;
        const int n = d->n, s = __builtin_amdgcn_readfirstlane(d->s), flags = __builtin_amdgcn_readfirstlane(d->flags);
        clk.tick(2);                                                 // stores
        meet(true);                                                  // X(r)
        clk.tick(3);                                                 // waiting at X
        const int lane_best = comm->best[r & 1][pair.upper ? 1 : 0];
        const Choice<PROXY> c = comm->choice[r & 1][lane];           // (of this lane's replica: no second trip to LDS)
        const int best = PACK == 2 ? lane_best & (HALF - 1) : lane_best;
        const bool is_best = lane == lane_best && pair.there;
        // (several previous owners: the evicting wavefront looks them up in the rows as they still are, and stores the changes)
        if (__builtin_expect(ballot(is_best && c.owner == OWN_WALK) != 0, 0))
            while (ld(&comm->walked) < r) __builtin_amdgcn_s_sleep(1);
        // every segment of the request is now last touched by r on the chosen replica (lanes k, k + 8, ...: segment k); fresh ones
        // start over (see book_wave)
        {
            const int rep = reset_lane ? reset_rep : best;
            const int32_t val = reset_lane && rep != best ? NEVER_CACHED : r;
            const uint32_t off = reset_lane ? (lane - 32 < R ? of_tail : spare_row) : of_seg;
            st(cell_of(off, rep), val);
            if (PACK == 2) st(cell_at(in ? of_tail : spare_row), is_best ? r : NEVER_CACHED);
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
        st(&log[is_best && c.owner >= 0 ? c.owner : N].own, (uint16_t)(c.hit_end >> 16));
        tail_r = is_best ? r : tail_r;
        if ((r & (DESC_GROUP - 1)) == 3) {
            // (the rows of the eight requests from the next multiple of eight on: their descriptors are there but for the last words)
            touched.done();
            const SegDesc& x = comm->ring[((r & ~(DESC_GROUP - 1)) + DESC_AHEAD + lane / SEG_CHUNK) & (DESC_RING - 1)];
            const uint32_t off = x.rowoff[lane % SEG_CHUNK];
            touched.rows(rows, off, wide ? row_bytes - 4u : 0u, other_replay);
            touched.also = touch_trace(r + 5 * DESC_GROUP, d->j0);
        }
        const int slot = r & (BATCH - 1);
        const bool mine = pair.rl == slot;
        auto of_best = [&](int x) {
            const int a = __builtin_amdgcn_readlane(x, __builtin_amdgcn_readfirstlane(lane_best));
            if (PACK == 1) return a;
            const int b = __builtin_amdgcn_readlane(x, __builtin_amdgcn_readlane(lane_best, WAVE - 1));
            return pair.upper ? b : a;
        };
        const int hit = of_best((int)(c.hit_end & 0xFFFFu));          // (by all lanes together)
        o_route = mine ? best : o_route;
        o_hit = mine ? hit : o_hit;
        if constexpr (PROXY) {
            const int seen = of_best(c.seen);
            o_seen = mine ? seen : o_seen;
        }
        if (slot == BATCH - 1 || r == N - 1) {
            const int x = r - slot + pair.rl;
            if (pair.rl <= slot && pair.there) {
                const size_t o = pair.p * N + x;
                if (a.route) a.route[o] = (uint8_t)o_route;
                if (a.hit) a.hit[o] = (uint16_t)o_hit;
                if (PROXY && a.believed) a.believed[o] = (uint16_t)o_seen;
            }
        }
        if (flags & DESC_SYNC) meet(false);                          // Y(r)
    }
    touched.done();
    if (TIMED) write_sections<PACK>(a, p0, 2, 2, 3, clk, lane);
}

// ---------------------------------------------------------------------------------------------- retiring
// Retiring wavefront: the lists of requests in flight (all of SlotQueues but the times the slots become free).  After X(r)
// it enters r - 1, which has not completed by the arrival of r + 1 (else the serving wavefront has dealt with it), and retires
// what completes by the arrival of r + 2, r itself aside.
template <bool PROXY, int PACK, bool TIMED, class Comm>
__device__ __forceinline__ void apart_retire_wave(const SegArgs& a, size_t p0, int which, int lane, SlotQueues& Q, Comm* comm) {
    const int N = (int)a.N;
    const size_t p = p0 + (pair_has<PACK>(a, p0, which) ? which : 0);       // (one that is not there is served, but never enters)
    Rec* const rec = a.rec + p * N;
    const double sc = a.scale[p];
    if (lane == 0) comm->served[which][1].at = -1;   // (there is nothing before the first request)
    meet(true);                               // the first descriptors are there
    double t1 = (double)a.ts[N > 1 ? 1 : 0] * sc;
    meet(true);
    auto retire = [&](unsigned due, double t, int r) { Q.template retire<!PROXY>(due, t, rec, lane, &comm->gone[r & 1][which * HALF]); };
    SectionClock<TIMED> clk;
    clk.start();
    for (int r = 0; r < N; ++r) {
        const SegDesc& d = comm->ring[r & (DESC_RING - 1)];
        const bool sync = (__builtin_amdgcn_readfirstlane(d.flags) & DESC_SYNC) != 0;
        const double t2 = d.t2[which];
        clk.tick(2);                                                 // retiring
        meet(true);                                                  // X(r)
        clk.tick(3);                                                 // waiting at X
        const Served x = comm->served[which][(r - 1) & 1];
        const int at = __builtin_amdgcn_readfirstlane(x.at);
        if (at >= 0) Q.template enter<PROXY>(at, r - 1, x.done, x.weight, rec, lane);
        if (sync) {
            retire(Q.due(t1, lane), t1, r + 1);
            meet(true);                                              // Y(r)
        }
        retire(Q.due(t2, lane), t2, r + 2);
        t1 = t2;
    }
    if (TIMED && pair_has<PACK>(a, p0, which)) write_sections<1>(a, p, 1, 2, 3, clk, lane);
}

// ---------------------------------------------------------------------------------------------- serving
// Serving wavefront: after X(r) it serves r and hands it to the retiring wavefront, unless r completes by the arrival of
// r + 2: then it takes r from the load signal itself.  The times at which the slots become free are its own.
template <int MODE, bool ENGINE, bool PROXY, int PACK, bool TIMED, class Comm>
__device__ __forceinline__ void apart_serve_wave(const SegArgs& a, size_t p0, int which, int lane, SlotQueues& Q, double* window, Comm* comm) {
    constexpr bool COUNTS = MODE == MODE_LEAST_REQUEST;      // the load signal is the number of requests, not their tokens
    const int N = (int)a.N;
    const bool there = pair_has<PACK>(a, p0, which);
    const size_t p = p0 + (there ? which : 0);
    const double sc = a.scale[p];
    Tuner<MODE == MODE_ONLINE> tuner(a, p, window, lane, there);
    if (MODE == MODE_ONLINE && lane < 3) comm->w[which][lane] = a.params[3 * p + lane];
    ProbeEpochs<PROXY> probes(a, lane);
    const double a_pf = PROXY ? kept(a.a_pf) : 0.0, slowdown = ENGINE ? kept(a.eng_slowdown) : 0.0;
    // proxy variants: half the round trip time of replica = lane, the request in hand's and the next two's
    double half0 = 0.0, half1 = 0.0, half2 = 0.0;
    if constexpr (!PROXY) comm->half[lane] = lane < a.R ? 0.5 * a.rtt[lane] : 0.0;
    // engine model: this lane's replica has its own rates and KV budget
    const double my_a_pf = ENGINE && lane < a.R ? a.eng_a_pf[lane] : 0.0;
    const double my_a_dec = ENGINE && lane < a.R ? a.eng_a_dec[lane] : 0.0;
    const double my_budget = ENGINE && lane < a.R ? a.eng_budget[lane] : 0.0;
    meet(true);                               // the first descriptors are there
    for (int b = 0; b < 2; ++b)
        if (PACK == 1 || lane < HALF) comm->gone[b][which * HALF + lane] = 0.0;
    // arrival times of the request in hand and the two after it
    double t0 = (double)a.ts[0] * sc, t1 = (double)a.ts[N > 1 ? 1 : 0] * sc;
    if (PROXY) {
        half0 = probes.template at<PACK>(t0, 0, comm, which);
        if (N > 1) half1 = probes.template at<PACK>(t1, 1, comm, which);
    }
    meet(true);                               // (nothing has completed yet: the first request can be decided)
    double o_ttft = 0.0, o_e2e = 0.0;
    SectionClock<TIMED> clk;
    clk.start();
    for (int b0 = 0; b0 < N; b0 += WAVE) {
        const int in_batch = N - b0 < WAVE ? N - b0 : WAVE;
        for (int i = 0; i < in_batch; ++i) {
            const int r = b0 + i;
            const SegDesc& d = comm->ring[r & (DESC_RING - 1)];
            const int4 h = *reinterpret_cast<const int4*>(&d.L);
            const int L = h.x, O = ENGINE ? d.O : 0;
            const double t2 = d.t2[which], dec = ENGINE ? 0.0 : d.dec;
            const bool sync = (__builtin_amdgcn_readfirstlane(h.w) & DESC_SYNC) != 0;
            clk.tick(0);
            meet(true);                                                  // X(r)
            clk.tick(1);                                                 // waiting at X
            const int lane_best = __builtin_amdgcn_readfirstlane(comm->best[r & 1][which]);
            const double prefill = (double)comm->choice[r & 1][lane_best].prefill;
            const int best = PACK == 2 ? lane_best & (HALF - 1) : lane_best;
            double half;
            if constexpr (PROXY) half = readlane_f64(half0, best);
            else half = comm->half[best];
            double ttft, e2e, done;
            int k;
            if constexpr (ENGINE)
                k = Q.start_engine(best, t0, half, readlane_f64(my_a_pf, best) * prefill, readlane_f64(my_a_dec, best) * (double)O,
                            (unsigned)L + (unsigned)O, readlane_f64(my_budget, best), slowdown, lane, &ttft, &e2e, &done);
            else
                k = Q.template start_linear<PROXY>(best, t0, half, PROXY ? a_pf * prefill : prefill, dec, lane, &ttft, &e2e, &done);
            clk.tick(9);                                                 // service
            const int weight = COUNTS ? 1 : L;
            bool left = done <= (sync ? t1 : t2);
            // (the same in every lane)
            auto leave = [&](int to) {
                if (lane == 0)
                    __hip_atomic_fetch_add(&comm->gone[to & 1][lane_best], -(double)weight, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            if (__builtin_expect(ballot(left) != 0, 0)) leave(sync ? r + 1 : r + 2);
            o_ttft = lane == i ? ttft : o_ttft;
            o_e2e = lane == i ? e2e : o_e2e;
            if constexpr (MODE == MODE_ONLINE) tuner.sample(ttft, comm->w[which]);
            clk.tick(5);                                                 // outputs, tuner
            if (sync) {
                meet(true);                                              // Y(r)
                const bool now = !left && done <= t2;
                if (ballot(now) != 0) leave(r + 2);
                left = left || now;
            }
            comm->served[which][r & 1] = Served{done, left || !there ? -1 : best * Q.B + k, weight};
            if (PROXY) {
                half2 = probes.template at<PACK>(t2, r + 2, comm, which);
                half0 = half1;
                half1 = half2;
            }
            t0 = t1;
            t1 = t2;
        }
        // the batch is done: its outputs go out
        if (lane < in_batch && there) {
            const size_t o = p * N + b0 + lane;
            if (a.ttft) a.ttft[o] = o_ttft;
            if (a.e2e) a.e2e[o] = o_e2e;
        }
    }
    if (TIMED && there) {
        write_sections<1>(a, p, 1, 0, 1, clk, lane);
        write_sections<1>(a, p, 1, 4, SECTIONS - 1, clk, lane);
    }
    tuner.results();
}

// ---------------------------------------------------------------------------------------------- deciding
template <int MODE, bool ENGINE, bool PROXY, int PACK, bool TIMED, class Comm>
__device__ __forceinline__ void apart_decide_wave(const SegArgs& a, size_t p0, int lane, Comm* comm) {
    constexpr bool ONLINE = MODE == MODE_ONLINE;
    constexpr bool SCORED = MODE == MODE_COST_MODEL || MODE == MODE_ONLINE;
    constexpr bool COUNTS = MODE == MODE_LEAST_REQUEST;
    constexpr bool DICTATED = MODE == MODE_AFFINITY || MODE == MODE_RANDOM || MODE == MODE_GIVEN;
    const int R = a.R, N = (int)a.N;
    const Pair<PACK> pair(a, p0, lane);
    const size_t p = pair.p;
    const int rl = pair.rl;
    const bool in = rl < R;
    const int block_tokens = kept(a.block_tokens);
    const double a_pf = kept(a.a_pf);
    double w_rtt = a.params[3 * p + 0], w_prefill = a.params[3 * p + 1], w_queue = a.params[3 * p + 2];
    double my_rtt = !PROXY && in ? a.rtt[rl] : 0.0;            // (proxy variants: comes from the serving wavefront)
    // first product of Eq. 3 (lanes without a replica: a score above any)
    double rtt_term = in ? w_rtt * my_rtt : INFINITY;
    double q = COUNTS && !in ? INFINITY : 0.0;       // load signal of replica = lane (an integer below 2^53, exact in fp64)
    double tokens = 0.0;                             // what the request before adds to it where it went
    const bool own_index = PROXY && a.index_blocks >= 0;
    unsigned long long went1 = 0, went2 = 0, went3 = 0;  // where the three requests before went
    const char* const rows = reinterpret_cast<const char*>(a.last + p0 * (size_t)a.nseg * R);
    const unsigned row_bytes = (unsigned)R * 4u;
    const unsigned lane_off = (pair.upper && pair.there ? (unsigned)a.nseg * row_bytes : 0u) + (unsigned)(in ? rl : 0) * 4u;
    auto cell_at = [&](uint32_t rowoff) { return reinterpret_cast<const int32_t*>(rows + (rowoff + lane_off)); };
    const int spare = N;                      // the log record behind the last request's
    // the request before, on this lane's replica: blocks it would have added, oldest request it matched blocks of
    int added1 = 0, oldest1 = INT32_MAX;
    // where this replica's eviction cursors are (`hi` is read last)
    struct {
        int32_t cur_r, cur_r2, hi;
        uint32_t k_room;
        int32_t cur_k2;
    } at{-1, -1, -1, 0, 0};
    auto look = [&]() {
        at.cur_r = ld(&comm->cur_r[0][lane]);
        at.k_room = ld(&comm->k_room[lane]);
        if constexpr (PROXY) {
            at.cur_r2 = ld(&comm->cur_r[1][lane]);
            at.cur_k2 = ld(&comm->cur_k2[lane]);
        }
        in_order();
        at.hi = ld(&comm->hi[lane]);
    };
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
    int before = 0;           // flags of the request before
    meet(true);                               // the first descriptors and cells are there
    take(0, 0);
    meet(true);                               // the other wavefronts have set themselves up
    clk.start();
    for (int next = 0; next < N; ++next) {
        const int r = __builtin_amdgcn_readfirstlane(next);
        const SegDesc* const dr = &comm->ring[r & (DESC_RING - 1)];
        const int target = DICTATED && MODE != MODE_GIVEN ? dr->target : 0;
        double left = DICTATED ? 0.0 : comm->gone[r & 1][lane];      // (read again behind Y(r - 1))
        // (what the choice before adds to the load signal, while LDS is read)
        if (COUNTS) q += of_mask(went1) ? 1.0 : 0.0;
        else if (!DICTATED) q += of_mask(went1) ? tokens : 0.0;
        if constexpr (PROXY) my_rtt = comm->rtt[r & 1][lane];
        look();       // (behind the other reads: online tuner and proxy 0.5 % faster than before them)
        const int flags = __builtin_amdgcn_readfirstlane(word);
        const int was = __builtin_amdgcn_readfirstlane(before);
        bool behind = (was & DESC_SYNC) != 0;
        auto caught_up = [&]() {
            meet(false);
            behind = false;
            if (!DICTATED) left = comm->gone[r & 1][lane];
            if (ONLINE) {
                w_rtt = comm->w[pair.upper ? 1 : 0][0];
                w_prefill = comm->w[pair.upper ? 1 : 0][1];
                w_queue = comm->w[pair.upper ? 1 : 0][2];
                rtt_term = in ? w_rtt * my_rtt : INFINITY;
            }
        };
        // ---- the rows were loaded before the stores of the three requests before were sure to be there: the leading
        // segments that the paths share get the cells that those requests wrote on their replicas
        if (flags & DESC_SHARED) {
#pragma unroll
            for (int k = 0; k < SEG_CHUNK; ++k) {
                cell[k] = of_mask(went3) && k < ((flags >> 20) & 15) ? r - 3 : cell[k];
                cell[k] = of_mask(went2) && k < ((flags >> 12) & 15) ? r - 2 : cell[k];
                cell[k] = of_mask(went1) && k < ((flags >> 8) & 15) ? r - 1 : cell[k];
            }
        }
        // ---- prefix match as in decide_wave: max(e_gt, min(cur_k, e_ge)) with e_gt, e_ge the ends of the last segment whose
        // cell is above, respectively not below, the cursor's request
        int my_m, my_seen = 0, k_end, oldest;
        unsigned long long holders, single;      // lanes that match, and whose match has one previous owner
        const unsigned long long tight = (ballot(added1 > (int)(at.k_room >> 16)) | ballot(oldest1 <= at.hi)) & went1;
        const unsigned long long late = (unsigned)((was & DESC_SYNC) | (flags & DESC_DEEP));
        auto match = [&]() {
            int e_gt = 0, e_ge = 0;
            int32_t own_ge = INT32_MAX;      // previous owner of the last segment counted in e_ge
            int e_gt2 = 0, e_ge2 = 0;        // proxy variants: the same against the index's cursor
            int32_t own_ge2 = INT32_MAX;
            auto compare = [&](int k) {
                const bool gt = cell[k] > at.cur_r;
                const bool ge = cell[k] >= at.cur_r;
                e_gt = gt ? end[k] : e_gt;
                e_ge = ge ? end[k] : e_ge;
                own_ge = ge ? cell[k] : own_ge;
                if (PROXY) {
                    const bool gt2 = cell[k] > at.cur_r2;
                    const bool ge2 = cell[k] >= at.cur_r2;
                    e_gt2 = gt2 ? end[k] : e_gt2;
                    e_ge2 = ge2 ? end[k] : e_ge2;
                    own_ge2 = ge2 ? cell[k] : own_ge2;
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
            const int cur_k = (int)(at.k_room & 0xFFFFu);
            const int below_cursor = cur_k < e_ge ? cur_k : e_ge;
            const bool some_eq = below_cursor > e_gt;       // blocks of the cursor's own request are matched
            my_m = some_eq ? below_cursor : e_gt;
            const int below_cursor2 = at.cur_k2 < e_ge2 ? at.cur_k2 : e_ge2;
            const bool some_eq2 = below_cursor2 > e_gt2;
            my_seen = PROXY ? (some_eq2 ? below_cursor2 : e_gt2) : 0;       // blocks in the proxy's index (>= my_m)
            // For the ownership update: where the cached prefix ends on this replica (rounded up to the end of a segment
            // that the cursor's request owns: what lies beyond the cursor is evicted anyway) and whether all cached segments
            // had the same previous owner: the evicting wavefront is told that one, and finds several by itself.  (A segment of
            // the cursor's request beyond the cursor is taken for one more owner: rare, and the walk knows better.)
            k_end = PROXY ? (some_eq2 ? e_ge2 : e_gt2) : (some_eq ? e_ge : e_gt);
            holders = ballot((PROXY ? my_seen : my_m) > 0);
            single = ballot((PROXY ? own_ge2 : own_ge) == cell[0]);
            oldest = PROXY ? own_ge2 : own_ge;
        };
        match();
        int owner = of_mask(holders & single) ? cell[0] : spare;
        owner = of_mask(holders & ~single) ? OWN_WALK : owner;
        // The evicting wavefront may still be moving the cursor of the replica that the request before went to.  Where it is,
        // read before, while or after it moves, makes no difference if it cannot pass the youngest record of the look-ahead ring
        // and everything matched is younger -- by this request, and for `room` to be what it says by the one before.  One
        // request in a hundred waits with 32 replicas, one in twelve with three.  The other rare cases share the branch:
        // Y(r - 1), as late as this, and a path longer than is preloaded.
        const unsigned long long unsure = (ballot(oldest <= at.hi) & went1) | tight;
        if (__builtin_expect((unsure | late) != 0, 0)) {
            if (behind) caught_up();
            if (unsure != 0 || (flags & DESC_DEEP)) {
                while (ld(&comm->evicted) < r - 1) __builtin_amdgcn_s_sleep(1);
                in_order();
                look();
                match();
                owner = of_mask(holders & single) ? cell[0] : spare;
                owner = of_mask(holders & ~single) ? OWN_WALK : owner;
            }
            if (flags & DESC_DEEP) {
                // more than eight segments (memory is up to date behind Y(r - 1)): the rest of the path is read from the
                // trace, eight references at a time, as long as some replica's prefix is still open
                const int64_t j0 = dr->j0;
                const int s = __builtin_amdgcn_readfirstlane(dr->s);
                const int cur_k = (int)(at.k_room & 0xFFFFu);
                int pos = end[7];
                bool open = my_m == pos;
                bool open_seen = PROXY && my_seen == pos;
                if (ballot((PROXY ? open_seen : open) && in) != 0) {
                    owner = of_mask(holders) ? OWN_WALK : spare;
                    oldest = -1;                     // (older than the preloaded ones)
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
                                const int cnt = cached_in(more[k], pos, send[k], at.cur_r, cur_k);
                                my_m += open ? cnt : 0;
                                open = open && cnt == send[k] - pos;
                                if (PROXY) {
                                    const int cnt_seen = cached_in(more[k], pos, send[k], at.cur_r2, at.cur_k2);
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
        }
        if (!DICTATED) comm->gone[r & 1][lane] = 0.0;
        clk.tick(1);                                                 // patch, match

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
            my_score = rl == target ? 0.0 : 1.0;      // the replica is dictated
        }
        // ---- what every replica would mean for the request, whatever the choice
        const unsigned hit_end = (unsigned)my_m | ((unsigned)k_end << 16);
        if constexpr (PROXY) comm->choice[r & 1][lane] = Choice<true>{my_u, own_index ? my_seen : my_m, owner, hit_end};
        else comm->choice[r & 1][lane] = Choice<false>{my_prefill, owner, hit_end};
        // (what is still needed of this request's numbers, and the next one's: its reads are under way during the minimum)
        added1 = n - my_m;                      // (not below what the index would add)
        oldest1 = oldest;
        tokens = (double)L;
        set = set == CELL_SETS - 1 ? 0 : set + 1;
        take(r + 1, set);
        const unsigned long long bests = argmin_mask<PACK>(my_score, pair.upper);
        if (PACK == 1) comm->best[r & 1][0] = __builtin_ctzll(bests);
        else comm->best[r & 1][pair.upper ? 1 : 0] = pair.upper ? HALF + __builtin_ctz((unsigned)(bests >> 32)) : __builtin_ctz((unsigned)bests);
        clk.tick(3);                                                 // score, minimum, announcement
        went3 = went2;
        went2 = went1;
        went1 = bests;
        meet(true);                                                  // X(r)
        clk.tick(0);                                                 // waiting at X
        before = flags;
    }
    if (TIMED) write_sections<PACK>(a, p0, 0, 0, 7, clk, lane);     // (the evicting wavefront writes the counts)
}

// Replay p0, or replays p0 and p0 + 1, by one workgroup.  Three of a replay each fit a CU by their registers, two in the proxy
// variant with engine model and tuner; LDS may allow fewer (30,592 bytes of hand-over words in the proxy variants and 53,248 of
// slots and window make 84 KB: one).  The launch rule counts both.
template <int PACK>
constexpr int apart_threads() { return (APART_WAVES + 2 * (PACK - 1)) * WAVE; }

// What the wavefronts of a workgroup do.  The one with number w runs on the same SIMD as those with w + 4, so which two share one is
// a matter of this order; the longest chains go with the shortest.  (4,000 blocks a cache.  One replay: with decide, serve, retire,
// book, evict, front -- deciding and evicting on one SIMD -- 64 replays of 6,000 requests on 32 replicas took 0.495 us a
// request, so 0.485, proxy 0.656 / 0.591; 512 of them 0.547 / 0.523, proxy 0.717 / 0.679, engine model 0.681 / 0.631.
// Two replays, 1,023 on 32 replicas: decide, serve, serve, evict, book, retire, retire, front 0.591, tuner 0.660, proxy 0.693; so 0.582,
// 0.657, 0.684.  With the engine model, whose serving wavefront is among the longest, 0.689, so 0.717, and in its own order 0.677.)
enum ApartRole { DECIDE, SERVE, RETIRE, BOOK, EVICT, FRONT, SERVE_2, RETIRE_2 };       // (_2: of the workgroup's second replay)
template <bool ENGINE, int PACK>
__device__ __forceinline__ int apart_role(int wave) {
    constexpr unsigned long long ONE = DECIDE | SERVE << 4 | EVICT << 8 | RETIRE << 12 | BOOK << 16 | FRONT << 20;
    constexpr unsigned long long TWO = ENGINE
        ? DECIDE | SERVE << 4 | SERVE_2 << 8 | EVICT << 12 | RETIRE << 16 | RETIRE_2 << 20 | BOOK << 24 | (unsigned long long)FRONT << 28
        : DECIDE | EVICT << 4 | RETIRE << 8 | RETIRE_2 << 12 | FRONT << 16 | BOOK << 20 | SERVE << 24 | (unsigned long long)SERVE_2 << 28;
    return (int)((PACK == 1 ? ONE : TWO) >> (4 * wave)) & 15;
}

// args: where a role gets the launch's arguments from.
template <int MODE, bool ENGINE, bool PROXY, int PACK, bool TIMED, class Args>
__device__ __forceinline__ void apart_replay(Args args, size_t p0, unsigned char* lds_raw) {
    __shared__ ApartHandover<PROXY, PACK> comm;
    const SegArgs& a = args();
    const int lane = threadIdx.x & (WAVE - 1);
    const int role = apart_role<ENGINE, PACK>(__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE)));
    const int which = PACK == 2 && role >= SERVE_2 ? 1 : 0;
    unsigned char* const queues = lds_raw + which * replay_queue_lds_bytes(a.R, a.B, ENGINE, MODE == MODE_ONLINE ? a.window : 0);
    if (role == SERVE || (PACK == 2 && role == SERVE_2)) {
        double* const window = reinterpret_cast<double*>(queues + SlotQueues::bytes(a.R, a.B, ENGINE));
        if (a.N == 0) {       // (an empty trace still reports the tuner's initial state)
            if (pair_has<PACK>(a, p0, which)) Tuner<MODE == MODE_ONLINE>(a, p0 + which, window, lane).results();
            return;
        }
        __builtin_amdgcn_s_setprio(2);
        SlotQueues Q;
        Q.init(queues, a.R, a.B, ENGINE, lane);
        apart_serve_wave<MODE, ENGINE, PROXY, PACK, TIMED>(args(), p0, which, lane, Q, window, &comm);
    } else if (a.N == 0) {
        return;
    } else if (role == DECIDE) {
        __builtin_amdgcn_s_setprio(3);      // the wavefront on the chain goes first at issue
        apart_decide_wave<MODE, ENGINE, PROXY, PACK, TIMED>(args(), p0, lane, &comm);
    } else if (role == RETIRE || (PACK == 2 && role == RETIRE_2)) {
        __builtin_amdgcn_s_setprio(2);
        SlotQueues Q;
        Q.attach(queues, a.R, a.B);
        apart_retire_wave<PROXY, PACK, TIMED>(args(), p0, which, lane, Q, &comm);
    } else if (role == BOOK) {
        __builtin_amdgcn_s_setprio(1);
        apart_book_wave<PROXY, PACK, TIMED>(args(), p0, lane, &comm);
    } else if (role == EVICT) {
        __builtin_amdgcn_s_setprio(2);
        apart_evict_wave<PROXY, PACK, TIMED>(args(), p0, lane, &comm);
    } else {
        front_wave<MODE, PROXY, PACK, TIMED>(args(), lane, &comm);
    }
}

template <int MODE, bool ENGINE, bool PROXY, bool TIMED = false>
__global__ void __launch_bounds__(apart_threads<1>(), 4) replay_apart_kernel(SegArgs a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    apart_replay<MODE, ENGINE, PROXY, 1, TIMED>([]() -> const SegArgs& { return kernel_args<SegArgs>(); }, blockIdx.x, lds_raw);
}

// Two replays per workgroup: the wavefronts that look at replicas have them in their halves, each replay has a serving and a retiring
// wavefront of its own.
template <int MODE, bool ENGINE, bool PROXY>
__global__ void __launch_bounds__(apart_threads<2>(), 4) replay_apart_pairs_kernel(SegArgs a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    apart_replay<MODE, ENGINE, PROXY, 2, false>([]() -> const SegArgs& { return kernel_args<SegArgs>(); }, 2 * (size_t)blockIdx.x, lds_raw);
}

// The timed instantiation.
template <int MODE, bool ENGINE, bool PROXY>
__global__ void __launch_bounds__(apart_threads<2>(), 4) replay_apart_pairs_timed_kernel(SegArgs a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    apart_replay<MODE, ENGINE, PROXY, 2, true>([]() -> const SegArgs& { return kernel_args<SegArgs>(); }, 2 * (size_t)blockIdx.x, lds_raw);
}

}  // namespace gorgo
