// Replay kernel, block-table formulation (any trace).
//
// The cache of a replica is a hashed table key -> stamp of the last touch (stamp = request * stride + (stride - 1 -
// position): within a request the root is the newest), and "cached" means "stamp not below the replica's eviction
// threshold".  Least-recently-used eviction only raises that threshold: the cursor behind it walks the replica's
// log of routed requests, oldest first, deepest block first, and a logged touch still counts iff the table holds
// exactly its stamp.  Nothing about the trace is assumed (the same id may follow different ids in different
// requests), so the match probes block by block.
//
// A replay is run by three wavefronts of one workgroup.  The queue wavefront is the segment formulation's: service
// slots, service step, what leaves the load signal (Eq. 2), per-request outputs, and with them the online tuner, the
// engine model and the epochs of the proxy's round-trip estimates.  The deciding wavefront scores a request (Eq. 3) or
// applies the baseline policy, takes the lowest-index minimum and announces the choice; meeting X.  Then the updating
// wavefront updates the chosen replica's table and evicts, the queue wavefront serves the request, and the deciding
// wavefront matches the next request against the tables of all other replicas, which the choice does not change;
// meeting Y; the chosen replica is matched then.  A request is a chain of memory round trips and nothing else: with the
// match and the update one after the other in one wavefront 65 replays of 3,001 requests on 7 replicas took 26.6 ms, so
// 23.8; 1,024 replays of 4,000 requests on 32 replicas take 24.5 either way.  Every wavefront executes exactly two
// barriers per request, whatever the data.
//
// The proxy's own index of a replica (Sec. 7: the proxy does not see replica-side eviction) is a second LRU over
// the same touches with a capacity of its own.  Touches give an entry the same stamp in both, so the index is the
// same table read against a second threshold, with a cursor of its own on the same log.
#pragma once
#include "device_common.h"
#include "internal.h"
#include "replay_segments.h"

namespace gorgo {

constexpr int BLOCK_THREADS = 3 * WAVE;      // deciding, updating and queue wavefront

// One cache-table slot.  key 0 = never used (then stamp = -1).  An entry is held by an LRU iff stamp >= that
// LRU's threshold; entries below every threshold are garbage whose slots can be taken over by inserts.
struct Slot {
    uint64_t key;
    int64_t stamp;
};

struct BlockArgs {
    SegArgs q;               // what the queue wavefront reads, and the model, weights and policy inputs
    const int64_t* blk_off;  // [N+1]
    const uint32_t* key;     // [T] dense block keys, 0 never occurs
    const uint8_t* first;    // [T] 1 where the key occurs for the first time within its request
    Slot* tables;            // [P][R][cap]
    Slot* spare;             // [P][cap] scratch of the compaction
    uint8_t* routed;         // [P][N] the updating wavefront's log of choices (what its eviction cursors walk)
    int64_t cap;             // slots per table, a power of two
    int32_t cap_log2;
};

// per replica: two thresholds (int64), then live x2, cursor request x2, cursor position x2, used slots (int32)
__host__ __device__ inline size_t replay_blocks_state_bytes(int R) { return (size_t)R * (2 * 8 + 7 * 4); }
__host__ __device__ inline size_t replay_blocks_lds_bytes(int R, int B, bool engine, int window) {
    return ((replay_queue_lds_bytes(R, B, engine, window) + 15) & ~(size_t)15) + replay_blocks_state_bytes(R);
}

__device__ __forceinline__ bool cas_stamp(int64_t* p, int64_t expected, int64_t desired) {
    return __hip_atomic_compare_exchange_strong(p, &expected, desired, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ uint64_t home_slot(uint64_t key, int cap_log2) {
    return (key * 0x9E3779B97F4A7C15ull) >> (64 - cap_log2);
}

// Physical lookup of G keys per lane, in a table each, all lanes of the wavefront together: slot index and stamp of the
// key, or -1 (a stamp below every threshold) where the probe sequence reaches a never-used slot.  A probe is a serial
// chain of memory round trips of 600 cycles and more, so every step reads U whole slots of all G sequences before it
// looks at any of them.  (One slot of one sequence at a time, key before stamp: 65 replays of 3,001 requests on 7
// replicas 37.1 ms, 1,024 of 4,000 on 32 replicas 33.3 ms; so 26.6 and 24.5.  Only what `active` has a bit for is looked up; the other loads stay where the sequence ended.)
// FREE: also the first slot on the way that an insert may take over (stamp below `tau`), with that stamp.
template <int G>
struct Found {
    int64_t slot[G], stamp[G];
    int64_t free_slot[G], free_stamp[G];
};
template <int G, int U, bool FREE = false>
__device__ __forceinline__ Found<G> find_slots(const Slot* const (&tab)[G], const uint64_t (&key)[G], unsigned active, uint64_t mask,
                                               int cap_log2, int64_t tau = 0) {
    Found<G> f;
    uint64_t h[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        h[g] = home_slot(key[g], cap_log2);
        f.slot[g] = f.stamp[g] = f.free_slot[g] = f.free_stamp[g] = -1;
    }
    unsigned open = active;
    while (ballot(open != 0) != 0) {
        Slot e[G][U];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < G; ++g) e[g][u] = tab[g][(h[g] + u) & mask];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            bool on = (open >> g & 1u) != 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t at = (int64_t)((h[g] + u) & mask);
                if (FREE) {
                    const bool take = on && f.free_slot[g] < 0 && e[g][u].stamp < tau;
                    f.free_slot[g] = take ? at : f.free_slot[g];
                    f.free_stamp[g] = take ? e[g][u].stamp : f.free_stamp[g];
                }
                const bool hit = on && e[g][u].key == key[g];
                f.slot[g] = hit ? at : f.slot[g];
                f.stamp[g] = hit ? e[g][u].stamp : f.stamp[g];
                on = on && !hit && e[g][u].key != 0;
            }
            h[g] = on ? (h[g] + U) & mask : h[g];
            open &= on ? ~0u : ~(1u << g);
        }
    }
    return f;
}

// Takes over the first never-used or garbage slot of the probe sequence (stamp below `tau`, the lowest threshold) from
// slot h on.  Returns true when a never-used slot was consumed.  Only called for keys known to be physically absent, by
// lanes with distinct keys.
__device__ __forceinline__ bool insert_new(Slot* tab, uint64_t h, uint64_t key, int64_t stamp, int64_t tau, uint64_t mask) {
    for (;;) {
        int64_t s = ld(&tab[h].stamp);
        if (s < tau && cas_stamp(&tab[h].stamp, s, stamp)) {
            st(&tab[h].key, key);
            return s == -1;
        }
        h = (h + 1) & mask;
    }
}

__global__ void __launch_bounds__(256) fill_slots(Slot* s, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        s[i].key = 0;
        s[i].stamp = -1;
    }
}

// What the lanes of this wavefront have written to global memory is there for its other lanes to read (the updating
// wavefront is the only one that writes the tables and the log of choices; a table is read by the deciding wavefront only
// while it is not being written: meetings X and Y).
__device__ __forceinline__ void wave_settle() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// The replicas' LRU state, shared by the two wavefronts (LDS).
struct LruState {
    int64_t *tau1, *tau2;      // [R] eviction thresholds: the cache's, the index's
    int32_t *live1, *live2;    // [R] blocks held
    int32_t *cur_r1, *cur_r2;  // [R] eviction cursors: request ...
    int32_t *cur_k1, *cur_k2;  // [R] ... and position (blocks >= cur_k are gone)
    int32_t *used;             // [R] slots ever used since the last compaction
    __device__ __forceinline__ LruState(unsigned char* state, int R) {
        tau1 = reinterpret_cast<int64_t*>(state);
        tau2 = tau1 + R;
        live1 = reinterpret_cast<int32_t*>(tau2 + R);
        live2 = live1 + R;
        cur_r1 = live2 + R;
        cur_r2 = cur_r1 + R;
        cur_k1 = cur_r2 + R;
        cur_k2 = cur_k1 + R;
        used = cur_k2 + R;
    }
};

// Where a request's blocks are, how many, input tokens, and its first 128 keys with their first-occurrence marks (lane =
// block).  Read ahead of the request.
struct Blocks {
    int64_t off;
    int n, L;
    uint32_t key[2];
    int first[2];
    __device__ __forceinline__ void read_scalars(const BlockArgs& b, int64_t r) {
        const int64_t x = r < b.q.N ? r : b.q.N - 1;
        off = b.blk_off[x];
        n = (int)(b.blk_off[x + 1] - off);
        L = b.q.in_len[x];
    }
    __device__ __forceinline__ uint64_t key_at(const BlockArgs& b, int k) const { return k < n ? b.key[off + k] : 0u; }
    __device__ __forceinline__ void read_keys(const BlockArgs& b, int lane) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int k = g * WAVE + lane;
            key[g] = k < n ? b.key[off + k] : 0u;
        }
    }
    __device__ __forceinline__ void read_marks(const BlockArgs& b, int lane) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            const int k = g * WAVE + lane;
            first[g] = k < n ? b.first[off + k] : 0;
        }
    }
};

// Deciding wavefront of a replay over block tables.  Lane = replica for the first-block probe, the scores and the
// minimum; lane = block of the request for the prefix match.
template <int MODE, bool ENGINE, bool PROXY>
__device__ __forceinline__ void block_decide_wave(const BlockArgs& b, int p, int lane, const LruState& lru, QueueHandover<PROXY>* comm) {
    constexpr bool ONLINE = MODE == MODE_ONLINE;
    constexpr bool SCORED = MODE == MODE_COST_MODEL || MODE == MODE_ONLINE;
    const SegArgs& a = b.q;
    const int R = a.R;
    const int64_t N = a.N;
    const bool in = lane < R;
    const uint64_t mask = (uint64_t)b.cap - 1;
    const int cap_log2 = b.cap_log2;
    const bool two = PROXY && a.index_blocks >= 0;      // the proxy has an index of its own
    int64_t *const tau1 = lru.tau1, *const tau2 = lru.tau2;
    for (int i = lane; i < R; i += WAVE) {
        tau1[i] = tau2[i] = 0;
        lru.live1[i] = lru.live2[i] = 0;
        lru.cur_r1[i] = lru.cur_r2[i] = -1;
        lru.cur_k1[i] = lru.cur_k2[i] = 0;
        lru.used[i] = 0;
    }

    double w_rtt = a.params[3 * (size_t)p + 0];
    double w_prefill = a.params[3 * (size_t)p + 1];
    double w_queue = a.params[3 * (size_t)p + 2];
    double q = 0.0;                                               // load signal of replica = lane
    double my_rtt = !PROXY && in ? a.rtt[lane] : 0.0;             // (proxy variants: comes from the queue wavefront)
    const uint64_t seed = MODE == MODE_RANDOM ? a.seeds[p] : 0;
    const Slot* const tables = b.tables + (size_t)p * R * b.cap;

    Blocks now, next, after;
    now.read_scalars(b, 0);
    now.read_keys(b, lane);
    next.read_scalars(b, 1);
    next.read_keys(b, lane);
    after.read_scalars(b, 2);

    // ---- prefix match of a request against the cache's threshold and, with an index, against the index's as well: the
    // whole list on the replicas in `holders`, four at a time (their probes do not depend on each other)
    int my_m = 0, my_seen = 0;
    auto match_on = [&](const Blocks& of, unsigned long long holders) {
        const int n = of.n;
        auto match = [&](auto count) {          // the next `count` holders
            constexpr int G = decltype(count)::value;
            int id[G], m1[G], m2[G];
            int64_t t1[G], t2[G];
            const Slot* tab[G];
            bool open1[G], open2[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const bool there = holders != 0;
                id[g] = there ? __builtin_ctzll(holders) : id[0];
                holders &= holders - (there ? 1 : 0);
                tab[g] = tables + (size_t)id[g] * b.cap;
                t1[g] = tau1[id[g]];
                t2[g] = two ? tau2[id[g]] : t1[g];
                m1[g] = m2[g] = 0;
                open1[g] = there;
                open2[g] = there && two;
            }
            for (int base = 0; base < n; base += WAVE) {
                const int k = base + lane;
                const uint64_t mine = base == 0 ? of.key[0] : (base == WAVE ? of.key[1] : of.key_at(b, k));
                uint64_t key[G];
                unsigned active = 0;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    key[g] = mine;
                    active |= k < n && (open1[g] || open2[g]) ? 1u << g : 0u;
                }
                const Found<G> f = find_slots<G, 2>(tab, key, active, mask, cap_log2);
                const int width = n - base < WAVE ? n - base : WAVE;
                const unsigned long long want = width == WAVE ? ~0ull : ((1ull << width) - 1);
                bool more = false;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const unsigned long long got1 = ballot(k < n && f.stamp[g] >= t1[g]);
                    const unsigned long long got2 = ballot(k < n && f.stamp[g] >= t2[g]);
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
    // ---- the same on the replicas in `among` that hold the first block
    auto match_among = [&](const Blocks& of, unsigned long long among) {
        if (of.n == 0) return;
        const bool mine = (among >> lane & 1) != 0;
        const Slot* const tab[1] = {tables + (size_t)(mine ? lane : 0) * b.cap};
        const uint64_t key[1] = {(uint32_t)__builtin_amdgcn_readlane((int)of.key[0], 0)};
        const int64_t stamp = find_slots<1, 4>(tab, key, mine ? 1u : 0u, mask, cap_log2).stamp[0];
        const int64_t t1 = mine ? tau1[lane] : 0, t2 = two && mine ? tau2[lane] : t1;
        match_on(of, ballot(mine && stamp >= (t2 < t1 ? t2 : t1)));
    };
    const unsigned long long all = R >= WAVE ? ~0ull : (1ull << R) - 1;

    meet(true);         // (the queue wavefront has set itself up)
    // (nothing is cached yet: the first request matches nowhere)
    int previous = -1;
    for (int64_t r = 0; r < N; ++r) {
        const int n = now.n, L = now.L;
        // the replica that the previous request went to was still being updated: its turn now
        if (previous >= 0 && n > 0) match_on(now, 1ull << previous);
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
        after.read_keys(b, lane);
        my_m = my_seen = 0;
        if (r + 1 < N) match_among(next, all & ~(1ull << best));
        now = next;
        next = after;
        after.read_scalars(b, r + 3);
        previous = best;
        meet(true);                                                  // Y(r): what completes by the next arrival is known
        if (ONLINE) {
            w_rtt = comm->w[0][0];
            w_prefill = comm->w[0][1];
            w_queue = comm->w[0][2];
        }
    }
}

// Updating wavefront: between X(r) and Y(r) it brings the chosen replica up to date.  Lane = block.
template <bool PROXY>
__device__ __forceinline__ void block_update_wave(const BlockArgs& b, int p, int lane, const LruState& lru, QueueHandover<PROXY>* comm) {
    const SegArgs& a = b.q;
    const int64_t N = a.N;
    const uint64_t mask = (uint64_t)b.cap - 1;
    const int cap_log2 = b.cap_log2;
    // the proxy's own index: a second LRU (capacity index_blocks, 0 = it never forgets) over the same touches
    const bool two = PROXY && a.index_blocks >= 0;
    const int64_t C1 = a.C, C2 = two ? a.index_blocks : 0;
    int64_t *const tau1 = lru.tau1, *const tau2 = lru.tau2;
    int32_t *const live1 = lru.live1, *const live2 = lru.live2, *const cur_r1 = lru.cur_r1, *const cur_r2 = lru.cur_r2,
            *const cur_k1 = lru.cur_k1, *const cur_k2 = lru.cur_k2, *const used = lru.used;
    Slot* const tables = b.tables + (size_t)p * a.R * b.cap;
    Slot* const spare = b.spare + (size_t)p * b.cap;
    uint8_t* const routed = b.routed + (size_t)p * N;
    const int64_t rebuild_at = b.cap - b.cap / 8;

    Blocks now, next;
    now.read_scalars(b, 0);
    now.read_keys(b, lane);
    now.read_marks(b, lane);
    next.read_scalars(b, 1);
    meet(true);
    for (int64_t r = 0; r < N; ++r) {
        const int64_t off = now.off;
        const int n = now.n;
        next.read_keys(b, lane);
        next.read_marks(b, lane);
        Blocks after;
        after.read_scalars(b, r + 2);
        meet(true);                                                  // X(r): the choice is there
        const int best = __builtin_amdgcn_readfirstlane(comm->best[r & 1][0]);
        if (lane == 0) st(&routed[r], (uint8_t)best);

        // ---- update on the chosen replica
        Slot* const tab = tables + (size_t)best * b.cap;
        if ((int64_t)used[best] + n > rebuild_at) {
            // compact: keep what some LRU still holds, so that never-used slots exist again
            const int64_t t1 = tau1[best], t2 = two ? tau2[best] : t1;
            const int64_t keep_from = t2 < t1 ? t2 : t1;
            int64_t kept = 0;
            for (int64_t base = 0; base < b.cap; base += WAVE) {
                const uint64_t k = ld(&tab[base + lane].key);
                const int64_t s = ld(&tab[base + lane].stamp);
                const bool keep = k != 0 && s >= keep_from;
                const unsigned long long mk = ballot(keep);
                if (keep) {
                    const int64_t pos = kept + __builtin_popcountll(mk & ((1ull << lane) - 1));
                    st(&spare[pos].key, k);
                    st(&spare[pos].stamp, s);
                }
                kept += __builtin_popcountll(mk);
            }
            wave_settle();
            for (int64_t base = 0; base < b.cap; base += WAVE) {
                st(&tab[base + lane].key, (uint64_t)0);
                st(&tab[base + lane].stamp, (int64_t)-1);
            }
            wave_settle();
            for (int64_t base = 0; base < kept; base += WAVE) {
                if (base + lane < kept) {
                    const uint64_t k = ld(&spare[base + lane].key);
                    insert_new(tab, home_slot(k, cap_log2), k, ld(&spare[base + lane].stamp), 0, mask);
                }
                wave_settle();
            }
            if (lane == 0) used[best] = (int32_t)kept;
            wave_sync();
        }
        {
            // every block of the request becomes (or stays) held, with this request's stamp
            const int64_t t1 = tau1[best], t2 = two ? tau2[best] : t1;
            const int64_t garbage_below = t2 < t1 ? t2 : t1;
            int add1 = 0, add2 = 0, add_used = 0;
            for (int base = 0; base < n; base += 2 * WAVE) {
                bool mine[2];
                uint64_t key[2];
                const Slot* const tabs[2] = {tab, tab};
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int k = base + g * WAVE + lane;
                    key[g] = base == 0 ? now.key[g] : now.key_at(b, k);
                    mine[g] = base == 0 ? now.first[g] != 0 : k < n && b.first[off + k] != 0;
                }
                const Found<2> f = find_slots<2, 2, true>(tabs, key, (mine[0] ? 1u : 0u) | (mine[1] ? 2u : 0u), mask, cap_log2, garbage_below);
                auto stamp_at = [&](int g) { return r * STAMP_STRIDE + (STAMP_STRIDE - 1 - (base + g * WAVE + lane)); };
#pragma unroll
                for (int g = 0; g < 2; ++g)
                    if (mine[g] && f.slot[g] >= 0) st(&tab[f.slot[g]].stamp, stamp_at(g));     // touch, or revive an evicted entry in place
                wave_settle();
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    // (the slot seen on the way is taken unless it has been revived or taken meanwhile)
                    bool took_fresh = false;
                    if (mine[g] && f.slot[g] < 0) {
                        if (cas_stamp(&tab[f.free_slot[g]].stamp, f.free_stamp[g], stamp_at(g))) {
                            st(&tab[f.free_slot[g]].key, key[g]);
                            took_fresh = f.free_stamp[g] == -1;
                        } else {
                            took_fresh = insert_new(tab, (uint64_t)f.free_slot[g], key[g], stamp_at(g), garbage_below, mask);
                        }
                    }
                    add1 += __builtin_popcountll(ballot(mine[g] && f.stamp[g] < t1));
                    add2 += __builtin_popcountll(ballot(mine[g] && f.stamp[g] < t2));
                    add_used += __builtin_popcountll(ballot(took_fresh));
                }
                wave_settle();
            }
            if (lane == 0) {
                live1[best] += add1;
                live2[best] += add2;
                used[best] += add_used;
            }
            wave_sync();
        }

        // ---- eviction: advance the threshold past the least recently used blocks until the LRU fits.  The log of
        // (request, position) touches on this replica is the log of choices, walked from the oldest request routed
        // here; a logged touch still counts iff the table holds exactly its stamp.
        auto evict = [&](int64_t C, int64_t* tau, int32_t* live, int32_t* cur_r, int32_t* cur_k) {
            if (C <= 0 || live[best] <= C) return;
            int E = (int)(live[best] - C);
            int cr = __builtin_amdgcn_readfirstlane(cur_r[best]), ck = __builtin_amdgcn_readfirstlane(cur_k[best]);
            while (E > 0) {
                if (ck == 0) {
                    const int64_t x = next_routed(routed, cr, r, best, lane);
                    if (x >= r) break;          // cannot happen while E > 0; bounds the loop regardless
                    cr = __builtin_amdgcn_readfirstlane((int)x);
                    ck = (int)(b.blk_off[cr + 1] - b.blk_off[cr]);
                    continue;
                }
                // 128 positions of the request, lane order = eviction order (deepest first)
                const int64_t ooff = b.blk_off[cr];
                bool mine[2];
                uint64_t key[2];
                const Slot* const tabs[2] = {tab, tab};
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int k = ck - 1 - g * WAVE - lane;
                    const int64_t at = ooff + (k > 0 ? k : 0);
                    key[g] = b.key[at];
                    mine[g] = b.first[at] != 0 && k >= 0;
                }
                const Found<2> f = find_slots<2, 2>(tabs, key, (mine[0] ? 1u : 0u) | (mine[1] ? 2u : 0u), mask, cap_log2);
                const int from = ck;
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int k = from - 1 - g * WAVE - lane;
                    const bool alive = mine[g] && f.stamp[g] == (int64_t)cr * STAMP_STRIDE + (STAMP_STRIDE - 1 - k);
                    const unsigned long long mk = ballot(alive);
                    const int cnt = __builtin_popcountll(mk);
                    if (E == 0) continue;
                    if (cnt <= E) {
                        E -= cnt;
                        ck = ck > WAVE ? ck - WAVE : 0;
                    } else {
                        const int rank = __builtin_popcountll(mk & ((1ull << lane) - 1));
                        const unsigned long long last = ballot(alive && rank == E - 1);
                        ck = ck - 1 - __builtin_ctzll(last);
                        E = 0;
                    }
                }
            }
            if (lane == 0) {
                cur_r[best] = cr;
                cur_k[best] = ck;
                tau[best] = (int64_t)cr * STAMP_STRIDE + (STAMP_STRIDE - ck);
                live[best] = (int32_t)C + E;
            }
            wave_sync();
        };
        evict(C1, tau1, live1, cur_r1, cur_k1);
        if (two) evict(C2, tau2, live2, cur_r2, cur_k2);
        wave_settle();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");              // (the deciding wavefront reads this replica next)
        now = next;
        next = after;
        meet(true);                                                  // Y(r)
    }
}

template <int MODE, bool ENGINE, bool PROXY>
__global__ void __launch_bounds__(BLOCK_THREADS, 4) replay_blocks_kernel(BlockArgs b) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ QueueHandover<PROXY> comm;
    const int lane = threadIdx.x & (WAVE - 1);
    const int p = blockIdx.x;
    if (threadIdx.x >= 2 * WAVE) {
        queue_wave<MODE, ENGINE, PROXY, 1, true, false>(b.q, 0, lane, lds_raw, &comm);
    } else if (b.q.N > 0) {
        const LruState lru(lds_raw + ((replay_queue_lds_bytes(b.q.R, b.q.B, ENGINE, MODE == MODE_ONLINE ? b.q.window : 0) + 15) & ~(size_t)15),
                           b.q.R);
        if (threadIdx.x < WAVE) block_decide_wave<MODE, ENGINE, PROXY>(b, p, lane, lru, &comm);
        else block_update_wave<PROXY>(b, p, lane, lru, &comm);
    }
}

}  // namespace gorgo
