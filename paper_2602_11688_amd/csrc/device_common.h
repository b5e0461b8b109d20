// Device helpers shared by the replay kernels: workgroup-scope memory accessors, wavefront reductions and
// the per-replay queue state (service slots, in-flight records, load signal) kept in LDS.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace gorgo {

constexpr int64_t STAMP_STRIDE = 65536;   // stamp = request * stride + (stride - 1 - position): root newest
constexpr int WAVE = 64;

// In-flight request record, linked per (replica, service slot) in dispatch order.
struct Rec {
    double done;       // time the completion event reaches the proxy
    int32_t next;      // next request on the same service slot, -1 = none
    int32_t tokens;    // input tokens counted in the load signal
};

// All mutable per-replay state in global memory is private to one workgroup; relaxed workgroup-scope
// atomics plus workgroup barriers between phases are what the memory model asks for.
template <class T>
__device__ __forceinline__ T ld(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class T>
__device__ __forceinline__ void st(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The kernel's (first) argument, as one of a workgroup's roles reads it: taken as it stands the compiler loads what any role needs
// before it branches to them, and with that many scalars keeps some in lanes of a vector register, to be read back in the loops.
template <class T>
__device__ __forceinline__ const T& kernel_args() {
    auto k = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(k));
    return *(const T*)k;
}

// A scalar argument that a loop keeps: the compiler otherwise reads it again each time round, where all of a wavefront's accesses
// to LDS have to be waited for along with it.
template <class T>
__device__ __forceinline__ T kept(T x) {
    asm volatile("" : "+s"(x));
    return x;
}

__device__ __forceinline__ double readlane_f64(double v, int src) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, src);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ int64_t readlane_i64(int64_t v, int src) {
    const int lo = __builtin_amdgcn_readlane((int)v, src);
    const int hi = __builtin_amdgcn_readlane((int)(v >> 32), src);
    return ((int64_t)hi << 32) | (unsigned int)lo;
}

// Unsigned minimum of x over the wavefront on the data-parallel-primitive path (no LDS round trip): shifts by
// 1, 2, 4, 8 inside each row of 16 lanes, then the last lane of a row is broadcast into the next row (rows 1
// and 3), then lane 31 into rows 2 and 3; lane 63 holds the result.  Each step is one instruction (the moved
// operand is folded into the minimum); lanes without a source see 0xffffffff.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned dpp_min_u32(unsigned x) {
    const unsigned moved = (unsigned)__builtin_amdgcn_update_dpp((int)0xffffffffu, (int)x, CTRL, ROW_MASK, 0xf, false);
    return moved < x ? moved : x;
}
__device__ __forceinline__ unsigned wave_min_u32(unsigned x) {
    x = dpp_min_u32<0x111, 0xf>(x);   // row_shr:1
    x = dpp_min_u32<0x112, 0xf>(x);   // row_shr:2
    x = dpp_min_u32<0x114, 0xf>(x);   // row_shr:4
    x = dpp_min_u32<0x118, 0xf>(x);   // row_shr:8
    x = dpp_min_u32<0x142, 0xa>(x);   // row_bcast:15 into rows 1, 3
    x = dpp_min_u32<0x143, 0xc>(x);   // row_bcast:31 into rows 2, 3
    return (unsigned)__builtin_amdgcn_readlane((int)x, 63);
}

// Sum of x over the wavefront on the same path (lanes without a source add 0); the sum must fit 32 bits.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ unsigned dpp_add_u32(unsigned x) {
    return x + (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, 0xf, false);
}
// wave_scan_u32: of the lanes up to this one.
__device__ __forceinline__ unsigned wave_scan_u32(unsigned x) {
    x = dpp_add_u32<0x111, 0xf>(x);   // row_shr:1
    x = dpp_add_u32<0x112, 0xf>(x);   // row_shr:2
    x = dpp_add_u32<0x114, 0xf>(x);   // row_shr:4
    x = dpp_add_u32<0x118, 0xf>(x);   // row_shr:8: lane 15 of each row holds the row's sum
    x = dpp_add_u32<0x142, 0xa>(x);   // row_bcast:15 into rows 1, 3
    return dpp_add_u32<0x143, 0xc>(x);   // row_bcast:31 into rows 2, 3
}
__device__ __forceinline__ unsigned wave_sum_u32(unsigned x) { return (unsigned)__builtin_amdgcn_readlane((int)wave_scan_u32(x), 63); }

// Lowest-index minimum over the lanes below `count` (count >= 1; values must not be NaN).  The values are
// compared through the usual order-preserving map of an IEEE double to an unsigned 64-bit key (zeros of
// either sign made equal first), high word first, then the low word among the lanes that tie on the high
// word: two 32-bit reductions instead of one on register pairs, and only one when the high words already decide
// (scores that differ by more than a part in a million).
__device__ __forceinline__ int wave_argmin(double v, int lane, int count) {
    const unsigned long long bits = (unsigned long long)__double_as_longlong(v + 0.0);
    const unsigned hi = (unsigned)(bits >> 32), lo = (unsigned)bits;
    const unsigned neg = (unsigned)((int)hi >> 31);
    const bool in = lane < count;
    const unsigned khi = in ? hi ^ (neg | 0x80000000u) : 0xffffffffu;
    const unsigned klo = lo ^ neg;
    const unsigned mhi = wave_min_u32(khi);
    const bool tie = in && khi == mhi;
    const unsigned long long ties = __ballot(tie);
    if ((ties & (ties - 1)) == 0) return __ffsll(ties) - 1;      // one lane holds the smallest high word: done
    const unsigned mlo = wave_min_u32(tie ? klo : 0xffffffffu);
    const unsigned long long at = __ballot(tie && klo == mlo);
    return __ffsll(at) - 1;
}

__device__ __forceinline__ unsigned long long ballot(bool c) { return __builtin_amdgcn_ballot_w64(c); }

// Queue side of one replay: the R * B service slots (slot b of replica i at index i * B + b) and the requests in
// flight, all of it in LDS.  The in-flight requests of a slot form a list in the order of their completion times; the
// two oldest are in LDS, deeper ones are Rec records in global memory linked in that order.  A request concerns the B
// slots of one replica: lane b looks at slot b, so a ballot finds one that is free, and the one lane that has it writes.
// What has completed is found by comparing every slot's oldest request with the time, 64 slots at a time; every lane
// drops one of its slots' requests at a time, all lanes in parallel.  (Slot state in registers, a set per 64 slots, made
// the service step four copies of itself behind a switch and the compiler carry the sets through every join; with a set
// of 64 to 256 slots and 1,024 replays that queue wavefront was busy 1,110 timed cycles of a request 0.98 us long, this
// one 1,150 of 0.65 us, all of it one request behind the decisions.)
// The load signal itself lives with the cache side, which adds what it dispatches; what completes is subtracted here
// with LDS atomics (integers below 2^53 in doubles: exact in any order).
// These words decide how many replays a CU holds.  A slot's state is therefore told from the completion times and the
// youngest request alone -- none in flight, one, two, a longer list -- and there is no count of requests.
struct SlotQueues {
    struct Slot {
        double free_at;  // time the service slot becomes free
        double h_done;   // completion time of the oldest in-flight request (+inf: none)
        double s_done;   // ... of the second oldest (+inf: none; finite, not yet valid, while its record is on its way)
        int32_t h_tok;   // what the oldest takes from the load signal when it completes
        int32_t s_tok;   // what the second oldest takes from the load signal
        int32_t s_next;  // request after the second oldest (-1: none)
        int32_t tail;    // youngest request of a list of three or more (-1: at most two)
    };
    Slot* slot;          // (40 bytes apart: 16 neighbouring slots lie in different LDS banks)
    uint32_t* kv;        // [slots] engine model: KV tokens held by the request that frees the slot at free_at
    int B, passes;       // passes: sets of 64 slots, at least four
    unsigned inv_b;      // replica of slot g = g * inv_b >> 16 (exact for g < 1,024 + 256, B <= 64)
    unsigned long long lanes;  // lanes that hold a slot of the replica in hand
    double last_start;   // engine model: admission time of the latest request of replica = lane
    // One record per lane can be on its way from global memory: the new second oldest of slot f_slot (-1: none), whose
    // LDS words are not valid until settle() has written them -- one request later, so that a slot whose list goes
    // deeper than two does not make the wavefront wait for memory when its oldest request completes.  (While the
    // record is on its way the slot's `next` word in LDS already works: -1, or the request queued behind the record
    // since; the loaded `next` replaces it only if the record had a successor when it was requested.)
    int f_slot, f_tok, f_next;
    double f_done;

    // (Four sets at least: with only as many as there are, the look at them in a loop, 8 replicas of 8 slots took 3 % longer.)
    static __host__ __device__ constexpr int slots(int R, int B) {
        return R * B <= 4 * WAVE ? 4 * WAVE : (R * B + WAVE - 1) / WAVE * WAVE;
    }
    static __host__ __device__ constexpr size_t bytes(int R, int B, bool engine) {
        return (size_t)slots(R, B) * (sizeof(Slot) + (engine ? 4 : 0));
    }

    // (attach: the words are there already)
    __device__ __forceinline__ void attach(unsigned char* lds, int R, int B_) {
        const int n = slots(R, B_);
        B = B_;
        passes = n / WAVE;
        inv_b = (65536u + (unsigned)B - 1u) / (unsigned)B;
        lanes = B >= WAVE ? ~0ull : (1ull << B) - 1;
        slot = reinterpret_cast<Slot*>(lds);
        kv = reinterpret_cast<uint32_t*>(slot + n);
        last_start = 0.0;
        f_slot = f_next = -1;
        f_tok = 0;
        f_done = INFINITY;
    }
    __device__ __forceinline__ void init(unsigned char* lds, int R, int B_, bool engine, int lane) {
        attach(lds, R, B_);
        for (int g = lane; g < passes * WAVE; g += WAVE) {
            slot[g] = Slot{0.0, INFINITY, INFINITY, 0, 0, -1, -1};
            if (engine) kv[g] = 0;
        }
    }

    // The record that was requested by an earlier retirement has arrived: it becomes the slot's second oldest.
    __device__ __forceinline__ void settle() {
        if (ballot(f_slot >= 0) == 0) return;
        if (f_slot >= 0) {
            slot[f_slot].s_done = f_done;
            slot[f_slot].s_tok = f_tok;
            if (f_next >= 0) slot[f_slot].s_next = f_next;
        }
        f_slot = -1;
    }

    // Bit p: the oldest request of slot p * 64 + lane has completed by t.  Four sets are looked at together, the last four
    // once more where they are not a multiple.
    __device__ __forceinline__ unsigned due(double t, int lane) const {
        auto four = [&](int p) {
            const Slot* const h = &slot[p * WAVE + lane];
            const double d0 = h[0].h_done, d1 = h[WAVE].h_done, d2 = h[2 * WAVE].h_done, d3 = h[3 * WAVE].h_done;
            return (d0 <= t ? 1u : 0u) | (d1 <= t ? 2u : 0u) | (d2 <= t ? 4u : 0u) | (d3 <= t ? 8u : 0u);
        };
        unsigned bits = four(0);
        if (__builtin_expect(passes > 4, 0))                           // (more than 256 slots: rare)
            for (int p = 4; p < passes; p += 4) {
                const int q = p < passes - 4 ? p : passes - 4;
                bits |= four(q) << q;
            }
        return bits;
    }
    // Drop requests whose completion event has reached the proxy (done <= t): the oldest of the slots in `due` and
    // whatever else of theirs has completed.  gone: [R] in LDS, what has left the load signal of each replica.
    // DEFER: the record that moves up in a deep list is fetched without waiting.
    template <bool DEFER>
    __device__ __forceinline__ void retire(unsigned due, double t, const Rec* rec, int lane, double* gone) {
        if (ballot(due != 0) == 0) return;
        if (DEFER) settle();
        do {
            if (due != 0) {
                const int g = __builtin_ctz(due) * WAVE + lane;
                Slot* const l = &slot[g];
                const int h_tok = l->h_tok, up_tok = l->s_tok, x = l->s_next, tail = l->tail;
                const double up = l->s_done;
                const bool deep = tail >= 0;
                __hip_atomic_fetch_add(&gone[(unsigned)g * inv_b >> 16], -(double)h_tok, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                l->h_done = up;
                l->h_tok = up_tok;
                l->s_done = deep ? up : INFINITY;
                l->tail = x == tail ? -1 : tail;
                const bool again = up <= t;                     // the new head has completed too
                if (deep) {
                    // the request that moves into second position (x) comes from memory
                    if (DEFER && !again && f_slot < 0) {
                        f_slot = g;
                        l->s_next = -1;
                        f_done = ld(&rec[x].done);
                        f_tok = ld(&rec[x].tokens);
                        f_next = ld(&rec[x].next);
                    } else {
                        const double x_done = ld(&rec[x].done);
                        const int x_tok = ld(&rec[x].tokens), x_next = ld(&rec[x].next);
                        l->s_done = x_done;
                        l->s_tok = x_tok;
                        l->s_next = x_next;
                    }
                }
                due = again ? due : due & (due - 1);
            }
        } while (ballot(due != 0) != 0);
    }

    // The completion times along a slot's in-flight list increase as long as a replica's round trip time is
    // constant.  When it changes between dispatches (probe epochs), a request can complete at the proxy before one
    // dispatched earlier on the same slot; the list is then kept sorted by completion time instead: this inserts
    // request r (completion `done`, `tok` tokens) into the list of slot s, which holds at least one, the last of which
    // completes after `done`.  An element that has to leave the two LDS positions moves into the record of request r,
    // which r itself does not need then.  `tail` stays the record of the last element (of three or more).
    __device__ __forceinline__ void insert_sorted(int s, int r, double done, int32_t tok, Rec* rec) {
        const bool two = slot[s].s_done < INFINITY, deep = slot[s].tail >= 0;
        if (done < slot[s].h_done || (two && done < slot[s].s_done)) {
            // r goes into LDS; the element in second position, if any, moves to global memory behind it
            if (two) {
                st(&rec[r].done, slot[s].s_done);
                st(&rec[r].tokens, slot[s].s_tok);
                st(&rec[r].next, deep ? slot[s].s_next : (int32_t)-1);
                slot[s].s_next = r;
                if (!deep) slot[s].tail = r;
            } else {
                slot[s].s_next = -1;
            }
            if (done < slot[s].h_done) {
                slot[s].s_done = slot[s].h_done;
                slot[s].s_tok = slot[s].h_tok;
                slot[s].h_done = done;
                slot[s].h_tok = tok;
            } else {
                slot[s].s_done = done;
                slot[s].s_tok = tok;
            }
        } else {
            // r goes between two elements further down: walk to the last one that completes no later
            int32_t prev = -1;               // -1: the second position
            int32_t x = slot[s].s_next;
            for (int steps = 0; steps < r && x >= 0 && !(done < ld(&rec[x].done)); ++steps) {
                prev = x;
                x = ld(&rec[x].next);
            }
            st(&rec[r].done, done);
            st(&rec[r].tokens, tok);
            st(&rec[r].next, x);
            if (prev < 0) slot[s].s_next = r;
            else st(&rec[prev].next, (int32_t)r);
        }
    }

    // Request r joins the list of slot s, which holds at least one (called by one lane).  REORDER: round trip times
    // change.
    template <bool REORDER>
    __device__ __forceinline__ void queue_behind(int s, int r, double done, int weight, Rec* rec) {
        const bool two = slot[s].s_done < INFINITY;
        const int32_t tail = slot[s].tail;
        if (REORDER && done < (!two ? slot[s].h_done : (tail < 0 ? slot[s].s_done : ld(&rec[tail].done)))) {
            insert_sorted(s, r, done, weight, rec);
            return;
        }
        if (!two) {
            slot[s].s_done = done;
            slot[s].s_tok = weight;
            slot[s].s_next = -1;
        } else {
            // third or deeper: goes to global memory, linked behind the youngest
            st(&rec[r].done, done);
            st(&rec[r].next, (int32_t)-1);
            st(&rec[r].tokens, (int32_t)weight);
            if (tail < 0) slot[s].s_next = r;    // (behind the second oldest, whose record may still be on its way)
            else st(&rec[tail].next, (int32_t)r);
            slot[s].tail = r;
        }
    }
    // Request r takes slot s, the k-th of its replica, in the lane concerned; it ends at `end`.  none: the lanes whose slot
    // has nothing in flight.
    template <bool REORDER>
    __device__ __forceinline__ void take_slot(int s, int k, unsigned long long none, int r, double end, double done, int weight, Rec* rec) {
        const unsigned long long it = 1ull << k;
        const unsigned long long empty = it & none;
        if (__builtin_amdgcn_inverse_ballot_w64(empty)) {
            slot[s].free_at = end;
            slot[s].h_done = done;
            slot[s].h_tok = weight;
        }
        if (empty == 0) {
            if (__builtin_amdgcn_inverse_ballot_w64(it)) {
                slot[s].free_at = end;
                queue_behind<REORDER>(s, r, done, weight, rec);
            }
        }
    }

    // The slot with the smallest free time, lowest index on ties.  (Times are >= 0: the order of the bits is the order of the
    // values; mostly one slot alone holds the smallest high word and the low words need not be looked at.)
    __device__ __forceinline__ int earliest(double f, int lane) const {
        const unsigned long long bits = (unsigned long long)__double_as_longlong(f);
        const unsigned hi = lane < B ? (unsigned)(bits >> 32) : 0xffffffffu, lo = (unsigned)bits;
        const unsigned mhi = wave_min_u32(hi);
        unsigned long long ties = ballot(hi == mhi);
        if ((ties & (ties - 1)) != 0) {
            const unsigned mlo = wave_min_u32(hi == mhi ? lo : 0xffffffffu);
            ties &= ballot(lo == mlo);
        }
        return __builtin_ctzll(ties);
    }

    // Service of request r on replica `best` (the stated linear model; reproduces Eq. 1: ttft = rtt + wait +
    // prefill).  Which of the slots that are free takes the request changes no latency and no load signal as long as no
    // later request can arrive at the replica before they are free: with fixed round trip times those free by this
    // arrival, with changing ones (REORDER) those free by the request's own time; one with nothing in flight keeps the
    // lists short.  Only when there is none are they searched for the earliest free time (lowest index on ties).
    // half: half the chosen replica's round trip time; pf, dec: prefill and decode time; weight: what the request takes
    // from the load signal when it completes; due: the slots whose oldest request has completed by `until`, to be brought
    // up to date.  The latencies come back the same in every lane.
    template <bool REORDER>
    __device__ __forceinline__ void serve(int r, int best, double t, double half, double pf, double dec, int weight, Rec* rec,
                                          int lane, double* ttft_out, double* e2e_out, double until, unsigned& due) {
        const int s = best * B + (lane < B ? lane : B - 1);
        const double f = slot[s].free_at;
        const unsigned long long none = ballot(slot[s].h_done == INFINITY);
        const double arrive = t + half;
        double start = arrive;
        int k;
        const unsigned long long ready = ballot(f <= (REORDER ? t : arrive)) & lanes;
        if (ready != 0) {
            const unsigned long long idle = ready & none;
            k = __builtin_ctzll(idle != 0 ? idle : ready);
        } else {
            k = earliest(f, lane);
            const double fv = readlane_f64(f, k);
            start = arrive > fv ? arrive : fv;
        }
        const double first_tok = start + pf;
        const double end = first_tok + dec;
        const double done = end + half;
        *ttft_out = (first_tok + half) - t;
        *e2e_out = done - t;
        due |= due_bit(best, k, lane, done, until);
        take_slot<REORDER>(s, k, none, r, end, done, weight, rec);
    }

    // The bit of `due` of the k-th slot of replica `best`, in its lane, if its request has completed by `until`.  (Told by the
    // lane: as a test of the request first it became a branch on a vector comparison.  1,024 replays of 20,000 requests on 32
    // replicas 12.63 -> 12.47 ms, tuners 14.90 -> 14.68, 777 of the engine model 17.51 -> 17.18.)
    __device__ __forceinline__ unsigned due_bit(int best, int k, int lane, double done, double until) const {
        const unsigned at = (unsigned)(best * B + k);
        const unsigned bit = (unsigned)lane == (at & (WAVE - 1)) ? 1u << (at / WAVE) : 0u;
        return done <= until ? bit : 0u;
    }

    // Engine model: from `start` on, the time at which a request holding `tokens` is admitted, the number of requests running
    // then and a slot that is free.  f, h: when this lane's slot becomes free and the tokens held by what runs in it.
    __device__ __forceinline__ int admission(double f, unsigned h, unsigned tokens, double budget, int lane, double& start, int& n) const {
        int k;
        for (int scans = 0;; ++scans) {
            const bool late = f > start;
            const unsigned long long run_mask = ballot(late) & lanes;
            n = __builtin_popcountll(run_mask);
            k = __ffsll(~run_mask & lanes) - 1;
            if (n == 0) break;
            const bool running = late && lane < B;
            bool fits = n < B;
            if (fits && budget != 0.0) {
                // tokens held by the running requests: two 16-bit halves summed apart (each sum below 2^22)
                const unsigned lo = wave_sum_u32(running ? h & 0xffffu : 0u);
                const unsigned hi = wave_sum_u32(running ? h >> 16 : 0u);
                const double held = (double)hi * 65536.0 + (double)lo;
                fits = held + (double)tokens <= budget;
            }
            if (fits || scans >= B) break;       // (the second test is not reached: every repeat has fewer running)
            // the next time a running request ends (running ones end after `start`: positive, finite)
            const double ends = running ? f : INFINITY;
            start = readlane_f64(ends, wave_argmin(ends, lane, WAVE));
        }
        return k < 0 ? 0 : k;                    // (a free slot exists whenever fewer than B are running)
    }

    // ---- the two halves of a service where they are in the hands of two wavefronts: this one keeps the times the slots become
    // free (and the tokens held, and the latest admissions), the other one the requests in flight.  Any slot that is ready
    // will do, see serve().  They return the slot taken; done: when the completion event reaches the proxy.
    template <bool REORDER>
    __device__ __forceinline__ int start_linear(int best, double t, double half, double pf, double dec, int lane, double* ttft_out,
                                                double* e2e_out, double* done_out) {
        Slot* const l = &slot[best * B + (lane < B ? lane : B - 1)];
        const double f = l->free_at;
        const double arrive = t + half;
        double start = arrive;
        const unsigned long long ready = ballot(f <= (REORDER ? t : arrive)) & lanes;
        int k = __builtin_ctzll(ready | 1ull << 63);
        if (ready == 0) {
            k = earliest(f, lane);
            const double fv = readlane_f64(f, k);
            start = arrive > fv ? arrive : fv;
        }
        const double first_tok = start + pf;
        const double end = first_tok + dec;
        const double done = end + half;
        *ttft_out = (first_tok + half) - t;
        *e2e_out = done - t;
        *done_out = done;
        if (lane == k) l->free_at = end;
        return k;
    }
    __device__ __forceinline__ int start_engine(int best, double t, double half, double pf, double dec_alone, unsigned tokens, double budget,
                                                double slowdown, int lane, double* ttft_out, double* e2e_out, double* done_out) {
        const double arrive = t + half;
        const double before = readlane_f64(last_start, best);
        double start = arrive > before ? arrive : before;
        const int s = best * B + (lane < B ? lane : B - 1);
        int n;
        const int k = admission(slot[s].free_at, kv[s], tokens, budget, lane, start, n);
        last_start = lane == best ? start : last_start;
        const double first_tok = start + pf;
        const double factor = 1.0 + slowdown * (double)n;
        const double dec = dec_alone * factor;
        const double end = first_tok + dec;
        const double done = end + half;
        *ttft_out = (first_tok + half) - t;
        *e2e_out = done - t;
        *done_out = done;
        if (lane == k) {
            slot[s].free_at = end;
            kv[s] = tokens;
        }
        return k;
    }
    // Request r joins the requests in flight on slot s.
    template <bool REORDER>
    __device__ __forceinline__ void enter(int s, int r, double done, int weight, Rec* rec, int lane) {
        Slot* const l = &slot[s];
        const double h_done = l->h_done, s_done = l->s_done;
        const int tail = l->tail;
        if (ballot(h_done == INFINITY) != 0) {
            if (lane == 0) {
                l->h_done = done;
                l->h_tok = weight;
            }
        } else if (REORDER) {
            if (lane == 0) queue_behind<true>(s, r, done, weight, rec);
        } else if (ballot(s_done == INFINITY) != 0) {
            if (lane == 0) {
                l->s_done = done;
                l->s_tok = weight;
                l->s_next = -1;
            }
        } else {
            // the third or deeper; the record that is on its way first, whose wait would be one for these stores as well
            settle();
            if (lane == 0) {
                const long long bits = __double_as_longlong(done);
                *reinterpret_cast<int4*>(&rec[r]) = int4{(int)bits, (int)(bits >> 32), -1, weight};
                if (tail < 0) l->s_next = r;
                else st(&rec[tail].next, (int32_t)r);
                l->tail = r;
            }
        }
    }

    // Service of request r on replica `best` under the engine model of a replica (continuous batching, Sec. 2.2;
    // decode slow-down, Sec. 5 "Exploiting Continuous Batching"; replicas of different speed, Sec. 7).  Requests
    // are admitted in arrival order; a request holding `tokens` KV tokens is admitted at the first time s, not
    // before its arrival nor its predecessor's admission, at which fewer than B requests are running and either
    // none is or their KV tokens plus its own fit the replica's budget (0 = no budget); its decode takes
    // dec_alone * (1 + slowdown * n) with n the requests running at s.  All requests admitted earlier have
    // started by s, so those running at s are the slots with free_at > s: a ballot counts the running ones and finds a
    // free slot, their tokens are summed and the next time one ends is found with wavefront reductions; the scan is
    // repeated from that time until the request fits (at most B times: each repeat has one request fewer running).  The
    // request takes the lowest slot that is free at s; its record joins that slot's in-flight list.
    template <bool REORDER>
    __device__ __forceinline__ void serve_engine(int r, int best, double t, double half, double pf, double dec_alone, int weight,
                                                 unsigned tokens, double budget, double slowdown, Rec* rec, int lane,
                                                 double* ttft_out, double* e2e_out, double until, unsigned& due) {
        const double arrive = t + half;
        const double before = readlane_f64(last_start, best);
        double start = arrive > before ? arrive : before;
        const int s = best * B + (lane < B ? lane : B - 1);
        const double f = slot[s].free_at;
        const unsigned h = kv[s];
        const unsigned long long none = ballot(slot[s].h_done == INFINITY);
        int n;
        const int k = admission(f, h, tokens, budget, lane, start, n);
        last_start = lane == best ? start : last_start;
        const double first_tok = start + pf;
        const double factor = 1.0 + slowdown * (double)n;
        const double dec = dec_alone * factor;
        const double end = first_tok + dec;
        const double done = end + half;
        *ttft_out = (first_tok + half) - t;
        *e2e_out = done - t;
        due |= due_bit(best, k, lane, done, until);
        if (lane == k) kv[s] = tokens;           // two counts below 2^31 each
        take_slot<REORDER>(s, k, none, r, end, done, weight, rec);
    }
};

// Index of the next request after `after` (exclusive) and before `limit` that was routed to `replica`, or
// `limit` if there is none: the per-replica touch log is the route array itself.
__device__ __forceinline__ int64_t next_routed(const uint8_t* route, int64_t after, int64_t limit, int replica,
                                               int lane) {
    int64_t x = after + 1;
    while (x < limit) {
        const int64_t y = x + lane;
        const bool hitb = y < limit && ld(&route[y]) == (uint8_t)replica;
        const uint64_t mk = __ballot(hitb);
        if (mk) return x + __ffsll((unsigned long long)mk) - 1;
        x += WAVE;
    }
    return limit;
}

}  // namespace gorgo
