// Replays whose policy dictates the routes (session affinity, random), one workgroup per replay and replica.
//
// Where a request goes does not depend on the requests before it, so the replicas have nothing to do with each other: a
// replay is R replays of one replica, each with its share of the requests.  The shares are laid out as traces of their own, in
// order of arrival (three kernels), replay_apart.h's wavefronts run them side by side, and the outputs are put back in the
// order of the requests.  A segment's first request on a replica starts its row over there (SEG_FRESH): the loader links
// every reference to the request before it with the same segment, where it has the same place in the path.
// Bound by the longest share's chain, about 0.55 us a request.  One replay of 20,011 requests on 13
// replicas: affinity 10.2 -> 1.1 ms, random 11.0 -> 1.2, of which the layout and the way back take 30 to 45 us.
#pragma once
#include "device_common.h"
#include "internal.h"
#include "replay_apart.h"
#include "replay_segments.h"

namespace gorgo {

constexpr int EACH_CHUNK = 1024;         // requests, and threads, of a workgroup that lays out

struct EachArgs {
    const int64_t *ts, *seg_off, *blk_off;
    const int32_t *in_len, *out_len;
    const SegRef* seg;
    const int32_t* seg_prev;     // request before with the reference's segment, -1: none
    const uint32_t* first_hash;
    const uint64_t* seeds;
    int64_t N, T;                // requests, segment references
    int32_t R, chunks;
    uint8_t* where;              // [P][N] replica of a request
    EachCount* count;            // [P][chunks][R]: a chunk's share, then where it begins
    int32_t* from;               // [P][R+1] first place of a share
    int32_t* list;               // [P][N] request at a place
    int64_t *s_ts, *s_seg_off, *s_blk_off;       // [P][N], [P][N+R], [P][N+R]
    int32_t *s_in, *s_out;       // [P][N]
    SegRef* s_seg;               // [P][T+1]
    uint16_t* hit;               // [P][N] by place, null where nobody wants them
    double *ttft, *e2e;
};

// Routes, and what every chunk sends to every replica.
template <int MODE>
__global__ void __launch_bounds__(EACH_CHUNK) each_route(EachArgs a) {
    __shared__ uint32_t count[WAVE];
    __shared__ unsigned long long segs[WAVE], blocks[WAVE];
    const int tid = threadIdx.x, p = blockIdx.y;
    const int64_t r = (int64_t)blockIdx.x * EACH_CHUNK + tid;
    if (tid < WAVE) {
        count[tid] = 0;
        segs[tid] = blocks[tid] = 0;
    }
    __syncthreads();
    if (r < a.N) {
        const int64_t s = a.seg_off[r + 1] - a.seg_off[r];
        int i;
        if (MODE == MODE_AFFINITY) i = s > 0 ? spread(a.first_hash[r], a.R) : 0;
        else i = spread(philox4x32_10_first((uint32_t)r, 0u, (uint32_t)a.seeds[p], (uint32_t)(a.seeds[p] >> 32)), a.R);
        a.where[(size_t)p * a.N + r] = (uint8_t)i;
        atomicAdd(&count[i], 1u);
        atomicAdd(&segs[i], (unsigned long long)s);
        atomicAdd(&blocks[i], (unsigned long long)(a.blk_off[r + 1] - a.blk_off[r]));
    }
    __syncthreads();
    if (tid < a.R)
        a.count[((size_t)p * a.chunks + blockIdx.x) * a.R + tid] = EachCount{(int64_t)segs[tid], (int64_t)blocks[tid], count[tid]};
}

// Where the shares, and the chunks' parts of them, begin.  One wavefront per replay, lane = replica.
__global__ void __launch_bounds__(WAVE) each_begin(EachArgs a) {
    const int i = threadIdx.x, p = blockIdx.x, R = a.R;
    EachCount* const mine = a.count + (size_t)p * a.chunks * R + (i < R ? i : 0);
    EachCount sum{0, 0, 0};
    if (i < R)
        for (int c = 0; c < a.chunks; ++c) {
            const EachCount x = mine[(size_t)c * R];
            sum.segs += x.segs;
            sum.blocks += x.blocks;
            sum.count += x.count;
        }
    EachCount at{0, 0, 0};
    for (int j = 0; j < R; ++j) {
        const int64_t segs = __shfl(sum.segs, j), blocks = __shfl(sum.blocks, j), count = __shfl(sum.count, j);
        at.segs += j < i ? segs : 0;
        at.blocks += j < i ? blocks : 0;
        at.count += j < i ? count : 0;
    }
    if (i >= R) return;
    a.from[(size_t)p * (R + 1) + i] = (int32_t)at.count;
    const int64_t end = at.count + sum.count;
    if (i == R - 1) a.from[(size_t)p * (R + 1) + R] = (int32_t)end;
    const size_t closing = (size_t)p * (a.N + R) + end + i;          // (a share's offsets have one entry more than it has requests)
    a.s_seg_off[closing] = at.segs + sum.segs;
    a.s_blk_off[closing] = at.blocks + sum.blocks;
    for (int c = 0; c < a.chunks; ++c) {
        const EachCount x = mine[(size_t)c * R];
        mine[(size_t)c * R] = at;
        at.segs += x.segs;
        at.blocks += x.blocks;
        at.count += x.count;
    }
}

// The requests of a chunk, sorted by replica, to their places.
__global__ void __launch_bounds__(EACH_CHUNK) each_place(EachArgs a) {
    constexpr int WAVES = EACH_CHUNK / WAVE;
    __shared__ uint32_t before[WAVES][WAVE];                   // requests of a replica in the wavefronts before
    __shared__ uint32_t begin[WAVE];                           // first of a replica among the chunk's sorted requests
    __shared__ unsigned long long size[EACH_CHUNK], at_begin[WAVE], part[WAVES];      // segments << 32 | blocks
    __shared__ uint16_t who[EACH_CHUNK];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE, p = blockIdx.y, R = a.R;
    const int64_t r0 = (int64_t)blockIdx.x * EACH_CHUNK, N = a.N;
    const int n = (int)(N - r0 < EACH_CHUNK ? N - r0 : EACH_CHUNK);
    const uint8_t* const where = a.where + (size_t)p * N;
    const int mine = tid < n ? where[r0 + tid] : -1;
    int rank = 0;
    before[wave][lane] = 0;
    for (unsigned long long left = __ballot(mine >= 0); left != 0;) {
        const int i = __builtin_amdgcn_readlane(mine, __builtin_ctzll(left));
        const unsigned long long its = __ballot(mine == i);
        if (mine == i) rank = __builtin_popcountll(its & ((1ull << lane) - 1));
        if (lane == 0) before[wave][i] = (uint32_t)__builtin_popcountll(its);
        left &= ~its;
    }
    __syncthreads();
    if (wave == 0) {                     // lane = replica
        uint32_t sum = 0;
        for (int w = 0; w < WAVES; ++w) {
            const uint32_t x = before[w][lane];
            before[w][lane] = sum;
            sum += x;
        }
        uint32_t upto = sum;
        for (int d = 1; d < WAVE; d <<= 1) {
            const uint32_t x = __shfl_up(upto, d);
            upto += lane >= d ? x : 0u;
        }
        begin[lane] = upto - sum;
    }
    __syncthreads();
    if (mine >= 0) {
        const int64_t r = r0 + tid;
        const uint32_t k = begin[mine] + before[wave][mine] + (uint32_t)rank;
        who[k] = (uint16_t)tid;
        size[k] = (unsigned long long)(a.seg_off[r + 1] - a.seg_off[r]) << 32 | (unsigned long long)(a.blk_off[r + 1] - a.blk_off[r]);
    }
    __syncthreads();
    // from here on thread = place among the sorted
    const int64_t r = tid < n ? r0 + who[tid] : 0;
    const unsigned long long own = tid < n ? size[tid] : 0;
    unsigned long long upto = own;
    for (int d = 1; d < WAVE; d <<= 1) {
        const unsigned long long x = __shfl_up(upto, d);
        upto += lane >= d ? x : 0ull;
    }
    if (lane == WAVE - 1) part[wave] = upto;
    __syncthreads();
    for (int w = 0; w < wave; ++w) upto += part[w];
    const unsigned long long first = upto - own;
    const int i = tid < n ? where[r] : 0;
    if (tid < n && (uint32_t)tid == begin[i]) at_begin[i] = first;
    __syncthreads();
    if (tid >= n) return;
    const EachCount base = a.count[((size_t)p * a.chunks + blockIdx.x) * R + i];
    const unsigned long long here = first - at_begin[i];
    const int64_t place = base.count + (tid - (int)begin[i]), off = base.segs + (int64_t)(here >> 32);
    const size_t o = (size_t)p * N + place, oo = (size_t)p * (N + R) + place + i;
    a.list[o] = (int32_t)r;
    a.s_ts[o] = a.ts[r];
    a.s_in[o] = a.in_len[r];
    a.s_out[o] = a.out_len[r];
    a.s_seg_off[oo] = off;
    a.s_blk_off[oo] = base.blocks + (int64_t)(here & 0xFFFFFFFFull);
    SegRef* const to = a.s_seg + (size_t)p * (a.T + 1) + off;
    const int64_t j0 = a.seg_off[r];
    const int s = (int)(own >> 32);
    for (int k = 0; k < s; ++k) {
        SegRef ref = a.seg[j0 + k];
        int32_t q = a.seg_prev[j0 + k];
        while (q >= 0 && where[q] != i) q = a.seg_prev[a.seg_off[q] + k];
        ref.end = (ref.end & ~SEG_FRESH) | (q < 0 ? SEG_FRESH : 0);
        to[k] = ref;
    }
}

template <bool ENGINE>
__global__ void __launch_bounds__(APART_WAVES * WAVE, 4) replay_each_kernel(SegArgs a, EachArgs e) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int b = blockIdx.x, p = b / e.R, i = b % e.R;
    const int32_t from = __builtin_amdgcn_readfirstlane(e.from[(size_t)p * (e.R + 1) + i]);
    const int32_t to = __builtin_amdgcn_readfirstlane(e.from[(size_t)p * (e.R + 1) + i + 1]);
    if (to == from) return;
    const size_t at = (size_t)p * e.N + from, at1 = (size_t)p * (e.N + e.R) + from + i;
    a.N = to - from;
    a.R = 1;
    a.ts = e.s_ts + at;
    a.in_len = e.s_in + at;
    a.out_len = e.s_out + at;
    a.seg_off = e.s_seg_off + at1;
    a.blk_off = e.s_blk_off + at1;
    a.seg = e.s_seg + (size_t)p * (e.T + 1);
    a.last += (size_t)b * a.nseg;
    a.log += at1;
    a.rec += at;
    a.route = nullptr;
    a.hit = e.hit ? e.hit + at : nullptr;
    a.ttft = e.ttft ? e.ttft + at : nullptr;
    a.e2e = e.e2e ? e.e2e + at : nullptr;
    a.rtt += i;
    a.scale += p;
    a.params += 3 * p;
    if (ENGINE) {
        a.eng_a_pf += i;
        a.eng_a_dec += i;
        a.eng_budget += i;
    }
    apart_replay<MODE_GIVEN, ENGINE, false, 1, false>([&]() -> const SegArgs& { return a; }, 0, lds_raw);
}

// Outputs from the places to the requests.
__global__ void __launch_bounds__(EACH_CHUNK) each_return(EachArgs a, uint8_t* route, uint16_t* hit, double* ttft, double* e2e) {
    const int64_t k = (int64_t)blockIdx.x * EACH_CHUNK + threadIdx.x;
    if (k >= a.N) return;
    const size_t row = (size_t)blockIdx.y * a.N, from = row + k, to = row + a.list[from];
    if (route) route[to] = a.where[to];
    if (hit) hit[to] = a.hit[from];
    if (ttft) ttft[to] = a.ttft[from];
    if (e2e) e2e[to] = a.e2e[from];
}

}  // namespace gorgo
