// Vertex-inclusion probabilities, Proposition 1 (Sec. 3.1), in pull form over row blocks.
//
// Per hop h every vertex v carries y_h(v) = log1p(-x_h(v)), x_h(v) = min(1, f_h/d(v)) * p^[h-1](v)
// (0 for d(v) = 0), stored as fp32.  Then eq. (2) is
//     S_h(u) = sum over {v : u in adj(v)} of y_h(v)     (all terms <= 0: no cancellation; fp64 sums)
//     p^[h](u) = -expm1(S_h(u))
// and because log(1 - p^[h](u)) = S_h(u), eq. (1) is p(u) = -expm1(sum_h S_h(u)).
//
// Dense hops: the edges are stored grouped by blocks of 2^14 destination rows and sorted by source
// inside a block.  A workgroup keeps the block's fp64 sums in LDS (128 KB), streams a share of the
// block's edges (4 bytes each, read as 128-bit vectors) and adds y[source] to the row's sum with an
// LDS atomic; because the sources ascend, 64 consecutive edges need a short stretch of y, which the
// wavefront holds in LDS where the edges are dense, and a line fetched from L2 serves every edge of
// the block that needs it.  (A pull that walks one row's in-list at a time fetches a line per edge: it
// ran at a third of this rate on every graph measured, from 2.4M to 134M vertices.)  A second kernel
// adds the shares and finishes the vertex (p^[h], running total, next hop's y).
//
// Early hops touch few edges (hop 1 only the rows of T), so the kernel that writes a hop's y also
// lists the hop's frontier (vertices with y != 0) and counts its out-edges; when that is a small share of
// the graph the hop is done in push form instead: each frontier vertex adds its y to the fp64 accumulator of
// every member of its row (atomic adds, and one pass finishes all vertices; on large graphs through bins of
// the row blocks, which finish their vertices).  Which form a hop takes is decided on the device, by the last
// workgroup of the kernel that counts (reading the frontier's size back cost the host 35 to 60 us per hop, with nothing
// queued behind it); a launch then walks the hop in the form it takes.  A call is two launches and two per hop:
// on small graphs they set its time.
#include "spp_common.h"
#include "spp_device.h"
#include "spp_fp32.h"
#include "spp_fp64.h"

#include <type_traits>

namespace spp {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int64_t kPushShare = 16;       // push when the frontier's out-edges are at most M/16
constexpr int kSegments = 2048;          // most workgroups of a kernel that lists a frontier: each has a segment of the list
constexpr uint32_t kPushed = 1, kPulled = 2;

// What the kernel that writes a hop's y leaves for that hop's walk.  The frontier's vertices are listed per workgroup, in any
// order, in a segment of `seg_cap` entries (no workgroup waits for another's count): from its start on, and those with more
// than kLongRow entries from its end back: those are shared out edge by edge (see push_frontier), which costs every workgroup
// the look at all of them.  Hop 1 of 2.4M vertices: 1000 rows of 4000 entries 200 us shared out, 468 in portions of 64 rows;
// 2000 of 2000, 200 and 258; 10000 of 400, 229 and 200; the 24k training vertices of a power law (up to 20000 entries), 81 for
// limits of 1024 to 4096, 84 below.
constexpr int64_t kLongRow = 1024;
struct HopList {
    int32_t*  list;
    uint32_t* seg_count;                 // per segment how many from its start, and from its end; null: not listed here (large
                                         // graphs list the frontier in a launch of its own)
    int64_t   seg_cap;
    int       nseg;
};
struct HopPlan {
    int       h;                         // the hop whose frontier this is
    int64_t   M;
    unsigned long long* slots;           // see grid_total
    uint32_t* how;                       // [1 .. L]
    unsigned long long* cursor;          // of the list made in a launch of its own
    int64_t*  mirror;                    // pinned host memory: per hop pushed?, frontier edges or -1
    HopList   l;
};

struct VipHop {
    const int64_t* rowptr;     // forward CSR, for d(u)
    float*         y_next;     // next hop's y (unused at the last hop)
    double*        tot;        // running sum of S over hops
    float*         p_hop;      // p^[h] or null
    float*         p_total;    // written at the last hop
    double         f_next;     // f_{h+1}
    int            first;      // first hop and hop 0 not included: tot is not read
    int            last;
    HopPlan        next;       // unused at the last hop
    int*           bad;        // first hop: the flag for bad training ids, emptied again, and where it goes; else null
    int64_t*       bad_mirror;
};

// Finishes vertices u, u + step, ... (U of them, those below N).  S = their sums, told = their running totals (ignored
// at a first hop).  The loads and the chains of arithmetic of the U vertices are independent.  emit(vertex, degree) is
// called for the next hop's frontier.
template <int U, class Emit>
__device__ __forceinline__ void vip_finish_vertices(const VipHop& a, int64_t u, int64_t step, int64_t N, const double (&S)[U],
                                                    const double (&told)[U], unsigned long long& edges, Emit emit) {
    // A vertex that no frontier vertex points at has S = 0 exactly (most vertices, at the early hops):
    // its p^[h] is 0 and it needs no exponential; nor does p^[h] at the last hop when it is not asked for.
    double ph[U];
    bool some = false;
#pragma unroll
    for (int k = 0; k < U; ++k) { ph[k] = 0.0; some |= S[k] != 0.0; }
    if (some && (a.p_hop != nullptr || !a.last))
#pragma unroll
        for (int k = 0; k < U; ++k) ph[k] = one_minus_exp(S[k]);        // 0 for a sum of 0
    if (a.p_hop)
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (u + k * step < N) a.p_hop[u + k * step] = (float)ph[k];
    double T[U];
#pragma unroll
    for (int k = 0; k < U; ++k) T[k] = a.first ? S[k] : told[k] + S[k];
    if (a.last) {
        bool any = false;
#pragma unroll
        for (int k = 0; k < U; ++k) any |= T[k] != 0.0;
        double p[U] = {};
        if (any)
#pragma unroll
            for (int k = 0; k < U; ++k) p[k] = one_minus_exp(T[k]);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (u + k * step < N) a.p_total[u + k * step] = (float)p[k];
        return;
    }
    int64_t d[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        d[k] = 0;
        if (ph[k] > 0.0 && u + k * step < N) d[k] = a.rowptr[u + k * step + 1] - a.rowptr[u + k * step];
    }
    float yn[U];
#pragma unroll
    for (int k = 0; k < U; ++k) yn[k] = 0.0f;
    if (some)
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const double dd = (double)d[k];
            const double t = dd <= a.f_next ? 1.0 : small_quotient(a.f_next, dd);
            if (d[k] > 0) yn[k] = (float)log1p_neg(t * ph[k]);
            if (yn[k] != 0.0f) {
                edges += (unsigned long long)d[k];
                emit(u + k * step, d[k]);
            }
        }
#pragma unroll
    for (int k = 0; k < U; ++k)
        if (u + k * step < N) {
            a.tot[u + k * step] = T[k];
            a.y_next[u + k * step] = yn[k];
        }
}

// The next hop's weights of U vertices whose sums are not zero (the others' are).  All threads call it with their vertices'
// own ones; those without `has` come away with zeros.
template <int U>
__device__ __forceinline__ void vip_next_weights(const VipHop& a, const int64_t (&v)[U], const double (&S)[U], const bool (&has)[U],
                                                 float (&ph32)[U], float (&yn)[U], unsigned long long& edges) {
    double ph[U];
    int64_t d[U];
#pragma unroll
    for (int k = 0; k < U; ++k) d[k] = a.rowptr[has[k] ? v[k] + 1 : 0] - a.rowptr[has[k] ? v[k] : 0];
#pragma unroll
    for (int k = 0; k < U; ++k) ph[k] = has[k] ? one_minus_exp(S[k]) : 0.0;
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const double dd = (double)d[k];
        const double t = dd <= a.f_next ? 1.0 : small_quotient(a.f_next, dd);
        ph32[k] = (float)ph[k];
        yn[k] = d[k] > 0 ? (float)log1p_neg(t * ph[k]) : 0.0f;
        edges += yn[k] != 0.0f ? (unsigned long long)d[k] : 0ull;
    }
}

// The kWaveRows vertices from u0 on whose sums a wavefront holds in LDS, after a hop that is not the last: the arithmetic of those
// with a sum alone, 64 lanes at a time (most vertices have none at the early hops: 5 and 25 % of 14M vertices have, spread
// over nearly all wavefronts; the arithmetic of all of them took two thirds of the kernel).  queue: kTouchedQueue entries.
constexpr int kWaveRows = 1024, kTouchedQueue = 512;
__device__ __forceinline__ void vip_finish_touched(const VipHop& a, int64_t u0, int64_t N, double* acc, uint16_t* queue,
                                                   unsigned long long& edges) {
    constexpr int U = 4, kBatch = U * kWave;
    const int lane = lane_id();
    int queued = 0;
    auto finish = [&](int n) {                   // the last n of the queue, at most kBatch
        wave_lds_order();
        int i[U];
        int64_t v[U];
        double S[U];
        bool has[U];
        float ph[U], yn[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            has[k] = k * kWave + lane < n;
            i[k] = has[k] ? queue[queued - n + k * kWave + lane] : 0;
            v[k] = u0 + i[k];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) S[k] = acc[i[k]];
        vip_next_weights<U>(a, v, S, has, ph, yn, edges);
        wave_lds_order();
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (has[k]) acc[i[k]] = __hiloint2double(__float_as_int(ph[k]), __float_as_int(yn[k]));      // in place of its sum
        queued -= n;
        wave_lds_order();
    };
    for (int b = 0; b < kWaveRows && u0 + b < N; b += kBatch) {
        double S[U], T0[U];
#pragma unroll
        for (int k = 0; k < U; ++k) S[k] = acc[b + k * kWave + lane];
        if (!a.first)
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int64_t u = u0 + b + k * kWave + lane;
                T0[k] = a.tot[u < N ? u : N - 1];
            }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int i = b + k * kWave + lane;
            const bool inside = u0 + i < N, some = inside && S[k] != 0.0;
            if (a.first ? inside : some) a.tot[u0 + i] = a.first ? S[k] : T0[k] + S[k];
            const uint64_t m = __ballot(some);
            if (some) queue[queued + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] = (uint16_t)i;
            queued += __popcll(m);
        }
        if (queued >= kBatch) finish(kBatch);
    }
    if (queued > 0) finish(queued);              // fewer than kBatch
    wave_lds_order();
    for (int i = lane; i < kWaveRows && u0 + i < N; i += kWave) {
        const double r = acc[i];                 // zeros where there was no sum
        a.y_next[u0 + i] = __int_as_float(__double2loint(r));
        if (a.p_hop) a.p_hop[u0 + i] = __int_as_float(__double2hiint(r));
    }
}

// All vertices, grid-stride, four per thread and round: the four sums and running totals are in
// flight together (one vertex per round leaves a pass over 10^8 vertices waiting on its own loads:
// 0.87 ms where the bytes take 0.55).  sum_of(u) = S_h(u).
template <class SumOf, class Emit>
__device__ __forceinline__ void vip_finish_all(const VipHop& a, int64_t N, SumOf sum_of, unsigned long long& edges, Emit emit) {
    constexpr int U = 4;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x; u < N; u += U * stride) {
        double S[U], T0[U];
#pragma unroll
        for (int k = 0; k < U; ++k) S[k] = u + k * stride < N ? sum_of(u + k * stride) : 0.0;
#pragma unroll
        for (int k = 0; k < U; ++k) T0[k] = a.first || u + k * stride >= N ? 0.0 : a.tot[u + k * stride];
        vip_finish_vertices<U>(a, u, stride, N, S, T0, edges, emit);
    }
}

// The R vertices from u0 on whose sums a workgroup of 1024 threads holds in LDS.
template <int R>
__device__ __forceinline__ void vip_finish_block(const VipHop& a, int64_t u0, int64_t N, const double* acc,
                                                 unsigned long long& edges) {
    constexpr int U = 4, kThreads = 1024;
    for (int i = threadIdx.x; i < R && u0 + i < N; i += U * kThreads) {
        double S[U], T0[U];
#pragma unroll
        for (int k = 0; k < U; ++k) S[k] = acc[i + k * kThreads];
#pragma unroll
        for (int k = 0; k < U; ++k) T0[k] = a.first || u0 + i + k * kThreads >= N ? 0.0 : a.tot[u0 + i + k * kThreads];
        vip_finish_vertices<U>(a, u0 + i, kThreads, N, S, T0, edges, [](int64_t, int64_t) {});
    }
}

template <int kThreads>
__device__ __forceinline__ unsigned long long workgroup_sum(unsigned long long x) {      // in thread 0
    __shared__ unsigned long long red[kThreads / kWave];
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) x += __shfl_down((long long)x, off, kWave);
    if (lane_id() == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    unsigned long long all = 0;
    if (threadIdx.x == 0)
        for (int w = 0; w < kThreads / kWave; ++w) all += red[w];
    return all;
}

// Adds up one number per workgroup of a launch without a launch of its own: `slots` holds kTotalSlots words, all zero
// between uses.  A word counts its arrivals above bit 48 beside their sum, so the arrival that completes it has the
// sum and nothing has to be fenced; 64 workgroups share a word, the last of each group adds to the first word.  Atomics on
// one address cost about 15 ns each, and so do those on one 128-byte line: each word has a line of its own (side by side,
// 2048 workgroups took 9 us).  Called by one thread of every workgroup; true for the one that arrives
// last, which has the total.  A workgroup's number counts as 2^33 at most.
__device__ __forceinline__ bool grid_total(unsigned long long* slots, unsigned long long mine, unsigned long long& total) {
    constexpr unsigned long long kOne = 1ull << 48, kMost = 1ull << 33;
    unsigned long long* s = slots + (1 + blockIdx.x / 64) * kTotalLine;
    const unsigned first = blockIdx.x & ~63u, members = gridDim.x - first < 64u ? gridDim.x - first : 64u;
    unsigned long long v = (mine < kMost ? mine : kMost) + kOne;
    v += atomicAdd(s, v);
    if ((v >> 48) != members) return false;
    atomicExch(s, 0ull);
    v = (v & (kOne - 1)) + kOne;
    v += atomicAdd(slots, v);
    if ((v >> 48) != (gridDim.x + 63u) / 64u) return false;
    atomicExch(slots, 0ull);
    total = v & (kOne - 1);
    return true;
}

// How a hop is walked: pushed if its frontier's out-edges are at most M / kPushShare; pulled without looking after a pulled
// hop (frontiers that have grown large rarely shrink, and either form is correct for any frontier).  Called by all
// threads of every workgroup of the kernel that counted the edges.
template <int kThreads>
__device__ __forceinline__ void plan_hop(const HopPlan& p, unsigned long long edges) {
    const unsigned long long mine = workgroup_sum<kThreads>(edges);
    unsigned long long all;
    if (threadIdx.x == 0 && grid_total(p.slots, mine, all)) {
        const bool push = all * kPushShare <= (unsigned long long)p.M;
        p.how[p.h] = push ? kPushed : kPulled;
        *p.cursor = 0ull;
        p.mirror[2 * (p.h - 1)] = push ? 1 : 0;
        p.mirror[2 * (p.h - 1) + 1] = (int64_t)all;
    }
}
// By one thread of the kernel that finishes a hop's vertices.
__device__ __forceinline__ void hop_done(const VipHop& a, bool pulled) {
    if (a.bad) { *a.bad_mirror = *a.bad; *a.bad = 0; }
    if (!pulled || a.last) return;
    const HopPlan& p = a.next;
    p.how[p.h] = kPulled;
    p.mirror[2 * (p.h - 1)] = 0;
    p.mirror[2 * (p.h - 1) + 1] = -1;
}

__global__ void fill_f64_kernel(double* p, int64_t n, double v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {        // 128-bit stores for the bulk
        typedef double f64x2 __attribute__((ext_vector_type(2)));
        const f64x2 vv = {v, v};
        f64x2* p2 = reinterpret_cast<f64x2*>(p);
        for (int64_t i = tid; i < (n >> 1); i += stride) p2[i] = vv;
        if (tid == 0 && (n & 1)) p[n - 1] = v;
        return;
    }
    for (int64_t i = tid; i < n; i += stride) p[i] = v;
}

// What a propagation starts from: no weights, no totals (if hop 0 counts), empty accumulators (if hops add to them
// directly).
__global__ void __launch_bounds__(kBlock) vip_clear_kernel(float* __restrict__ y, double* __restrict__ tot, double* __restrict__ acc, int64_t N) {
    const int64_t stride = (int64_t)gridDim.x * kBlock, tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    for (int64_t i = tid; i < (N + 3) / 4; i += stride) reinterpret_cast<f32x4*>(y)[i] = z;      // y holds a vector more than N
    if (tot)
        for (int64_t i = tid; i < N; i += stride) tot[i] = 0.0;
    if (acc) {                                   // holds an even number
        typedef double f64x2 __attribute__((ext_vector_type(2)));
        for (int64_t i = tid; i < (N + 1) / 2; i += stride) reinterpret_cast<f64x2*>(acc)[i] = f64x2{0.0, 0.0};
    }
}

// Exclusive prefix sums over a workgroup of kThreads threads; ends with a barrier.
template <int kThreads>
__device__ __forceinline__ uint32_t bin_block_scan(uint32_t v, uint32_t (&wave_sum)[kThreads / kWave], uint32_t& total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t inc = (uint32_t)wave_inclusive_scan((int)v);
    if (lane == kWave - 1) wave_sum[wave] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) {
        const uint32_t x = wave_sum[w];
        if (w < wave) before += x;
        all += x;
    }
    total = all;
    __syncthreads();
    return before + inc - v;
}

// The frontier itself (any order): list[0 .. *cursor) = vertices whose y is not zero and whose row
// is not empty; a row of more than kPieceEdges entries is listed once per piece of that many
// entries (adjacent in the list), so that the kernels that walk the frontier's rows can hand the
// pieces of a long row to different workgroups.  A thread looks at kListPer vertices (as 128-bit vectors),
// first to count its entries and, once the workgroup has reserved its part of the list with one
// atomic, again to write them (the second look finds its lines in the caches).  Same-address
// atomics cost about 15 ns each, so what a round covers sets the pace on a large graph: with 8
// vertices per thread a dense frontier of 10^8 vertices took 0.72 ms (54k atomics), with 64 the
// pass is bound by reading y.  Small graphs keep 8 per thread (enough workgroups to fill the chip).
constexpr int64_t kPieceEdges = 4096;
__host__ __device__ inline int64_t frontier_list_capacity(int64_t N, int64_t M) { return N + M / kPieceEdges; }

// With `how`: only if the hop is pushed.
// `lds`: kThreads / kWave words for a scan, and two more.
template <int kThreads, int kListPer>
__device__ __forceinline__ void list_frontier(const float* __restrict__ y, const int64_t* __restrict__ rowptr, int64_t N,
                                              int32_t* __restrict__ list, unsigned long long* __restrict__ cursor,
                                              uint32_t* lds) {
    unsigned long long& start = *reinterpret_cast<unsigned long long*>(lds);
    uint32_t (&wave_sum)[kThreads / kWave] = *reinterpret_cast<uint32_t(*)[kThreads / kWave]>(lds + 2);
    const int64_t round = (int64_t)kThreads * kListPer;
    auto pieces = [&](int64_t v) { return (int)((rowptr[v + 1] - rowptr[v] + kPieceEdges - 1) / kPieceEdges); };
    for (int64_t r0 = (int64_t)blockIdx.x * round; r0 < N; r0 += (int64_t)gridDim.x * round) {
        // A wavefront covers kWave * kListPer consecutive vertices; lane l takes the 128-bit vectors
        // l, 64 + l, 128 + l, ... of them (whole lines per load).  Bit 4 k + c of nz: component c of the
        // lane's k-th vector is in the frontier.  (y is 16-byte aligned and w0 a multiple of four.)
        const int64_t w0 = r0 + (int64_t)(threadIdx.x >> 6) * (kWave * kListPer);
        auto vertex = [&](int bit) { return w0 + 4 * ((int64_t)(bit >> 2) * kWave + lane_id()) + (bit & 3); };
        uint64_t nz = 0;
#pragma unroll
        for (int k = 0; k < kListPer / 4; ++k) {
            const int64_t v = vertex(4 * k);
            if (v + 3 < N) {
                const f32x4 t = *reinterpret_cast<const f32x4*>(y + v);
                nz |= (uint64_t)((t.x != 0.0f) | ((t.y != 0.0f) << 1) | ((t.z != 0.0f) << 2) | ((t.w != 0.0f) << 3)) << (4 * k);
            } else {
                for (int c = 0; c < 4; ++c)
                    if (v + c < N && y[v + c] != 0.0f) nz |= 1ull << (4 * k + c);
            }
        }
        uint32_t mine = 0;
        for (uint64_t m = nz; m; m &= m - 1) mine += (uint32_t)pieces(vertex(__builtin_ctzll(m)));
        uint32_t total;
        uint32_t at = bin_block_scan<kThreads>(mine, wave_sum, total);
        if (total == 0) continue;        // uniform over the workgroup: the scan has synchronised it
        if (threadIdx.x == 0) start = atomicAdd(cursor, (unsigned long long)total);
        __syncthreads();
        const unsigned long long base = start;
        for (uint64_t m = nz; m; m &= m - 1) {
            const int64_t v = vertex(__builtin_ctzll(m));
            for (int c = pieces(v); c > 0; --c) list[base + at++] = (int32_t)v;
        }
        __syncthreads();
    }
}

template <int kListPer>
__global__ void __launch_bounds__(kBlock) vip_frontier_list_kernel(const float* __restrict__ y, const int64_t* __restrict__ rowptr,
                                                                   int64_t N, int32_t* __restrict__ list,
                                                                   unsigned long long* __restrict__ cursor,
                                                                   const uint32_t* __restrict__ how) {
    __shared__ __align__(8) uint32_t lds[2 + kBlock / kWave];
    if (how && *how != kPushed) return;
    list_frontier<kBlock, kListPer>(y, rowptr, N, list, cursor, lds);
}
inline void launch_frontier_list(int grid, hipStream_t st, const float* y, const int64_t* rowptr, int64_t N, int32_t* list,
                                 unsigned long long* cursor, const uint32_t* how = nullptr) {
    if (N >= (int64_t)1 << 22) vip_frontier_list_kernel<64><<<grid, kBlock, 0, st>>>(y, rowptr, N, list, cursor, how);
    else vip_frontier_list_kernel<8><<<grid, kBlock, 0, st>>>(y, rowptr, N, list, cursor, how);
}

// Entry i of that list: where its piece of the row starts in col[] and how many entries it has.
// The pieces of a row are adjacent and in order, so the number of the piece is the distance to
// the first entry with the same vertex (found by galloping, then bisection).
__device__ __forceinline__ int32_t frontier_entry(const int32_t* __restrict__ list, int64_t i,
                                                  const int64_t* __restrict__ rowptr, int64_t& row, uint32_t& deg) {
    const int32_t v = list[i];
    int64_t lo = i, step = 1;                               // list[lo] == v
    while (lo - step >= 0 && list[lo - step] == v) { lo -= step; step <<= 1; }
    int64_t a = lo - step < 0 ? -1 : lo - step;             // a == -1 or list[a] != v
    while (lo - a > 1) {
        const int64_t mid = (a + lo) >> 1;
        if (list[mid] == v) lo = mid; else a = mid;
    }
    const int64_t b = rowptr[v] + (i - lo) * kPieceEdges, e = rowptr[v + 1];
    row = b;
    deg = (uint32_t)(e - b < kPieceEdges ? e - b : kPieceEdges);
    return v;
}

// Puts a vertex of the next frontier on this workgroup's list; `n`: its two counters, in LDS.
__device__ __forceinline__ void list_vertex(const HopList& l, uint32_t (&n)[2], int64_t v, int64_t d) {
    int32_t* segment = l.list + (int64_t)blockIdx.x * l.seg_cap;
    if (d > kLongRow) segment[l.seg_cap - 1 - atomicAdd(&n[1], 1u)] = (int32_t)v;
    else segment[atomicAdd(&n[0], 1u)] = (int32_t)v;
}

// Finishes all vertices: after a push from the accumulators, which it empties again, after a pull from the shares' sums
// (unless the pull has finished its vertices itself).
__global__ void __launch_bounds__(kBlock) vip_finish_kernel(VipHop a, const uint32_t* __restrict__ how, int fused_pull,
                                                            double* __restrict__ acc, int parts, int64_t part_stride,
                                                            int64_t N) {
    __shared__ uint32_t listed[2];
    const bool push = *how == kPushed;
    if (blockIdx.x == 0 && threadIdx.x == 0) hop_done(a, !push);
    unsigned long long edges = 0;
    if (push) {
        if (threadIdx.x < 2) listed[threadIdx.x] = 0u;
        __syncthreads();
        vip_finish_all(a, N, [&](int64_t u) {
            const double S = acc[u];
            if (S != 0.0) acc[u] = 0.0;
            return S;
        }, edges, [&](int64_t v, int64_t d) { list_vertex(a.next.l, listed, v, d); });
        if (a.last) return;
        plan_hop<kBlock>(a.next, edges);         // its barrier: everything is listed
        if (threadIdx.x < 2) a.next.l.seg_count[2 * blockIdx.x + threadIdx.x] = listed[threadIdx.x];
        return;
    }
    if (fused_pull) return;
    vip_finish_all(a, N, [&](int64_t u) {
        double S = acc[u];
        for (int j = 1; j < parts; ++j) S += acc[(int64_t)j * part_stride + u];
        return S;
    }, edges, [](int64_t, int64_t) {});
}

// Dense hops, blocked: one workgroup takes the j-th of `parts` shares of the edges that end in one
// block of 2^rbits destination rows.  The block's fp64 sums live in LDS; the edges are sorted by
// source.  The share's sums are written to part[j][row]; the finish kernel adds the shares.  A share is
// the j-th part of each of the block's sixteenths, one per wavefront: stretches where the LDS adds
// set the pace and stretches where the gathers do then run side by side on a CU, and shares are alike
// (contiguous shares: 190 us instead of 171).
// An edge is one 32-bit word (low 18 bits of the source, row inside the block); the source's high
// bits follow from the edge's position: the block's chunk bounds sit in LDS next to the sums.
//
// Gathered from memory, a y per edge costs the CU's address path a clock per lane: 196 us for 121M edges,
// which is what the kernel took.  So a wavefront, which takes 512 consecutive edges per round, reads
// the stretch of y that they need into a window of its own in LDS where that is at most kTileSpan values
// (1.2 edges and more per source and row block: edges inside a partition), and the edges read the
// window.  The stretch is known as soon as the round's first and last words have arrived, so the words
// are asked for two rounds ahead and the window one round ahead.  Elsewhere the edges gather as before,
// eight gathers per lane in flight.  (Deciding per 64 edges instead of per 512 took 315 us: a
// wavefront's instruction occupies its SIMD for four clocks, and there were five times as many.)
// 2.4M vertices, 121M edges: 171 us per hop instead of 211.  What bounds it now: the word stream alone
// takes 98 us at the one workgroup per CU that the sums allow, the LDS adds (26 clocks per 64 edges)
// 78, clearing and writing the sums 23, and the three overlap in part; more rounds of words in flight
// (two, three or six more) change nothing.
constexpr int kTileBlock = 1024;
constexpr int kTileWaves = kTileBlock / kWave;
constexpr int kTileUnroll = 2;          // 128-bit vectors (four edges) per lane and round
constexpr int kTileRound = kTileUnroll * kWave;      // vectors of a wavefront's round
constexpr uint32_t kTileWin = 448;      // what 160 KB of LDS leave per wavefront beside the block's sums (16384 in fp64)
constexpr uint32_t kTileSpan = kTileWin - 4;
static_assert(kTileWaves * kTileWin * sizeof(float) == kTileWinBytes, "the layout was built for this much LDS beside the sums");
__device__ __forceinline__ void pull_tiles(double* acc, const uint32_t* __restrict__ t_edge,
                                           const int64_t* __restrict__ first, int nch, int64_t nrb, int parts,
                                           int rbits, uint32_t N, const float* __restrict__ y,
                                           double* __restrict__ part, int64_t part_stride) {
    const int R = 1 << rbits;
    float* win = reinterpret_cast<float*>(acc + R) + (threadIdx.x >> 6) * kTileWin;      // this wavefront's
    uint32_t* bound = reinterpret_cast<uint32_t*>(acc + R) + kTileWaves * kTileWin;
    // share-major order: the workgroups that run at the same time take the same share of different
    // blocks, i.e. the same parts of y
    if ((int64_t)blockIdx.x >= nrb * parts) return;
    const int64_t rb = blockIdx.x % nrb;
    const int j = (int)(blockIdx.x / nrb);
    const int64_t b0 = first[rb * nch], len = first[(rb + 1) * nch] - b0;
    for (int i = threadIdx.x; i < R; i += kTileBlock) acc[i] = 0.0;
    for (int c = threadIdx.x; c <= nch; c += kTileBlock) bound[c] = (uint32_t)(first[rb * nch + c] - b0);
    __syncthreads();
    const uint32_t lane = lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t piece = (int64_t)wave * parts + j;         // this wavefront's of the block's 16 * parts equal pieces
    const int64_t beg = b0 + len * piece / (kTileWaves * parts), end = b0 + len * (piece + 1) / (kTileWaves * parts);
    // The edge stream is read four edges per lane (one 128-bit load): a CU keeps a limited number
    // of misses in flight, so the bytes per request decide the streaming rate.
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    int64_t a4 = (beg + 3) & ~(int64_t)3, e4 = end & ~(int64_t)3;
    if (a4 > end) a4 = end;
    if (e4 < a4) e4 = a4;
    auto one = [&](int64_t e) {
        const uint32_t w = t_edge[e];
        const float v = y[tile_source(w, tile_chunk_of(bound, nch, (uint32_t)(e - b0)))];
        if (v != 0.0f) unsafeAtomicAdd(&acc[w & kTileRowMask], (double)v);
    };
    if (beg + lane < a4) one(beg + lane);        // unaligned head and tail, three edges at most
    if (e4 + lane < end) one(e4 + lane);
    const u32x4* __restrict__ vs = reinterpret_cast<const u32x4*>(t_edge + a4);
    const uint32_t nvec = (uint32_t)((e4 - a4) >> 2);
    const uint32_t p0 = (uint32_t)(a4 - b0);                                   // position of the first vector's first edge
    const f32x4* __restrict__ y4 = reinterpret_cast<const f32x4*>(y);          // 16-byte aligned, a vector longer than N
    constexpr uint32_t kStep = kTileRound;
    struct Words { u32x4 v[kTileUnroll]; };
    auto load = [&](uint32_t q0) {               // the words of the round that starts at vector q0
        Words w;
#pragma unroll
        for (int u = 0; u < kTileUnroll; ++u)
            if (q0 + u * kWave + lane < nvec) w.v[u] = __builtin_nontemporal_load(vs + (q0 + u * kWave + lane));
        return w;
    };
    // how a round's edges find their values: in the window (from source w0 on), by gathers from one chunk of
    // sources, or edge by edge (the last round, and rounds that cross into another chunk)
    enum { kWindow, kGather, kEach };
    int c = __builtin_amdgcn_readfirstlane(tile_chunk_of(bound, nch, p0));   // chunk of the latest round looked at; positions only grow
    uint32_t cend = (uint32_t)__builtin_amdgcn_readfirstlane((int)bound[c + 1]);
    f32x4 y0 = {0.f, 0.f, 0.f, 0.f}, y1 = y0;    // the window on its way
    auto look = [&](uint32_t q0, const Words& w, uint32_t& base, uint32_t& w0) {
        if (q0 + kTileRound > nvec) return (int)kEach;
        const uint32_t at = p0 + 4 * q0;         // at + 511 < len = bound[nch]: c stays below nch
        while (at >= cend) { ++c; cend = (uint32_t)__builtin_amdgcn_readfirstlane((int)bound[c + 1]); }
        if (at + 4 * kTileRound > cend) return (int)kEach;
        base = (uint32_t)c << kTileSrcLoBits;
        const uint32_t lo = base + ((uint32_t)__builtin_amdgcn_readlane((int)w.v[0].x, 0) >> kTileRowBits);
        const uint32_t hi = base + ((uint32_t)__builtin_amdgcn_readlane((int)w.v[kTileUnroll - 1].w, kWave - 1) >> kTileRowBits);
        if (hi - lo >= kTileSpan) return (int)kGather;
        w0 = lo & ~3u;
        const uint32_t v = (w0 >> 2) + lane;
        const uint32_t vhi = hi >> 2;            // nothing past the stretch (hi < N) is read: half of a window as a rule (2 % of a hop)
        if (v <= vhi) y0 = y4[v];
        if (lane < (kTileWin - 256) / 4 && v + kWave <= vhi) y1 = y4[v + kWave];
        return (int)kWindow;
    };
    uint32_t q0 = 0;
    if (nvec > 0) {
        Words cur = load(q0), nxt = load(q0 + kStep);
        uint32_t base = 0, w0 = 0, base_n = 0, w0_n = 0;
        int how = look(q0, cur, base, w0);
        for (; q0 < nvec; q0 += kStep) {
            const Words far = load(q0 + 2 * kStep);
            if (how == kWindow) {
                *reinterpret_cast<f32x4*>(win + 4 * lane) = y0;
                if (lane < (kTileWin - 256) / 4) *reinterpret_cast<f32x4*>(win + 256 + 4 * lane) = y1;
                wave_lds_order();
            }
            int how_n = kEach;
            if (q0 + kStep < nvec) how_n = look(q0 + kStep, nxt, base_n, w0_n);
            float v[kTileUnroll][4];
            if (how == kWindow) {
                const uint32_t off = base - w0;
#pragma unroll
                for (int u = 0; u < kTileUnroll; ++u) {
                    v[u][0] = win[off + (cur.v[u].x >> kTileRowBits)];
                    v[u][1] = win[off + (cur.v[u].y >> kTileRowBits)];
                    v[u][2] = win[off + (cur.v[u].z >> kTileRowBits)];
                    v[u][3] = win[off + (cur.v[u].w >> kTileRowBits)];
                }
                wave_lds_order();
            } else if (how == kGather) {
                const float* __restrict__ yc = y + base;
#pragma unroll
                for (int u = 0; u < kTileUnroll; ++u) {
                    v[u][0] = yc[cur.v[u].x >> kTileRowBits];
                    v[u][1] = yc[cur.v[u].y >> kTileRowBits];
                    v[u][2] = yc[cur.v[u].z >> kTileRowBits];
                    v[u][3] = yc[cur.v[u].w >> kTileRowBits];
                }
            } else {
#pragma unroll
                for (int u = 0; u < kTileUnroll; ++u) {
                    const uint32_t q = q0 + u * kWave + lane, p = p0 + 4 * q;
                    v[u][0] = v[u][1] = v[u][2] = v[u][3] = 0.0f;
                    if (q < nvec) {
                        v[u][0] = y[tile_source(cur.v[u].x, tile_chunk_of(bound, nch, p))];
                        v[u][1] = y[tile_source(cur.v[u].y, tile_chunk_of(bound, nch, p + 1))];
                        v[u][2] = y[tile_source(cur.v[u].z, tile_chunk_of(bound, nch, p + 2))];
                        v[u][3] = y[tile_source(cur.v[u].w, tile_chunk_of(bound, nch, p + 3))];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kTileUnroll; ++u) {
                if (v[u][0] != 0.0f) unsafeAtomicAdd(&acc[cur.v[u].x & kTileRowMask], (double)v[u][0]);
                if (v[u][1] != 0.0f) unsafeAtomicAdd(&acc[cur.v[u].y & kTileRowMask], (double)v[u][1]);
                if (v[u][2] != 0.0f) unsafeAtomicAdd(&acc[cur.v[u].z & kTileRowMask], (double)v[u][2]);
                if (v[u][3] != 0.0f) unsafeAtomicAdd(&acc[cur.v[u].w & kTileRowMask], (double)v[u][3]);
            }
            cur = nxt; nxt = far;
            how = how_n; base = base_n; w0 = w0_n;
        }
    }
    __syncthreads();
    double* __restrict__ out = part + (int64_t)j * part_stride + (rb << rbits);
    for (int i = threadIdx.x; i < R; i += kTileBlock) out[i] = acc[i];
}
// Shares per row block: what makes the fewest rounds of one workgroup per CU, counting 8192 edges' time for
// what a share costs besides its edges (clearing and writing 128 KB of sums).  147 blocks on 256 CUs: 5
// shares, 2.9 rounds of them (6 shares, the former rule's four workgroups per CU: 3.4, most of a
// round idle).
inline int tile_parts(int num_cu, int64_t nrb, int64_t M) {
    int best = 1;
    double best_cost = 0.0;
    for (int p = 1; p <= 16 && nrb > 0; ++p) {
        const double rounds = (double)((nrb * p + num_cu - 1) / num_cu);
        const double cost = rounds * ((double)M / (double)(nrb * p) + 8192.0);
        if (p == 1 || cost < best_cost) { best = p; best_cost = cost; }
    }
    return best;
}

// ---- dense hops over the chunked layout -------------------------------------------------------
// When y does not stay in the caches (10^8 vertices: 444 MB), the gathers of the kernel above fetch
// a 128-byte line per edge and the hop runs at a tenth of the edge stream's rate.  The chunked
// layout trades bytes for order.  First pass: a workgroup keeps the y of a chunk of 2^15 sources
// in LDS (128 KB) and writes y[source] for entries of the chunk, in entry order: 2 bytes read and 4
// written per entry, all of it streamed.  The workgroups, one per CU, take equal shares of all entries and go
// from chunk to chunk inside theirs (a workgroup per chunk left CUs idle in the last round: 428 chunks on 256 CUs
// took 629 us for 400M entries, shares 569; 546 now).  Second pass: one workgroup per row
// block keeps the block's fp64 sums in LDS and adds up the block's pieces, one from every chunk
// (4 + 2 bytes read per entry in runs of about a hundred entries, found through two tables that are
// staged in LDS 2048 pieces at a time), then finishes the block's vertices itself.  12 bytes per
// entry instead of 4, but no line is fetched for four of its bytes.
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
constexpr int kXBlock = 1024;
constexpr int64_t kExpandShare = 8192;   // fewest vectors per workgroup of the first pass: what a chunk's y costs to load
constexpr int kXUnroll = 4;              // vectors (four entries) per lane and round of the first pass (2, 4, 8: the same time)

__global__ void __launch_bounds__(kXBlock) vip_expand_kernel(const uint16_t* __restrict__ x_src,
                                                             const int64_t* __restrict__ chunk_first, int nch, int64_t N,
                                                             const float* __restrict__ y, float* __restrict__ vals,
                                                             const uint32_t* __restrict__ how) {
    extern __shared__ float ych[];
    __shared__ int c_first;
    if (*how != kPulled) return;
    constexpr int C = 1 << kXSrcBits;
    const int64_t nvec = chunk_first[nch] >> 2;
    const int64_t beg = nvec * blockIdx.x / gridDim.x, end = nvec * (blockIdx.x + 1) / gridDim.x;
    for (int c = threadIdx.x; c < nch; c += kXBlock)
        if ((chunk_first[c] >> 2) <= beg && beg < (chunk_first[c + 1] >> 2)) c_first = c;
    __syncthreads();
    if (beg >= end) return;
    for (int c = c_first; c < nch && (chunk_first[c] >> 2) < end; ++c) {
        int64_t q0 = chunk_first[c] >> 2, q1 = chunk_first[c + 1] >> 2;
        if (q0 < beg) q0 = beg;
        if (q1 > end) q1 = end;
        if (q0 >= q1) continue;          // no entries
        const int64_t v0 = (int64_t)c << kXSrcBits;
        int any = 0;
        if (v0 + C <= N) {               // y is 16-byte aligned and v0 a multiple of C
            const f32x4* __restrict__ y4 = reinterpret_cast<const f32x4*>(y + v0);
            f32x4 t[C / 4 / kXBlock];
#pragma unroll
            for (int k = 0; k < C / 4 / kXBlock; ++k) t[k] = y4[threadIdx.x + k * kXBlock];
#pragma unroll
            for (int k = 0; k < C / 4 / kXBlock; ++k) {
                reinterpret_cast<f32x4*>(ych)[threadIdx.x + k * kXBlock] = t[k];
                any |= (t[k].x != 0.0f) | (t[k].y != 0.0f) | (t[k].z != 0.0f) | (t[k].w != 0.0f);
            }
        } else {
            for (int i = threadIdx.x; i < C; i += kXBlock) {
                const float t = v0 + i < N ? y[v0 + i] : 0.0f;
                ych[i] = t;
                any |= t != 0.0f;
            }
        }
        if (threadIdx.x == 0) ych[C] = 0.0f;     // what a padding entry (source kXPad = C) looks up
        any = __syncthreads_or(any);
        const u16x4* __restrict__ sv = reinterpret_cast<const u16x4*>(x_src);
        f32x4* __restrict__ out = reinterpret_cast<f32x4*>(vals);
        // The chunk's vectors are cut into tiles of kXTile (32 KB of values); the workgroup's wavefronts
        // take the tiles in turn, so at any moment the workgroup writes a window of sixteen adjacent
        // tiles, each as a stream of 1 KB stores.  (The workgroup walking the chunk as one stream: 4.8 ms
        // per pass on the 10^8-vertex graph; a stream per wavefront, long or in tiles: 4.4 ms, the
        // rate at which this part writes long streams while it reads a third as much beside them.)
        constexpr int64_t kXTile = 2048;
        const int64_t ntile = (q1 - q0 + kXTile - 1) / kXTile;
        for (int64_t tile = threadIdx.x >> 6; tile < ntile; tile += kXBlock / kWave) {
            const int64_t wq0 = q0 + tile * kXTile;
            const int64_t wq1 = wq0 + kXTile < q1 ? wq0 + kXTile : q1;
            if (!any) {                  // nothing of this chunk is in the frontier: zeros, without reading the entries
                const f32x4 z = {0.f, 0.f, 0.f, 0.f};
                for (int64_t q = wq0 + (threadIdx.x & (kWave - 1)); q < wq1; q += kWave) __builtin_nontemporal_store(z, out + q);
                continue;
            }
            // The next round's entries are in flight while this round's values are looked up and stored.  They are asked for
            // before the stores, which a later load would wait for, and unconditionally (past the end the tile's last
            // vector once more): after a conditional load the compiler waits for all that is in flight.  400M entries: 546 us
            // instead of 572.
            constexpr int64_t kRound = (int64_t)kWave * kXUnroll;
            struct Sources { u16x4 v[kXUnroll]; };
            auto load = [&](int64_t q) {
                Sources s;
#pragma unroll
                for (int u = 0; u < kXUnroll; ++u) s.v[u] = __builtin_nontemporal_load(sv + (q + u * kWave < wq1 ? q + u * kWave : wq1 - 1));
                return s;
            };
            auto store = [&](const u16x4& s, int64_t q) {
                f32x4 w;
                w.x = ych[s.x];
                w.y = ych[s.y];
                w.z = ych[s.z];
                w.w = ych[s.w];
                __builtin_nontemporal_store(w, out + q);
            };
            int64_t q = wq0 + (threadIdx.x & (kWave - 1));
            Sources s = load(q);
            for (int64_t r = wq0; r + kRound <= wq1; r += kRound, q += kRound) {
                const Sources n = load(q + kRound);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < kXUnroll; ++u) store(s.v[u], q + u * kWave);
                s = n;
            }
#pragma unroll
            for (int u = 0; u < kXUnroll; ++u)
                if (q + u * kWave < wq1) store(s.v[u], q + u * kWave);
        }
        __syncthreads();                 // the next chunk overwrites ych
    }
}

// Second pass.  A row block's vectors form one sequence (vector q of the block: the pieces of chunks
// 0, 1, ... end to end); the j-th of `parts` equal shares of it is added up by this workgroup, a
// group of kXGroup pieces at a time: prefix[k] = first vector of piece k in that sequence, start[k]
// = where the piece lies in the arrays.  Ends with a barrier.
struct ReduceArgs {
    const float* vals;
    const uint16_t* x_row;
    const uint32_t *x_start, *x_prefix;
    int      nch;
};
__device__ __forceinline__ void reduce_share(const ReduceArgs& x, int64_t rb, int j, int parts, double* acc) {
    const uint16_t* __restrict__ x_row = x.x_row;
    const float* __restrict__ vals = x.vals;
    const uint32_t *__restrict__ x_start = x.x_start, *__restrict__ x_prefix = x.x_prefix;
    const int nch = x.nch;
    constexpr int R = 1 << kTileRowBits;
    uint32_t* prefix = reinterpret_cast<uint32_t*>(acc + R);     // [kXGroup + 1]
    uint32_t* start = prefix + kXGroup + 1;                      // [kXGroup]
    for (int i = threadIdx.x; i < R; i += kXBlock) acc[i] = 0.0;
    const uint32_t* __restrict__ pre_b = x_prefix + rb * (nch + 1);
    const uint32_t* __restrict__ sta_b = x_start + rb * nch;
    const uint32_t nvec = pre_b[nch];
    const uint32_t beg = (uint32_t)((uint64_t)nvec * j / parts), end = (uint32_t)((uint64_t)nvec * (j + 1) / parts);
    const f32x4* __restrict__ vv = reinterpret_cast<const f32x4*>(vals);
    const u16x4* __restrict__ rv = reinterpret_cast<const u16x4*>(x_row);
    for (int g0 = 0; g0 < nch; g0 += kXGroup) {
        const int gn = nch - g0 < kXGroup ? nch - g0 : kXGroup;
        __syncthreads();                 // the tables of the group before are no longer read; acc is cleared
        for (int k = threadIdx.x; k <= gn; k += kXBlock) prefix[k] = pre_b[g0 + k];
        for (int k = threadIdx.x; k < gn; k += kXBlock) start[k] = sta_b[g0 + k];
        __syncthreads();
        const uint32_t lo = prefix[0] > beg ? prefix[0] : beg, hi = prefix[gn] < end ? prefix[gn] : end;
        if (lo >= hi) continue;          // uniform over the workgroup
        // Every wavefront takes a contiguous run of the group's vectors and walks it 64 vectors at a
        // time, so a lane's piece is found by bisection once and then moves on by a piece or two per
        // round (pieces hold some tens of vectors).  (With the workgroup striding over the group
        // together, a lane skipped some sixty pieces between two of its vectors and spent its time
        // stepping through the table: 6.6 ms per hop of the 10^8-vertex graph instead of 3.)
        const uint32_t per_wave = ((hi - lo + (kXBlock / kWave) - 1) / (kXBlock / kWave) + kWave - 1) / kWave * kWave;
        const uint32_t wlo = lo + (threadIdx.x >> 6) * per_wave;
        const uint32_t whi = wlo + per_wave < hi ? wlo + per_wave : hi;     // wlo may lie beyond hi: then nothing to do
        uint32_t q = wlo + (threadIdx.x & (kWave - 1));
        int k = 0;
        {
            int l = 0, h = gn - 1;       // last piece with prefix[k] <= q (used only where q < whi <= prefix[gn])
            while (l < h) {
                const int mid = (l + h + 1) >> 1;
                if (prefix[mid] <= q) l = mid; else h = mid - 1;
            }
            k = l;
        }
        uint32_t kend = prefix[k + 1];
        constexpr int U = 4;             // vectors in flight per lane
        f32x4 v[U];
        u16x4 r[U];
        bool ok[U];
        auto fetch = [&](int u, uint32_t qq) {
            ok[u] = qq < whi && wlo < hi;
            if (ok[u]) {
                while (qq >= kend) { ++k; kend = prefix[k + 1]; }
                const uint32_t at = start[k] + (qq - prefix[k]);
                v[u] = __builtin_nontemporal_load(vv + at);
                r[u] = __builtin_nontemporal_load(rv + at);
            }
        };
        auto add = [&](const f32x4& w, const u16x4& rr) {
            if (w.x != 0.0f) unsafeAtomicAdd(&acc[rr.x], (double)w.x);
            if (w.y != 0.0f) unsafeAtomicAdd(&acc[rr.y], (double)w.y);
            if (w.z != 0.0f) unsafeAtomicAdd(&acc[rr.z], (double)w.z);
            if (w.w != 0.0f) unsafeAtomicAdd(&acc[rr.w], (double)w.w);
        };
#pragma unroll
        for (int u = 0; u < U; ++u) fetch(u, q + u * kWave);
        while (ok[0]) {
            f32x4 cv[U];
            u16x4 cr[U];
            bool cok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) { cv[u] = v[u]; cr[u] = r[u]; cok[u] = ok[u]; }
            q += U * kWave;
            // the next round's loads are in flight while this round's sums are formed
#pragma unroll
            for (int u = 0; u < U; ++u) fetch(u, q + u * kWave);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (cok[u]) add(cv[u], cr[u]);
        }
    }
    __syncthreads();
}
// With one share per block the workgroup finishes the block's vertices itself (p^[h], running total, next hop's y); otherwise
// it leaves its sums in part[j].  vip_finish_kernel follows either way.
__global__ void __launch_bounds__(kXBlock) vip_reduce_kernel(ReduceArgs x, int parts, int64_t N, double* __restrict__ part,
                                                             int64_t part_stride, VipHop a, const uint32_t* __restrict__ how) {
    extern __shared__ double acc[];
    if (*how != kPulled) return;
    constexpr int R = 1 << kTileRowBits;
    const int64_t nrb = gridDim.x / parts, rb = blockIdx.x % nrb, u0 = rb << kTileRowBits;
    const int j = (int)(blockIdx.x / nrb);
    reduce_share(x, rb, j, parts, acc);
    if (parts == 1) {
        unsigned long long edges = 0;            // not asked for: the hop after a pulled one is pulled
        vip_finish_block<R>(a, u0, N, acc, edges);
    } else {
        double* __restrict__ out = part + (int64_t)j * part_stride + u0;
        for (int i = threadIdx.x; i < R; i += kXBlock) out[i] = acc[i];
    }
}

// y_1(v) for the training vertices (p^[0] = min(1, B/|T|), Sec. 3.1); optionally hop 0 into the
// total; lists and counts hop 1's frontier on the way.  A vertex that T names twice is counted twice, and listed twice unless
// its row is long, which every workgroup of the walk reads the weight of: a compare-and-swap for every vertex cost calls
// with large sets, whose hops are all pulled, 95 us of 870 (8M vertices, all in T).
__global__ void __launch_bounds__(kBlock) vip_init_kernel(const int32_t* __restrict__ T, int64_t nT, int64_t N, double p0,
                                                          double f1, const int64_t* __restrict__ rowptr,
                                                          float* __restrict__ y, double* __restrict__ tot, int include_hop0,
                                                          int* __restrict__ bad, HopPlan plan) {
    __shared__ uint32_t listed[2];
    if (threadIdx.x < 2) listed[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    unsigned long long edges = 0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < nT; i += stride) {
        const int64_t v = T[i];
        if (v < 0 || v >= N) { *bad = 1; continue; }
        const int64_t d = rowptr[v + 1] - rowptr[v];
        if (d > 0) {
            double t = f1 / (double)d;
            if (t > 1.0) t = 1.0;
            const float yv = (float)log1p(-(t * p0));
            if (yv != 0.0f) {
                edges += (unsigned long long)d;
                const bool once = plan.l.seg_count && d > kLongRow;
                if (!once) y[v] = yv;
                if (plan.l.seg_count && (!once || atomicCAS(reinterpret_cast<uint32_t*>(&y[v]), 0u, __float_as_uint(yv)) == 0u))
                    list_vertex(plan.l, listed, v, d);
            }
        }
        if (include_hop0) tot[v] = log1p(-p0);
    }
    plan_hop<kBlock>(plan, edges);               // its barrier: everything is listed
    if (plan.l.seg_count && threadIdx.x < 2) plan.l.seg_count[2 * blockIdx.x + threadIdx.x] = listed[threadIdx.x];
}

// ---- Proposition 1 with arbitrary initial and transition probabilities (Sec. 3.1) -------------
// Push form over the CSR, whose edge order the transition probabilities share: every vertex with
// p^[h-1](v) > 0 adds log1p(-t_h(e) p^[h-1](v)) to the fp64 sum of every member of its row.

__device__ __forceinline__ float unit_or_flag(float x, int* bad) {
    if (x >= 0.0f && x <= 1.0f) return x;
    *bad = 1;                                     // also for NaN
    return 0.0f;
}

// How a hop of the general propagation fills its bins: from a list of its frontier, or (kWhole) from the whole CSR, tile
// by tile, where the frontier's rows hold at least half of the edges.  The kernel that writes a hop's
// probabilities counts their vertices' out-edges and decides; on large graphs it counts a part of them (either form is correct
// for any frontier).  Where the two cross depends on the graph, and one half lies between; a call of one hop, us:
//                                          by tiles   listed, with 40, 45, 50, 55, 60 and 100 % of the edges     equal at
//   2.4M vertices, 121M edges, power law     601      497  520  561  600  644  956                                 55 %
//   5M, 59M, power law                       417      381  406  432  458  484  684                                 47 %
//   4.2M, 65M, RMAT                      395 to 436   372  406  441  446  477  699                                 43 %
//   200k, 5.8M, power law                     65       88   91   93   95   99  120                           below 40 %
constexpr uint32_t kListed = 1, kWhole = 2;
struct FillRule {
    const int64_t* rowptr;               // null: always from the list (no tiles to walk)
    int64_t M;
    unsigned long long* slots;
    uint32_t* how;                       // the next hop's
    int sample;                          // looks at the vertices of one in so many rounds of a wavefront: a power of two
    // By whole workgroups of kBlock threads, whose threads have written the next hop's p[v], p[v + stride], ...; in a loop of its
    // own, after the one that writes them.  (Every vertex's degree, read in that loop: a call of three sparse hops on 8M vertices
    // 389 us, where it takes 350; only the frontier's, 381: a load under a condition keeps the loop's others from overlapping.)
    __device__ __forceinline__ void decide(const float* p, int64_t N) const {
        if (!rowptr) return;
        const int64_t stride = (int64_t)gridDim.x * kBlock, tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
        unsigned long long edges = 0;
        for (int64_t v = tid + ((tid >> 6) & (sample - 1)) * stride; v < N; v += sample * stride) {
            const unsigned long long deg = (unsigned long long)(rowptr[v + 1] - rowptr[v]);
            edges += p[v] > 0.0f ? deg : 0ull;
        }
        const unsigned long long mine = workgroup_sum<kBlock>(edges);
        unsigned long long all;
        if (threadIdx.x == 0 && grid_total(slots, mine, all)) *how = 2 * all * sample >= (unsigned long long)M ? kWhole : kListed;
    }
};

// What a hop's kernels count with: the frontier list's cursor, and the bins' (none without bins).
struct HopCounters {
    unsigned long long* listed;          // the list's cursor
    uint32_t* bins;
    int64_t   nbins;
    __device__ __forceinline__ void clear(int64_t tid, int64_t stride) const {
        for (int64_t i = tid; i < nbins; i += stride) bins[i] = 0u;
        if (tid == 0) *listed = 0ull;
    }
};

__global__ void __launch_bounds__(kBlock) vipg_init_kernel(const float* __restrict__ p0, int64_t N,
                                                           float* __restrict__ pcur, double* __restrict__ tot,
                                                           int include_hop0, int* __restrict__ bad, FillRule rule, HopCounters c) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    c.clear((int64_t)blockIdx.x * kBlock + threadIdx.x, stride);
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < N; v += stride) {
        const float p = unit_or_flag(p0[v], bad);
        pcur[v] = p;
        if (include_hop0) tot[v] = log1p(-(double)p);
    }
    rule.decide(pcur, N);
}

__global__ void __launch_bounds__(kBlock) vipg_push_kernel(const int32_t* __restrict__ list,
                                                           const unsigned long long* __restrict__ nf_ptr,
                                                           const float* __restrict__ pcur,
                                                           const int64_t* __restrict__ rowptr,
                                                           const int32_t* __restrict__ col,
                                                           const float* __restrict__ t, double* __restrict__ acc,
                                                           int* __restrict__ bad) {
    const int lane = lane_id();
    const int64_t nf = (int64_t)*nf_ptr;
    const int64_t wave = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * kBlock) >> 6;
    for (int64_t i = wave; i < nf; i += nwaves) {
        int64_t b;
        uint32_t deg;
        const int64_t v = frontier_entry(list, i, rowptr, b, deg);
        const double pv = (double)pcur[v];
        const int64_t e = b + deg;
        for (int64_t k = b + lane; k < e; k += kWave) {
            const double x = (double)unit_or_flag(t[k], bad) * pv;
            if (x > 0.0) unsafeAtomicAdd(&acc[col[k]], log1p(-x));
        }
    }
}

// Push without global atomics, for graphs that carry the row-block structure: the fp64 global
// atomic adds of vipg_push_kernel run at about 21 G/s whatever the walk, so a dense hop of 121M
// edges takes 5.7 ms.  Here every frontier edge v -> u becomes an entry (fp32 weight, row of u
// inside its block) in the bin of u's row block, and a second kernel adds a bin's entries into the
// block's fp64 sums in LDS, as the pull over row blocks does.  A bin has room for every edge that
// ends in its block (its base and size are the block's range in the transposed structure), so no
// counting pass over the hop is needed.  A workgroup takes a portion of the frontier and lays the
// rows of its vertices end to end (prefix sums of their lengths in LDS; a wavefront takes runs of
// 64 consecutive edges of that sequence whatever the row lengths, so its loads are contiguous).
// It walks them in rounds of 8192 edges: an LDS atomic per edge counts the round's entries per bin and gives
// the edge its place among them, one global atomic per bin reserves their range, and the entries, held by their
// threads meanwhile (in registers, of which eleven spill to memory: two workgroups per CU leave a lane 64), are stored.  2.4M vertices, a hop of a quarter of 121M edges: 274 -> 230 us since all loads of a round
// are under way together (a probability that was looked at where it was loaded, for the flag, had the next edge's wait for it).
// Before that 859 us per dense hop (900 with 256 threads
// that counted a portion in one walk over col[] and stored its entries in a second).  Nothing is busy for half of the time (vector units 35 %, LDS 44 %, a third of
// that bank conflicts; 2.3 GB of traffic, which a copy moves in 360 us): wavefronts wait three quarters of their clocks, for
// their loads, for the round's reservations (15k atomics on each bin's counter) and at the barriers around those, and the
// two workgroups of a CU do not fill each other's waits.  (Rounds of 2048 edges:
// 0.9 ms of reserving alone; 4096 and 6144: 884, 852; more registers for half the wavefronts, 1096.  Sorting 2048
// entries at a time by bin in LDS, so that neighbouring threads store neighbouring entries, was
// slower: 1.2 ms; a thread taking 8 consecutive edges instead of a wavefront taking 64: 1.25 ms.)  Hops whose
// frontier holds half of the edges and more take vipg_prepare_kernel instead.
constexpr int kBinBlock = 256;           // threads per workgroup of the walks below, and most frontier vertices per portion
constexpr int kFillBlock = 1024;         // the same of the general propagation's
constexpr int kFillPer = 8;                // and its edges per thread and round
constexpr int kBinPer = 8;               // edges per thread and round
constexpr int64_t kBinMaxBlocks = 16384; // row blocks whose two counters each fit the LDS of a workgroup

// Frontier entries per portion: every workgroup gets as many portions as every other, and small
// frontiers are cut into small portions so that they still spread over the chip.
template <int kThreads>
__device__ __forceinline__ int64_t bin_portion_size(int64_t nf) {
    const int64_t rounds = (nf + (int64_t)gridDim.x * kThreads - 1) / ((int64_t)gridDim.x * kThreads);
    const int64_t portions = rounds * gridDim.x;
    const int64_t per = portions > 0 ? (nf + portions - 1) / portions : kWave;
    return per < kWave ? kWave : per;
}

// Which list entries make up a portion.  A small frontier (at most two portions per workgroup) is
// dealt out entry by entry, so that the pieces of a long row, adjacent in the list, land in
// different portions; a large one is cut into runs of consecutive entries, whose rows lie
// side by side in col[] (dealt out entry by entry, the dense hop of the general propagation took
// 1.00 ms instead of 0.88).
template <int kThreads>
struct PortionMap {
    int64_t nf, per, nportions;
    bool dealt;
    __device__ __forceinline__ explicit PortionMap(int64_t nf_) : nf(nf_) {
        per = bin_portion_size<kThreads>(nf);
        nportions = (nf + per - 1) / per;
        dealt = nportions <= 2 * (int64_t)gridDim.x;
    }
    __device__ __forceinline__ int count(int64_t portion) const {
        if (dealt) return (int)((nf - portion + nportions - 1) / nportions);
        const int64_t rest = nf - portion * per;
        return (int)(rest < per ? rest : per);
    }
    __device__ __forceinline__ int64_t entry(int64_t portion, int t) const {
        return dealt ? portion + (int64_t)t * nportions : portion * per + t;
    }
};

template <int kThreads>
struct BinPortion {
    uint32_t prefix[kThreads + 1];       // edges of the portion before vertex i
    int64_t  row[kThreads];              // where vertex i's row starts in col[] and t[]
    float    p[kThreads];                // p^[h-1] of vertex i
    uint32_t wave_sum[kThreads / kWave];
};

// The vertex of the portion whose row holds edge x of the sequence (x < prefix[nv]): the last i
// with prefix[i] <= x.
template <int kThreads>
__device__ __forceinline__ int bin_vertex_of(const BinPortion<kThreads>& po, int nv, uint32_t x) {
    int lo = 0, hi = nv;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (po.prefix[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// Lays the rows of the portion's nv vertices end to end; row_of(t, start, length) = the t-th one's weight.  Returns the number of
// edges.  Ends with a barrier; the caller puts one between the last use of a portion and the next call.
template <int kThreads, class RowOf>
__device__ __forceinline__ uint32_t bin_load_portion(BinPortion<kThreads>& po, int nv, RowOf row_of) {
    uint32_t deg = 0;
    if ((int)threadIdx.x < nv) {
        int64_t b;
        po.p[threadIdx.x] = row_of((int)threadIdx.x, b, deg);
        po.row[threadIdx.x] = b;
    }
    uint32_t total;
    const uint32_t ex = bin_block_scan<kThreads>(deg, po.wave_sum, total);
    if ((int)threadIdx.x < nv) po.prefix[threadIdx.x] = ex;
    if (threadIdx.x == 0) po.prefix[nv] = total;
    __syncthreads();
    return total;
}

// A thread's walk over ascending edges of the portion's sequence: where edge x sits in col[] and
// t[], and the probability of its source.  Rows are entered by comparison with the row's end, so an
// edge inside the row of the edge before costs an add.
template <int kThreads>
struct BinCursor {
    using Portion = BinPortion<kThreads>;
    int      i;          // vertex of the portion
    uint32_t row_end;    // first x beyond its row
    int64_t  shift;      // position in col[] minus x, inside this row
    float    p;
    __device__ __forceinline__ void start(const Portion& po, int nv, uint32_t x) {
        i = bin_vertex_of(po, nv, x);
        enter(po);
    }
    __device__ __forceinline__ void enter(const Portion& po) {
        row_end = po.prefix[i + 1];
        shift = po.row[i] - (int64_t)po.prefix[i];
        p = po.p[i];
    }
    __device__ __forceinline__ int64_t at(const Portion& po, uint32_t x) {     // x < prefix[nv], not below the x before
        if (x >= row_end) {
            do { ++i; } while (x >= po.prefix[i + 1]);
            enter(po);
        }
        return shift + (int64_t)x;
    }
};

// Edge q of a thread in the round that starts at edge c0: a wavefront takes kPer runs of 64
// consecutive edges, so that its loads from col[] and t[] are contiguous.
template <int kPer = kBinPer>
__device__ __forceinline__ uint32_t bin_edge(uint32_t c0, int q) {
    return c0 + (threadIdx.x >> 6) * (kWave * kPer) + (uint32_t)q * kWave + (threadIdx.x & (kWave - 1));
}

// Calls f(u, weight) for the portion's edges x, x + 64, ... (`runs` of them, at most kBinPer, those below `total`): all of a
// thread's loads in flight, a wavefront's contiguous.
template <int kThreads, class F>
__device__ __forceinline__ void push_run(const BinPortion<kThreads>& po, int nv, uint32_t total, uint32_t x, int runs, const int32_t* __restrict__ col, F f) {
    if (x >= total) return;
    BinCursor<kThreads> cu;
    cu.start(po, nv, x);
    int32_t u[kBinPer];
    float w[kBinPer];
#pragma unroll
    for (int q = 0; q < kBinPer; ++q) {
        u[q] = -1;
        if (q < runs && x + q * kWave < total) {
            u[q] = col[cu.at(po, x + q * kWave)];
            w[q] = cu.p;
        }
    }
#pragma unroll
    for (int q = 0; q < kBinPer; ++q)
        if (u[q] >= 0) f((uint32_t)u[q], w[q]);
}

// Calls f(u, weight) for every edge of this workgroup's portions of a frontier of nf entries.
template <int kThreads, class RowOf, class F>
__device__ __forceinline__ void push_portions(BinPortion<kThreads>& po, int64_t nf,
                                              const int32_t* __restrict__ col, RowOf row_of, F f) {
    const PortionMap<kThreads> pm(nf);
    for (int64_t portion = blockIdx.x; portion < pm.nportions; portion += gridDim.x) {
        const int nv = pm.count(portion);
        const uint32_t total = bin_load_portion(po, nv, [&](int i, int64_t& b, uint32_t& deg) { return row_of(pm.entry(portion, i), b, deg); });
        for (uint32_t c0 = 0; c0 < total; c0 += kThreads * kBinPer) {
            // of few edges every wavefront gets some (a hop from 200k rows of one edge: 49 us; 83 with 512 edges to a wavefront)
            const uint32_t runs = total - c0 < kThreads * kBinPer ? (total - c0 + kThreads - 1) / kThreads : kBinPer;
            push_run(po, nv, total, c0 + ((threadIdx.x >> 6) * runs << 6) + (threadIdx.x & (kWave - 1)), (int)runs, col, f);
        }
        __syncthreads();
    }
}
template <class F>
__device__ __forceinline__ void push_walk(BinPortion<kBinBlock>& po, int64_t nf, const int32_t* __restrict__ list,
                                          const float* __restrict__ y, const int64_t* __restrict__ rowptr,
                                          const int32_t* __restrict__ col, F f) {
    push_portions(po, nf, col, [&](int64_t i, int64_t& b, uint32_t& deg) { return y[frontier_entry(list, i, rowptr, b, deg)]; }, f);
}

// Adds entries [beg, end) into a row block's sums, by a workgroup of kTileBlock threads.  A thread asks for its next vectors
// before it adds those it has: listed hops with all edges, 121M entries 196 us and 65M (RMAT) 159, where eight 8-byte loads
// at a time with none ahead take 213 and 166 on the same box (one at a time, on another: 325).
__device__ __forceinline__ void bin_add_entries(double* acc, const uint2* __restrict__ bins, int64_t beg, int64_t end) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int U = 4;                       // vectors of two entries per thread and round
    auto add = [&](uint32_t w, uint32_t row) { if (w != 0u) unsafeAtomicAdd(&acc[row], (double)__uint_as_float(w)); };
    if (threadIdx.x < 2) {                     // entries that share their vector with a neighbour's
        const int64_t e = threadIdx.x == 0 ? beg : end - 1;
        if (beg < end && ((e & 1) == 1) == (threadIdx.x == 0)) add(bins[e].x, bins[e].y);
    }
    const u32x4* __restrict__ pairs = reinterpret_cast<const u32x4*>(bins) + (beg + 1) / 2;
    const int n = (int)(end / 2 - (beg + 1) / 2);        // below 2^31: M is below 2^32
    if (n <= 0) return;
    u32x4 x[U], next[U];
    auto load = [&](u32x4 (&v)[U], int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kTileBlock;
            v[u] = __builtin_nontemporal_load(pairs + (i < n ? i : n - 1));
        }
    };
    load(x, (int)threadIdx.x);
    for (int64_t i0 = threadIdx.x; i0 < n; i0 += U * kTileBlock) {
        load(next, (int)(i0 + U * kTileBlock < n ? i0 + U * kTileBlock : n - 1));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kTileBlock < n) { add(x[u].x, x[u].y); add(x[u].z, x[u].w); }
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = next[u];
    }
}

// The same with the entries' weights and rows in arrays of their own, as a fill by tiles leaves them: 121M entries 172 us.
struct SplitBins {
    float*    w;
    uint16_t* row;
    __host__ __device__ SplitBins(void* mem, int64_t M) : w(reinterpret_cast<float*>(mem)), row(reinterpret_cast<uint16_t*>(w + ((M + 3) & ~3ll))) {}
};
__device__ __forceinline__ void bin_add_split(double* acc, const SplitBins& bins, int64_t beg, int64_t end) {
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    constexpr int U = 4;                       // vectors of four entries per thread and round
    auto add = [&](float w, uint32_t row) { if (w != 0.0f) unsafeAtomicAdd(&acc[row], (double)w); };
    const int64_t v0 = (beg + 3) / 4, v1 = end / 4;
    // the entries before the first whole vector and behind the last (all, if there is no whole one)
    const int64_t head = v0 * 4 < end ? v0 * 4 : end, tail = v1 > v0 ? v1 * 4 : head;
    if (beg + threadIdx.x < head) add(bins.w[beg + threadIdx.x], bins.row[beg + threadIdx.x]);
    if (tail + threadIdx.x < end) add(bins.w[tail + threadIdx.x], bins.row[tail + threadIdx.x]);
    if (v1 <= v0) return;
    const f32x4* __restrict__ w4 = reinterpret_cast<const f32x4*>(bins.w) + v0;
    const u16x4* __restrict__ r4 = reinterpret_cast<const u16x4*>(bins.row) + v0;
    const int n = (int)(v1 - v0);              // below 2^30: M is below 2^32
    f32x4 w[U], wn[U];
    u16x4 r[U], rn[U];
    auto load = [&](f32x4 (&a)[U], u16x4 (&b)[U], int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * kTileBlock < n ? i0 + u * kTileBlock : n - 1;
            a[u] = __builtin_nontemporal_load(w4 + i);
            b[u] = __builtin_nontemporal_load(r4 + i);
        }
    };
    load(w, r, (int)threadIdx.x);
    for (int i0 = (int)threadIdx.x; i0 < n; i0 += U * kTileBlock) {
        load(wn, rn, i0 + U * kTileBlock);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kTileBlock < n)
#pragma unroll
                for (int c = 0; c < 4; ++c) add(w[u][c], r[u][c]);
#pragma unroll
        for (int u = 0; u < U; ++u) { w[u] = wn[u]; r[u] = rn[u]; }
    }
}

// Push form of eq. (2) for the uniform weights: every frontier vertex adds y(v) into the
// accumulator of every member of adj(v) (fp64 global atomics).  Portions of frontier vertices walked as one
// edge sequence, as above: with one wavefront per vertex the longest row set the
// kernel's duration (138 us for the 1.2M out-edges of 24k training vertices, degrees up to 20k).  The frontier lies in
// segments; where each starts in the whole is summed up by every workgroup for itself.  A portion of a workgroup's own has at
// least 64 rows; one CU adds 0.5 G/s and forty reach the 21 G/s of all, so rows that are too long for that are walked by all
// workgroups: each lays (up to 1024 of) them end to end for itself and the wavefronts of the launch take 512 edges in turn.
struct PushLds {
    BinPortion<kTileBlock> po;
    uint32_t seg_first[kSegments];
};
__device__ __forceinline__ void push_frontier(PushLds& lds, const HopList& l, int h, float* __restrict__ y,
                                              const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                              double* __restrict__ acc) {
    static_assert(kSegments % kTileBlock == 0 && kWave * kBinPer == 512, "a thread's segments; a wavefront's edges");
    auto add = [&](uint32_t u, float w) { unsafeAtomicAdd(&acc[u], (double)w); };        // hardware fp64 add
    constexpr int kPer = kSegments / kTileBlock;
    uint32_t rows[kPer], longs[kPer], any = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = (int)threadIdx.x * kPer + k;
        rows[k] = i < l.nseg ? l.seg_count[2 * i] : 0u;
        longs[k] = i < l.nseg ? l.seg_count[2 * i + 1] : 0u;
        any |= longs[k];
    }
    auto lay_out = [&](const uint32_t (&c)[kPer]) {      // the segments' parts end to end; returns the number of entries
        uint32_t mine = 0, all;
#pragma unroll
        for (int k = 0; k < kPer; ++k) mine += c[k];
        uint32_t run = bin_block_scan<kTileBlock>(mine, lds.po.wave_sum, all);
#pragma unroll
        for (int k = 0; k < kPer; ++k) { lds.seg_first[threadIdx.x * kPer + k] = run; run += c[k]; }
        __syncthreads();
        return all;
    };
    auto row_of = [&](bool is_long, uint32_t i, int64_t& b, uint32_t& deg) {
        int s = 0;                               // the last segment that starts at or before entry i (empty ones start where the next does)
#pragma unroll
        for (int step = kSegments / 2; step > 0; step >>= 1)
            if (lds.seg_first[s + step] <= i) s += step;
        const int64_t at = i - lds.seg_first[s];
        const int32_t v = l.list[(int64_t)s * l.seg_cap + (is_long ? l.seg_cap - 1 - at : at)];
        b = rowptr[v];
        deg = (uint32_t)(rowptr[v + 1] - b);
        // a vertex that the training set names twice is listed twice (see vip_init_kernel): one of the entries takes the weight,
        // and nothing reads y after a push
        return h == 1 && !is_long ? __uint_as_float(atomicExch(reinterpret_cast<uint32_t*>(y) + v, 0u)) : y[v];
    };
    const uint32_t nf = lay_out(rows);
    push_portions(lds.po, (int64_t)nf, col, [&](int64_t i, int64_t& b, uint32_t& deg) { return row_of(false, (uint32_t)i, b, deg); }, add);
    if (!__syncthreads_or((int)any)) return;
    const uint32_t nlong = lay_out(longs);
    for (uint32_t f0 = 0; f0 < nlong; f0 += kTileBlock) {
        const int nv = (int)(nlong - f0 < kTileBlock ? nlong - f0 : kTileBlock);
        // below 2^28 edges: the frontier of a pushed hop has M / kPushShare at most
        const uint32_t total = bin_load_portion(lds.po, nv, [&](int t, int64_t& b, uint32_t& deg) { return row_of(true, f0 + (uint32_t)t, b, deg); });
        // a wavefront of every workgroup before a second one of any
        const uint32_t wave = (threadIdx.x >> 6) * gridDim.x + blockIdx.x;
        for (uint32_t x0 = wave * 512u; x0 < total; x0 += gridDim.x * (kTileBlock / kWave) * 512u)
            push_run(lds.po, nv, total, x0 + (threadIdx.x & (kWave - 1)), kBinPer, col, add);
        __syncthreads();
    }
}

// A hop in the form it takes: one launch, whose workgroups push the frontier or pull row blocks.  (A launch for each form,
// one of which leaves at once, cost a hop 5 us, and listing the frontier in a third the same again.)
__global__ void __launch_bounds__(kTileBlock) vip_hop_kernel(HopList l, int h, const int64_t* __restrict__ rowptr,
                                                             const int32_t* __restrict__ col, const uint32_t* __restrict__ t_edge,
                                                             const int64_t* __restrict__ first, int nch, int64_t nrb, int parts,
                                                             int rbits, uint32_t N, float* __restrict__ y,
                                                             double* __restrict__ acc, int64_t part_stride,
                                                             const uint32_t* __restrict__ how) {
    extern __shared__ double hop_lds[];
    if (*how == kPushed) push_frontier(*reinterpret_cast<PushLds*>(hop_lds), l, h, y, rowptr, col, acc);
    else if (t_edge) pull_tiles(hop_lds, t_edge, first, nch, nrb, parts, rbits, N, y, acc, part_stride);
}

// The same push through bins, for graphs in the chunked layout.  The atomics above run at 21 G/s whatever
// the walk (13.4M out-edges on 14M vertices: 616 us, counted and filled in 217 here, and the accumulators are cleared before and read
// after them); here they are adds in LDS.  Every edge of the frontier becomes an entry (weight, row inside
// its block of 2^kTileRowBits rows), the entries of a block lie side by side, and a workgroup per block
// sums them and finishes the block's vertices.  A frontier that is pushed has at most M / kPushShare
// out-edges, so the entries are packed (counted first, by a walk that reads 4 bytes per edge) and fit the
// memory where a pulled hop keeps its values; reserving every block's in-edges would take 8 M bytes
// beside it.  A fixed number of workgroups takes the portions in a fixed order in both walks, so
// one row of counts per workgroup says where its entries of each block go, without atomics.
constexpr int kPushGroups = 1024;        // workgroups of the two walks (four per CU)
constexpr int kOffBins = 16;             // row blocks per workgroup of vip_bin_offsets_kernel
constexpr int kOffRows = kPushGroups / (1024 / kOffBins);      // counts per thread there

// off[g][r] = edges of workgroup g that end in row block r.
__global__ void __launch_bounds__(kBinBlock) vip_bin_count_kernel(const int32_t* __restrict__ list,
                                                                  const unsigned long long* __restrict__ nf_ptr,
                                                                  const float* __restrict__ y,
                                                                  const int64_t* __restrict__ rowptr,
                                                                  const int32_t* __restrict__ col, int nrb,
                                                                  uint32_t* __restrict__ off,
                                                                  const uint32_t* __restrict__ how) {
    __shared__ BinPortion<kBinBlock> po;
    extern __shared__ uint32_t bin_lds[];
    if (*how != kPushed) return;
    for (int r = threadIdx.x; r < nrb; r += kBinBlock) bin_lds[r] = 0u;
    __syncthreads();
    push_walk(po, (int64_t)*nf_ptr, list, y, rowptr, col, [&](uint32_t u, float) { atomicAdd(&bin_lds[u >> kTileRowBits], 1u); });
    for (int r = threadIdx.x; r < nrb; r += kBinBlock) off[(int64_t)blockIdx.x * nrb + r] = bin_lds[r];
}

// Turns the counts of each row block into the entries that the workgroups before put there, and leaves the
// block's number of entries in total[].  A thread holds kOffRows counts of one block; a wavefront then
// scans the 64 partial sums of one block.
__global__ void __launch_bounds__(1024) vip_bin_offsets_kernel(uint32_t* __restrict__ off, int nrb,
                                                               uint32_t* __restrict__ total, const uint32_t* __restrict__ how) {
    __shared__ uint32_t sums[kOffBins][kWave + 1];
    static_assert(1024 / kOffBins == kWave && 1024 / kWave == kOffBins, "a wavefront per block, a lane per partial sum");
    if (*how != kPushed) return;
    const int b = threadIdx.x % kOffBins, g = threadIdx.x / kOffBins;
    const int r = blockIdx.x * kOffBins + b;
    uint32_t c[kOffRows], mine = 0;
#pragma unroll
    for (int k = 0; k < kOffRows; ++k) c[k] = r < nrb ? off[(int64_t)(g * kOffRows + k) * nrb + r] : 0u;
#pragma unroll
    for (int k = 0; k < kOffRows; ++k) mine += c[k];
    sums[b][g] = mine;
    __syncthreads();
    {
        const int w = threadIdx.x >> 6, lane = lane_id();
        const uint32_t v = sums[w][lane], inc = (uint32_t)wave_inclusive_scan((int)v);
        sums[w][lane] = inc - v;
        if (lane == kWave - 1 && (int)(blockIdx.x * kOffBins + w) < nrb) total[blockIdx.x * kOffBins + w] = inc;
    }
    __syncthreads();
    if (r >= nrb) return;
    uint32_t run = sums[b][g];
#pragma unroll
    for (int k = 0; k < kOffRows; ++k) {
        off[(int64_t)(g * kOffRows + k) * nrb + r] = run;
        run += c[k];
    }
}

// The entries; base[r] = first entry of row block r (base[nrb]: their number).
__global__ void __launch_bounds__(kBinBlock) vip_bin_fill_kernel(const int32_t* __restrict__ list,
                                                                 const unsigned long long* __restrict__ nf_ptr,
                                                                 const float* __restrict__ y,
                                                                 const int64_t* __restrict__ rowptr,
                                                                 const int32_t* __restrict__ col, int nrb,
                                                                 const uint32_t* __restrict__ off,
                                                                 const uint32_t* __restrict__ total,
                                                                 uint32_t* __restrict__ base, uint2* __restrict__ bins,
                                                                 const uint32_t* __restrict__ how) {
    __shared__ BinPortion<kBinBlock> po;
    extern __shared__ uint32_t bin_lds[];        // where this workgroup's next entry of each row block goes
    if (*how != kPushed) return;
    const int per = (nrb + kBinBlock - 1) / kBinBlock;
    const int r0 = (int)threadIdx.x * per, r1 = r0 + per < nrb ? r0 + per : nrb;
    for (int r = threadIdx.x; r < nrb; r += kBinBlock) bin_lds[r] = total[r];
    __syncthreads();
    uint32_t sum = 0, all;
    for (int r = r0; r < r1; ++r) sum += bin_lds[r];
    uint32_t run = bin_block_scan<kBinBlock>(sum, po.wave_sum, all);
    for (int r = r0; r < r1; ++r) {
        const uint32_t c = bin_lds[r];
        bin_lds[r] = run;
        run += c;
    }
    __syncthreads();
    for (int r = threadIdx.x; r < nrb; r += kBinBlock) {
        const uint32_t b = bin_lds[r];
        if (blockIdx.x == 0) base[r] = b;
        bin_lds[r] = b + off[(int64_t)blockIdx.x * nrb + r];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) base[nrb] = all;
    __syncthreads();
    push_walk(po, (int64_t)*nf_ptr, list, y, rowptr, col, [&](uint32_t u, float w) {
        bins[atomicAdd(&bin_lds[u >> kTileRowBits], 1u)] = make_uint2(__float_as_uint(w), u & kTileRowMask);
    });
}

// Sums a row block's entries in LDS and finishes its vertices.  14M vertices, 115 us with 13.4M entries, 58 with 0.8M, where the
// bytes take 62 and 27 (137 and 88 with the arithmetic of all vertices): four rounds of one workgroup per CU, whose
// phases nothing overlaps.
// The other form of the hop, the second pass of a pull, has the same workgroups: in one launch with it (one that finds nothing
// to do costs 4.6 us).
__global__ void __launch_bounds__(kTileBlock) vip_bin_finish_kernel(VipHop a, const uint2* __restrict__ bins,
                                                                    const uint32_t* __restrict__ base, int64_t N, ReduceArgs x,
                                                                    const uint32_t* __restrict__ how) {
    extern __shared__ double acc[];
    static_assert(kXBlock == kTileBlock, "either form's workgroups");
    constexpr int R = 1 << kTileRowBits;
    const bool pulled = *how == kPulled;
    if (pulled) {
        reduce_share(x, blockIdx.x, 0, 1, acc);
    } else {
        for (int i = threadIdx.x; i < R; i += kTileBlock) acc[i] = 0.0;
        __syncthreads();
        bin_add_entries(acc, bins, base[blockIdx.x], base[blockIdx.x + 1]);
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) hop_done(a, pulled);
    unsigned long long edges = 0;
    const int64_t u0 = (int64_t)blockIdx.x << kTileRowBits;
    if (a.last || pulled) {                      // the hop after a pulled one is pulled whatever its edges
        vip_finish_block<R>(a, u0, N, acc, edges);
        return;
    }
    static_assert(kTileWaves * kWaveRows == R, "a wavefront's vertices");
    const int wave = threadIdx.x >> 6;
    uint16_t* queue = reinterpret_cast<uint16_t*>(acc + R) + wave * kTouchedQueue;
    vip_finish_touched(a, u0 + wave * kWaveRows, N, acc + wave * kWaveRows, queue, edges);
    plan_hop<kTileBlock>(a.next, edges);
}

// The bins of a hop whose frontier holds most of the edges.  A tile of the CSR (kPartTile edges) puts its edges of a row block
// where the set-up's partition put them: tile_off[block * ntiles + tile] says where they start and the next word how
// many they are, so nothing is counted, no range is reserved and no list is read.  A thread reads four consecutive edges
// (128-bit loads); the rows' probabilities lie at the rows' first edges in LDS, where an edge finds its own by
// looking back; an LDS atomic on the block's cursor gives the edge its place among the tile's, which are laid out by
// block in LDS and stored from there as runs.
// Two barriers per tile: (1) the next tile's rows are marked and its cursors set while the tile before is stored, (2) its
// edges are weighed and laid out.  A load that is waited for after stores would wait for those too (they complete in
// order), so a tile's rows and offsets are asked for before the stores of two tiles back, its edges before those of
// the tile before, and nothing in the loop is loaded conditionally (after a conditional load the compiler waits for all).
// The entries' weights and rows go to arrays of their own: 6 bytes per entry where a pair of words takes 8.  (Not so the listed
// fill's, whose stores are scattered: it would store twice as often.)
// 2.4M vertices, 121M edges: 381 us, 1.7 GB (pairs: 424, 2.0 GB), where the listed fill takes 708 (852 before its loads
// were under way together); with seven barriers and waits
// for the stores 535 to 780.  What bounds it now: vector instructions half of the time (64 per 64 edges, the logarithm a third
// of them), LDS a third, and what two workgroups per CU leave uncovered of the two barriers.  (That a tile's rows are waited for
// together with most stores of the tile before costs nothing: 391 with a wait for the loads alone.)  Two registers of a lane's 64 spill to memory.
constexpr int kMaxTileBlocks = 512;      // row blocks of a graph that has tiles
struct PrepareLds {
    uint2    stage[kPartTile];           // the tile's entries by block: weight, destination
    uint32_t mark[2][kPartTile];         // p of the row that starts at an edge of the tile
    uint32_t cnt[kMaxTileBlocks], off[kMaxTileBlocks];           // of the next tile: edges per block and where they go
    uint32_t cursor[2][kMaxTileBlocks];  // the next entry of a block among the tile's, from its first up and from its last down
    uint32_t shift[2][kMaxTileBlocks];   // where a block's entries go, less where they start among the tile's
};

// The launch before the listed fill: lists the frontier or, where the whole CSR is walked, fills the bins itself.
__global__ void __launch_bounds__(kFillBlock, 8) vipg_prepare_kernel(const uint32_t* __restrict__ how, const uint32_t* __restrict__ tile_off,
                                                                     const int32_t* __restrict__ tile_row, int ntiles, int64_t M,
                                                                     const float* __restrict__ pcur,
                                                                     const int64_t* __restrict__ rowptr,
                                                                     const int32_t* __restrict__ col, const float* __restrict__ t,
                                                                     int rbits, int nrb, SplitBins bins,
                                                                     int* __restrict__ bad, int64_t N, int32_t* __restrict__ list,
                                                                     unsigned long long* __restrict__ cursor) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) char prepare_lds[];
    if (*how != kWhole) {
        uint32_t* lds = reinterpret_cast<uint32_t*>(prepare_lds);
        // a sparse frontier among 8M vertices 16 us instead of 20; small graphs and denser frontiers the other way round
        if (N >= (int64_t)1 << 22) list_frontier<kFillBlock, 16>(pcur, rowptr, N, list, cursor, lds);
        else list_frontier<kFillBlock, 8>(pcur, rowptr, N, list, cursor, lds);
        return;
    }
    PrepareLds& l = *reinterpret_cast<PrepareLds*>(prepare_lds);
    static_assert(kPartTile == 4 * kFillBlock, "four edges of a tile per thread");
    constexpr uint32_t kSpan = 4 * kWave;        // edges of a tile per wavefront
    constexpr uint32_t kNone = 0xFFFFFFFFu;      // no bits of a probability
    const int lane = lane_id();
    const uint32_t tid = threadIdx.x, rmask = (1u << rbits) - 1u;
    const int wave = __builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t off0 = ((int)tid < nrb ? tid : 0u) * (uint32_t)ntiles;       // below 2^30
    // a tile's rows and offsets (the first kFillBlock rows, one per thread; threads beyond take the last one once more)
    struct { int32_t v0, v1; uint32_t b, e; float p; uint32_t off, off_n; } r;
    const uint32_t* __restrict__ row32 = reinterpret_cast<const uint32_t*>(rowptr);      // the lower halves: offsets are below 2^32, like M
    auto load_row = [&](uint32_t v) { r.b = row32[2u * v]; r.e = row32[2u * v + 2u]; r.p = pcur[v]; };
    // where a tile's rows begin and end, in even and odd lanes, is asked for a tile before they are: by a vector load, as a scalar
    // one is waited for at the next read of LDS
    int32_t ends;
    auto load_ends = [&](int tile) { ends = tile_row[tile + (lane & 1)]; };
    auto load_rows = [&](int tile) {
        r.v0 = __builtin_amdgcn_readlane(ends, 0); r.v1 = __builtin_amdgcn_readlane(ends, 1);
        load_row((uint32_t)(r.v1 - r.v0 > (int32_t)tid ? r.v0 + (int32_t)tid : r.v1));
        const uint32_t at = off0 + (uint32_t)tile;
        r.off = tile_off[at];
        r.off_n = tile_off[at + 1u];             // behind the last one stands M
    };
    uint32_t u[4];
    float x[4];
    auto load_edges = [&](int tile) {            // of a full tile; col and t are 16-byte aligned
        const u32x4 a = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(col + (int64_t)tile * kPartTile) + tid);
        const f32x4 b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(t + (int64_t)tile * kPartTile) + tid);
        u[0] = a.x; u[1] = a.y; u[2] = a.z; u[3] = a.w;
        x[0] = b.x; x[1] = b.y; x[2] = b.z; x[3] = b.w;
    };
    bool wrong = false;
    auto mark_rows = [&](int tile, uint32_t n, uint32_t* mark) {
        const uint32_t base = (uint32_t)tile * (uint32_t)kPartTile, stop = base + n;       // at most M
        auto one = [&]() {                       // at its first edge, and at the first edge of every wavefront's part that begins inside it
            const uint32_t b = (r.b > base ? (r.b < stop ? r.b : stop) : base) - base, e = (r.e > base ? (r.e < stop ? r.e : stop) : base) - base;
            if (b < e) {
                mark[b] = __float_as_uint(r.p);
                for (uint32_t k = (b + kSpan) & ~(kSpan - 1); k < e; k += kSpan) mark[k] = __float_as_uint(r.p);
            }
        };
        if (r.v1 - r.v0 > kTileManyRows) {       // the same for all threads
#pragma unroll 1
            for (uint32_t e = 4 * tid; e < 4 * tid + 4 && e < n; ++e) mark[e] = __float_as_uint(pcur[row_of_edge(rowptr, r.v0, r.v1, base + e)]);
            return;
        }
        if (r.v1 - r.v0 >= (int32_t)tid) one();
        for (int64_t v = (int64_t)r.v0 + kFillBlock + tid; v <= r.v1; v += kFillBlock) { load_row((uint32_t)v); one(); }
    };
    auto keep_offsets = [&]() {                  // for the wavefronts that set the cursors
        if ((int)tid < nrb) { l.cnt[tid] = r.off_n - r.off; l.off[tid] = r.off; }
    };
    auto set_cursors = [&](uint32_t* shift) {    // 64 blocks to a wavefront, from the third on: the first ones have rows to mark
        const int b0 = (wave - 2) * kWave, b = b0 + lane;
        if (b0 < 0 || b0 >= nrb) return;
        uint32_t before = 0;
        for (int q = lane; q < b0; q += kWave) before += l.cnt[q];
        const uint32_t c = b < nrb ? l.cnt[b] : 0u, inc = (uint32_t)wave_inclusive_scan((int)c);
        const uint32_t start = (uint32_t)wave_sum((int)before) + inc - c;
        if (b < nrb) { l.cursor[0][b] = start; l.cursor[1][b] = start + c; shift[b] = l.off[b] - start; }
    };
    auto clear_marks = [&](uint32_t* mark) {
        const uint32_t none = here(kNone);
        reinterpret_cast<u32x4*>(mark)[here(tid)] = u32x4{none, none, none, none};
    };
    auto weigh = [&](const uint32_t* mark, auto full, uint32_t n) {
        // the last mark at or before an edge: among the lane's own four or in the lanes before
        const u32x4 m4 = reinterpret_cast<const u32x4*>(mark)[tid];
        uint32_t m[4] = {m4.x, m4.y, m4.z, m4.w};
        const uint32_t last = m[3] != kNone ? m[3] : m[2] != kNone ? m[2] : m[1] != kNone ? m[1] : m[0];
        const uint64_t below = __ballot(last != kNone) & ((1ull << lane) - 1ull);
        const uint32_t before = (uint32_t)__shfl((int)last, 63 - __clzll((long long)(below | 1ull)), kWave);
        m[0] = m[0] != kNone ? m[0] : before;
#pragma unroll
        for (int q = 1; q < 4; ++q) m[q] = m[q] != kNone ? m[q] : m[q - 1];
        // Rows are sorted, so edges side by side often end in one block: a run of them in the lane takes one atomic.  Even
        // lanes take a block's places from below, odd ones from above: where a whole wavefront ends in one block (a hub's
        // row), half as many adds meet on one address.
        uint32_t blk[4], len[4], place[4];
        bool run[4] = {};                        // the edge continues the run of the one before
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            blk[q] = u[q] >> rbits;
            if (q > 0) run[q] = blk[q] == blk[q - 1] && (full || 4 * tid + q < n);
        }
        len[3] = 1;
#pragma unroll
        for (int q = 2; q >= 0; --q) len[q] = run[q + 1] ? len[q + 1] + 1u : 1u;
        const bool down = lane & 1;
        uint32_t* cur = l.cursor[lane & 1];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if ((full || 4 * tid + q < n) && !run[q]) place[q] = atomicAdd(&cur[blk[q]], down ? 0u - len[q] : len[q]) - (down ? len[q] : 0u);
#pragma unroll
        for (int q = 1; q < 4; ++q)
            if (run[q]) place[q] = place[q - 1] + 1u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (full || 4 * tid + q < n) {
                const float p = __uint_as_float(m[q]), c = __builtin_amdgcn_fmed3f(x[q], 0.0f, 1.0f);
                wrong |= p > 0.0f && !(c == x[q]);
                l.stage[place[q]] = make_uint2(__float_as_uint(bin_log1p_neg(c == x[q] ? c * p : 0.0f)), u[q]);
            }
    };
    auto store = [&](const uint32_t* shift, auto full, uint32_t n) {
#pragma unroll
        for (int k = 0; k < kPartTile / kFillBlock; ++k) {
            const uint32_t i = here(tid) + k * kFillBlock;
            if (full || i < n) {
                const uint2 e = l.stage[i];
                const uint32_t to = shift[e.y >> rbits] + i;
                bins.w[to] = __uint_as_float(e.x);
                bins.row[to] = (uint16_t)(e.y & rmask);
            }
        }
    };
    // neighbouring tiles store to neighbouring places: an XCD (workgroups go to the eight in turn) takes a run of the full tiles
    const int nfull = (int)(M / kPartTile), per_xcd = (nfull + 7) / 8, step = (int)(gridDim.x >> 3), x0 = (int)(blockIdx.x & 7) * per_xcd;
    const int end = x0 + per_xcd < nfull ? x0 + per_xcd : nfull;
    int tile = x0 + (int)(blockIdx.x >> 3);
    if (tile < end) {
        auto at = [&](int tl) { return tl < end ? tl : end - 1; };
        load_ends(tile);
        load_rows(tile);
        load_ends(at(tile + step));
        load_edges(tile);
        clear_marks(l.mark[0]);
        keep_offsets();
        __syncthreads();
        mark_rows(tile, kPartTile, l.mark[0]);
        set_cursors(l.shift[0]);
        load_rows(at(tile + step));
        load_ends(at(tile + 2 * step));
        __syncthreads();
        for (int k = 0; tile < end; tile += step, k ^= 1) {      // k: which of the two marks and shifts
            clear_marks(l.mark[k ^ 1]);
            keep_offsets();
            weigh(l.mark[k], std::true_type{}, kPartTile);
            load_edges(at(tile + step));
            __syncthreads();
            mark_rows(at(tile + step), kPartTile, l.mark[k ^ 1]);
            set_cursors(l.shift[k ^ 1]);
            load_rows(at(tile + 2 * step));
            load_ends(at(tile + 3 * step));
            store(l.shift[k], std::true_type{}, kPartTile);
            __syncthreads();
        }
    }
    if (nfull < ntiles && blockIdx.x == gridDim.x - 1) {         // the rest
        const uint32_t n = (uint32_t)(M - (int64_t)nfull * kPartTile);
        load_ends(nfull);
        load_rows(nfull);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u[q] = 4 * tid + q < n ? (uint32_t)col[(int64_t)nfull * kPartTile + 4 * tid + q] : 0u;
            x[q] = 4 * tid + q < n ? t[(int64_t)nfull * kPartTile + 4 * tid + q] : 0.0f;
        }
        clear_marks(l.mark[0]);
        keep_offsets();
        __syncthreads();
        mark_rows(nfull, n, l.mark[0]);
        set_cursors(l.shift[0]);
        __syncthreads();
        weigh(l.mark[0], std::false_type{}, n);
        __syncthreads();
        store(l.shift[0], std::false_type{}, n);
    }
    if (wrong) *bad = 1;
}

__global__ void __launch_bounds__(kFillBlock, 8) vipg_bin_fill_kernel(const int32_t* __restrict__ list,
                                                                      const unsigned long long* __restrict__ nf_ptr,
                                                                      const float* __restrict__ pcur,
                                                                      const int64_t* __restrict__ rowptr,
                                                                      const int32_t* __restrict__ col,
                                                                      const float* __restrict__ t, int rbits, int nrb,
                                                                      const int64_t* __restrict__ first, int nch,
                                                                      uint32_t* __restrict__ cursor,
                                                                      uint2* __restrict__ bins, int* __restrict__ bad,
                                                                      const uint32_t* __restrict__ how) {
    __shared__ BinPortion<kFillBlock> po;
    extern __shared__ uint32_t lds_u32[];
    if (how && *how != kListed) return;
    uint32_t* count = lds_u32;           // the round's entries per row block; zero between rounds
    uint32_t* base = lds_u32 + nrb;      // the entry (index into bins[], below 2^32) where they start
    const int64_t nf = (int64_t)*nf_ptr;
    const PortionMap<kFillBlock> pm(nf);
    const uint32_t rmask = (1u << rbits) - 1u;
    bool wrong = false;
    for (int r = threadIdx.x; r < nrb; r += kFillBlock) count[r] = 0u;
    // Portions are handed out through a counter (the slot after the bins' cursors): their sizes
    // differ by the degrees of their vertices, and with fixed shares half of the wavefronts had
    // left before the kernel's end.
    __shared__ uint32_t portion;
    for (;;) {
        if (threadIdx.x == 0) portion = atomicAdd(&cursor[nrb], 1u);
        __syncthreads();
        if ((int64_t)portion >= pm.nportions) break;
        const int nv = pm.count(portion);
        const uint32_t total = bin_load_portion(po, nv, [&](int i, int64_t& b, uint32_t& deg) {
            return pcur[frontier_entry(list, pm.entry(portion, i), rowptr, b, deg)];
        });
        for (uint32_t c0 = 0; c0 < total; c0 += kFillBlock * kFillPer) {
            uint32_t key[kFillPer], rank[kFillPer];
            float x[kFillPer], p[kFillPer];
#pragma unroll
            for (int q = 0; q < kFillPer; ++q) { key[q] = ~0u; x[q] = p[q] = 0.0f; }
            if (bin_edge<kFillPer>(c0, 0) < total) {
                BinCursor<kFillBlock> cu;
                cu.start(po, nv, bin_edge<kFillPer>(c0, 0));
#pragma unroll
                for (int q = 0; q < kFillPer; ++q) {             // beyond the last edge that one again: no load is conditional
                    const uint32_t e = bin_edge<kFillPer>(c0, q);
                    const int64_t k = cu.at(po, e < total ? e : total - 1);
                    key[q] = (uint32_t)col[k];
                    x[q] = t[k];
                    p[q] = cu.p;
                }
            }
            // only here: looked at where it is loaded, a probability was waited for before the next edge's was asked for
#pragma unroll
            for (int q = 0; q < kFillPer; ++q) {
                if (bin_edge<kFillPer>(c0, q) >= total) key[q] = ~0u;
                const float c = __builtin_amdgcn_fmed3f(x[q], 0.0f, 1.0f);
                wrong |= !(c == x[q]);
                x[q] = c == x[q] ? c * p[q] : 0.0f;
            }
#pragma unroll
            for (int q = 0; q < kFillPer; ++q)
                if (key[q] != ~0u) rank[q] = atomicAdd(&count[key[q] >> rbits], 1u);
            __syncthreads();
            for (int r = threadIdx.x; r < nrb; r += kFillBlock) {
                const uint32_t c = count[r];
                if (c != 0u) {
                    base[r] = (uint32_t)first[(int64_t)r * nch] + atomicAdd(&cursor[r], c);
                    count[r] = 0u;
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kFillPer; ++q)
                if (key[q] != ~0u) {
                    bins[base[key[q] >> rbits] + rank[q]] =
                        make_uint2(__float_as_uint(x[q] > 0.0f ? bin_log1p_neg(x[q]) : 0.0f), key[q] & rmask);
                }
        }
        __syncthreads();
    }
    if (wrong) *bad = 1;
}

// Adds the entries of one share of one bin into the block's fp64 sums (LDS) and writes them to
// part[j][row], like pull_tiles but with the weights already in place.
__global__ void __launch_bounds__(kTileBlock) vip_bin_sum_kernel(uint2* __restrict__ bins, int64_t M,
                                                                 const uint32_t* __restrict__ cursor,
                                                                 const int64_t* __restrict__ first, int nch, int parts,
                                                                 int rbits, double* __restrict__ part, int64_t part_stride,
                                                                 const uint32_t* __restrict__ how) {
    extern __shared__ double acc[];
    const int R = 1 << rbits;
    const int64_t rb = blockIdx.x / parts;
    const int j = blockIdx.x % parts;
    for (int i = threadIdx.x; i < R; i += kTileBlock) acc[i] = 0.0;
    __syncthreads();
    const int64_t b0 = first[rb * nch], len = how && *how == kWhole ? first[(rb + 1) * nch] - b0 : (int64_t)cursor[rb];
    const int64_t beg = b0 + len * j / parts, end = b0 + len * (j + 1) / parts;
    if (how && *how == kWhole) bin_add_split(acc, SplitBins(bins, M), beg, end);
    else bin_add_entries(acc, bins, beg, end);
    __syncthreads();
    double* __restrict__ out = part + (int64_t)j * part_stride + (rb << rbits);
    for (int i = threadIdx.x; i < R; i += kTileBlock) out[i] = acc[i];
}

// The state that a call leaves clean for the next, where it may not be.
__global__ void __launch_bounds__(kBlock) vip_state_clear_kernel(unsigned long long* __restrict__ slots, int* __restrict__ bad) {
    for (int i = threadIdx.x; i < kTotalSlots; i += kBlock) slots[i] = 0ull;
    if (threadIdx.x == 0) *bad = 0;
}

// Also empties the counters for the next hop; the last one leaves the flag where the host reads it, and empties it.
__global__ void __launch_bounds__(kBlock) vipg_finish_kernel(const double* __restrict__ acc, double* __restrict__ tot,
                                                             int first, int last, float* __restrict__ p_hop,
                                                             float* __restrict__ p_total, float* __restrict__ pnext,
                                                             int64_t N, int parts, int64_t part_stride, HopCounters c,
                                                             FillRule rule, int* __restrict__ bad, int64_t* __restrict__ bad_mirror) {
    if (last && blockIdx.x == 0 && threadIdx.x == 0) { *bad_mirror = *bad; *bad = 0; }
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    c.clear((int64_t)blockIdx.x * kBlock + threadIdx.x, stride);
    for (int64_t u = (int64_t)blockIdx.x * kBlock + threadIdx.x; u < N; u += stride) {
        double S = acc[u];
        for (int j = 1; j < parts; ++j) S += acc[(int64_t)j * part_stride + u];
        const double ph = -expm1(S);
        if (p_hop) p_hop[u] = (float)ph;
        const double T = first ? S : tot[u] + S;
        if (last) p_total[u] = (float)(-expm1(T));
        else { tot[u] = T; pnext[u] = (float)ph; }
    }
    if (!last) rule.decide(pnext, N);
}

// The context's words for grid_total and the flag for bad input.  They are empty from the context's creation on, whether calls
// run or are only recorded, and each call leaves them so; only after one whose launches were refused they are emptied here.
static int vip_state(spp_ctx* ctx, unsigned long long** slots, int** bad, int* left_clean) {
    *slots = reinterpret_cast<unsigned long long*>(ctx->totals + kTotalsWords);
    *bad = reinterpret_cast<int*>(*slots + kTotalSlots);
    hipStreamCaptureStatus recording = hipStreamCaptureStatusNone;
    if (!ctx->vip_state_clean) {
        SPP_HIP(hipStreamIsCapturing(ctx->stream, &recording));
        vip_state_clear_kernel<<<1, kBlock, 0, ctx->stream>>>(*slots, *bad);
    }
    ctx->vip_state_clean = 0;
    *left_clean = recording == hipStreamCaptureStatusNone;           // what is only recorded empties nothing now
    return SPP_OK;
}

}  // namespace spp

extern "C" int spp_vip_propagate_general(spp_ctx* ctx, const spp_graph* g, const float* d_p0,
                                         const float* const* d_t, int32_t L, float* d_p_total, float* d_p_hop,
                                         uint32_t flags) {
    using namespace spp;
    SPP_CHECK(ctx && g && d_p0 && d_t && d_p_total, SPP_E_ARG, "spp_vip_propagate_general: null argument");
    SPP_CHECK(L >= 1 && L <= SPP_MAX_L, SPP_E_ARG, "spp_vip_propagate_general: L = %d not in [1, %d]", L, SPP_MAX_L);
    for (int h = 0; h < L; ++h)
        SPP_CHECK(d_t[h] || g->M == 0, SPP_E_ARG, "spp_vip_propagate_general: no transition probabilities for hop %d", h + 1);
    SPP_HIP(hipSetDevice(ctx->device));
    hipStream_t st = ctx->stream;
    const int64_t N = g->N;
    SPP_TRY(ctx->y0.reserve((size_t)N * sizeof(float)));
    SPP_TRY(ctx->y1.reserve((size_t)N * sizeof(float)));
    SPP_TRY(ctx->tot.reserve((size_t)N * sizeof(double)));
    SPP_TRY(ctx->acc.reserve((size_t)N * sizeof(double)));
    const int64_t lcap = frontier_list_capacity(N, g->M);
    SPP_TRY(ctx->frontier.reserve((size_t)(lcap + 2) * sizeof(int32_t) + (4 + SPP_MAX_L + 2) * sizeof(unsigned long long)));
    unsigned long long* slots;
    int *d_bad, left_clean;
    SPP_TRY(vip_state(ctx, &slots, &d_bad, &left_clean));
    int32_t* flist = ctx->frontier.as<int32_t>();
    unsigned long long* fcount = reinterpret_cast<unsigned long long*>(flist + (lcap + (lcap & 1)));
    uint32_t* how = reinterpret_cast<uint32_t*>(fcount + 4);                 // [1 .. L]: how each hop fills its bins
    float* pcur = ctx->y0.as<float>();
    float* pnext = ctx->y1.as<float>();
    double* tot = ctx->tot.as<double>();
    double* acc = ctx->acc.as<double>();
    int64_t* bad_mirror = ctx->h_pinned + kHopMirror + 2 * SPP_MAX_L;
    const int include0 = (flags & SPP_VIP_INCLUDE_HOP0) ? 1 : 0;
    // a workgroup per 256 vertices, up to eight per CU: launching and counting 2048 of them cost a 10k-vertex graph more than
    // its vertices (122 us a call; 97 with forty)
    int fill_grid = ctx->num_cu * 8 < kTotalMax ? ctx->num_cu * 8 : kTotalMax;
    if ((N + kBlock - 1) / kBlock < fill_grid) fill_grid = (int)((N + kBlock - 1) / kBlock);
    // With the row-block structure at hand the push goes through bins (no global fp64 atomics).
    const bool binned = g->has_in && g->nrb > 0 && g->nrb <= kBinMaxBlocks && g->M > 0;
    int parts = 1;
    const int64_t part_stride = binned ? g->nrb << g->tile_rbits : N;
    uint2* bins = nullptr;
    uint32_t* cursor = nullptr;
    // the tiles are read as 128-bit vectors
    uintptr_t low = reinterpret_cast<uintptr_t>(g->col);
    for (int h = 0; h < L; ++h) low |= reinterpret_cast<uintptr_t>(d_t[h]);
    const bool tiles = binned && g->tile_off != nullptr && (low & 15) == 0;
    // two workgroups per CU, fewer where neither the tiles nor the rounds of the list need them; a multiple of eight
    const int64_t prepare_most = g->part_tiles > N / (8 * kFillBlock) ? g->part_tiles : N / (8 * kFillBlock) + 1;
    const int prepare_grid = prepare_most < ctx->num_cu * 2 ? (int)((prepare_most + 7) / 8 * 8) : ctx->num_cu * 2 / 8 * 8;
    const size_t fill_lds = binned ? 2 * (size_t)g->nrb * sizeof(uint32_t) : 0;
    const size_t sum_lds = binned ? sizeof(double) << g->tile_rbits : 0;
    if (binned) {
        parts = tile_parts(ctx->num_cu, g->nrb, g->M);
        SPP_TRY(ctx->acc.reserve((size_t)parts * (size_t)part_stride * sizeof(double)));
        acc = ctx->acc.as<double>();
        const int64_t room = g->M > 8 ? g->M : 8;        // entries, or as many weights, rounded up, and rows
        SPP_TRY(ctx->bins.reserve(((size_t)room + (size_t)g->nrb + 1) * sizeof(uint2)));
        bins = ctx->bins.as<uint2>();
        cursor = reinterpret_cast<uint32_t*>(bins + room);
        if (ctx->bin_lds_set < (int)fill_lds) {
            SPP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&vipg_bin_fill_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)fill_lds));
            ctx->bin_lds_set = (int)fill_lds;
        }
        if (tiles && !ctx->prepare_lds_set) {
            SPP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&vipg_prepare_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(PrepareLds)));
            ctx->prepare_lds_set = 1;
        }
        if (ctx->sum_lds_set < (int)sum_lds) {
            SPP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&vip_bin_sum_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)sum_lds));
            ctx->sum_lds_set = (int)sum_lds;
        }
    }
    {
        ScopedTimer tt(ctx, SPP_T_VIP_TOTAL, st);
        const HopCounters counters{fcount + 2, cursor, binned ? g->nrb + 1 : 0};
        int sample = 1;                          // of a graph of up to 8M vertices, one to two rounds of the launch are looked at
        while (sample < 8 && N >= 2 * sample * (int64_t)fill_grid * kBlock) sample *= 2;
        FillRule rule{tiles ? g->rowptr : nullptr, g->M, slots, how + 1, sample};
        vipg_init_kernel<<<fill_grid, kBlock, 0, st>>>(d_p0, N, pcur, tot, include0, d_bad, rule, counters);
        for (int h = 1; h <= L; ++h) {
            ScopedTimer th(ctx, SPP_T_VIP_HOP_FIRST + h - 1, st);
            const uint32_t* how_h = tiles ? how + h : nullptr;
            if (tiles)
                vipg_prepare_kernel<<<prepare_grid, kFillBlock, sizeof(PrepareLds), st>>>(
                    how_h, g->tile_off, g->tile_row, (int)g->part_tiles, g->M, pcur, g->rowptr, g->col, d_t[h - 1], g->tile_rbits,
                    (int)g->nrb, SplitBins(bins, g->M), d_bad, N, flist, fcount + 2);
            else
                launch_frontier_list(fill_grid, st, pcur, g->rowptr, N, flist, fcount + 2);
            if (binned) {
                // a bin is the range of the edges that end in its row block: block_first, with a stride of one
                vipg_bin_fill_kernel<<<ctx->num_cu * 2, kFillBlock, fill_lds, st>>>(
                    flist, fcount + 2, pcur, g->rowptr, g->col, d_t[h - 1], g->tile_rbits, (int)g->nrb,
                    g->block_first, 1, cursor, bins, d_bad, how_h);
                vip_bin_sum_kernel<<<(unsigned)(g->nrb * parts), kTileBlock, sum_lds, st>>>(
                    bins, g->M, cursor, g->block_first, 1, parts, g->tile_rbits, acc, part_stride, how_h);
            } else {
                fill_f64_kernel<<<fill_grid, kBlock, 0, st>>>(acc, N, 0.0);
                vipg_push_kernel<<<ctx->num_cu * 32, kBlock, 0, st>>>(flist, fcount + 2, pcur, g->rowptr, g->col,
                                                                     d_t[h - 1], acc, d_bad);
            }
            rule.how = how + h + 1;
            vipg_finish_kernel<<<fill_grid, kBlock, 0, st>>>(acc, tot, (h == 1 && !include0) ? 1 : 0, h == L ? 1 : 0,
                                                             d_p_hop ? d_p_hop + (int64_t)(h - 1) * N : nullptr,
                                                             d_p_total, pnext, N, parts, part_stride, counters, rule, d_bad, bad_mirror);
            float* tmp = pcur; pcur = pnext; pnext = tmp;
        }
    }
    SPP_HIP(hipGetLastError());
    ctx->vip_state_clean = left_clean;
    ctx->vip_hops = -L;
    if (flags & SPP_SYNC) {
        SPP_HIP(hipStreamSynchronize(st));
        SPP_CHECK(*bad_mirror == 0, SPP_E_ARG, "spp_vip_propagate_general: a probability lies outside [0, 1]; it was taken as 0");
    }
    return SPP_OK;
}

extern "C" int spp_vip_propagate(spp_ctx* ctx, const spp_graph* g, const int32_t* d_T, int64_t nT,
                                 int32_t B, const int32_t* fanouts, int32_t L,
                                 float* d_p_total, float* d_p_hop, uint32_t flags) {
    using namespace spp;
    SPP_CHECK(ctx && g && d_T && fanouts && d_p_total, SPP_E_ARG, "spp_vip_propagate: null argument");
    SPP_CHECK(g->has_in, SPP_E_ARG, "spp_vip_propagate: the graph was created without SPP_GRAPH_IN_LISTS");
    SPP_CHECK(L >= 1 && L <= SPP_MAX_L, SPP_E_ARG, "spp_vip_propagate: L = %d not in [1, %d]", L, SPP_MAX_L);
    SPP_CHECK(nT > 0 && B > 0, SPP_E_ARG, "spp_vip_propagate: nT = %lld, B = %d must be positive", (long long)nT, B);
    for (int h = 0; h < L; ++h)
        SPP_CHECK(fanouts[h] >= 1, SPP_E_ARG, "spp_vip_propagate: fanout %d of hop %d", fanouts[h], h + 1);
    SPP_HIP(hipSetDevice(ctx->device));
    hipStream_t st = ctx->stream;
    const int64_t N = g->N;
    SPP_TRY(ctx->y0.reserve((size_t)(N + 4) * sizeof(float)));       // dense hops read y as whole vectors of four
    SPP_TRY(ctx->y1.reserve((size_t)(N + 4) * sizeof(float)));
    static_assert(2 * SPP_MAX_L + 1 <= 64, "fits the mirror");
    SPP_TRY(ctx->tot.reserve((size_t)N * sizeof(double)));
    int parts = tile_parts(ctx->num_cu, g->nrb, g->M);
    // the chunked layout: with a row block per CU or more, one workgroup takes a whole block and
    // finishes its vertices itself (no partial sums leave the chip)
    if (g->has_x && g->nrb >= ctx->num_cu) parts = 1;
    const int64_t part_stride = g->nrb << g->tile_rbits;
    {
        const size_t tile_bytes = (size_t)parts * (size_t)part_stride * sizeof(double);
        const size_t push_bytes = (size_t)(N + 1) * sizeof(double);
        SPP_TRY(ctx->acc.reserve(tile_bytes > push_bytes ? tile_bytes : push_bytes));
    }
    // The push goes through bins where the chunked layout's value memory holds the entries (8 bytes for at most
    // M / kPushShare edges), the counts and the offsets, and a workgroup per row block fills the chip: graphs of
    // 4.2M vertices and more.  On 14M vertices it takes 396 us for a hop of 13.4M edges (atomics, with the clearing and
    // the finishing pass: 773) and, as its launches cost what they cost, 156 for one of 0.8M (149).
    const size_t bin_entries = (size_t)(g->M / kPushShare) + 1;
    const size_t bin_words = (size_t)kPushGroups * (size_t)g->nrb + 2 * (size_t)g->nrb + 1;
    const bool binned = g->has_x && parts == 1 && g->nrb <= kBinMaxBlocks &&
                        bin_entries * sizeof(uint2) + bin_words * sizeof(uint32_t) <= (size_t)g->x_entries * sizeof(float);
    const size_t bin_lds = (size_t)g->nrb * sizeof(uint32_t), bin_sum_lds = (sizeof(double) << kTileRowBits) + kTileWaves * kTouchedQueue * sizeof(uint16_t);
    const size_t lds_bytes = (sizeof(double) << g->tile_rbits) + (size_t)(kTileWaves * kTileWin + g->nch + 1) * sizeof(uint32_t);
    const size_t x_lds_expand = (sizeof(float) << kXSrcBits) + sizeof(float);
    static_assert(kXPad == (1u << kXSrcBits), "a padding entry indexes the slot after the chunk's values");
    const size_t x_lds_reduce = (sizeof(double) << kTileRowBits) + (2 * kXGroup + 1) * sizeof(uint32_t);
    const size_t bin_finish_lds = bin_sum_lds > x_lds_reduce ? bin_sum_lds : x_lds_reduce;
    const size_t hop_lds = g->has_x || lds_bytes < sizeof(PushLds) ? sizeof(PushLds) : lds_bytes;
    if (!binned && ctx->tile_lds_set < (int)hop_lds) {        // more than the 64 KB a launch may ask for by default
        SPP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&vip_hop_kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)hop_lds));
        ctx->tile_lds_set = (int)hop_lds;
    }
    if (g->has_x) {
        if (!ctx->x_lds_set) {
            SPP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&vip_expand_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)x_lds_expand));
            SPP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&vip_reduce_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)x_lds_reduce));
            ctx->x_lds_set = 1;
        }
        if (binned && ctx->push_lds_set < (int)bin_lds) {
            for (const void* k : {reinterpret_cast<const void*>(&vip_bin_count_kernel), reinterpret_cast<const void*>(&vip_bin_fill_kernel)})
                SPP_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bin_lds));
            SPP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&vip_bin_finish_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)bin_finish_lds));
            ctx->push_lds_set = (int)bin_lds;
        }
        SPP_TRY(ctx->xvals.reserve((size_t)(g->x_entries > 0 ? g->x_entries : 4) * sizeof(float)));
    }
    // A workgroup per 256 vertices, up to eight per CU (the finishing pass takes four vertices per thread and round: its
    // workgroups see no more than a round's vertices in kSegments segments, or ceil of their share).
    const int most = ctx->num_cu * 8 < kSegments ? ctx->num_cu * 8 : kSegments;
    auto groups = [&](int64_t n) { const int64_t w = (n + kBlock - 1) / kBlock; return (int)(w < 1 ? 1 : w < most ? w : most); };
    auto per_group = [&](int64_t n) { return (n + (int64_t)groups(n) * kBlock - 1) / ((int64_t)groups(n) * kBlock) * kBlock; };
    const int vgrid = groups(N), tgrid = groups(nT);
    // the frontier: in segments of the workgroups that list it, or (bins) as one list with the pieces of long rows
    const int64_t seg_all = vgrid * per_group(N) > tgrid * per_group(nT) ? vgrid * per_group(N) : tgrid * per_group(nT);
    int64_t lcap = binned ? frontier_list_capacity(N, g->M) : seg_all + 2 * kSegments;
    lcap += lcap & 1;
    SPP_TRY(ctx->frontier.reserve((size_t)lcap * sizeof(int32_t) + (1 + SPP_MAX_L + 2) * sizeof(unsigned long long)));
    unsigned long long* slots;
    int *d_bad, left_clean;
    SPP_TRY(vip_state(ctx, &slots, &d_bad, &left_clean));
    int32_t* flist = ctx->frontier.as<int32_t>();
    uint32_t* seg_count = reinterpret_cast<uint32_t*>(flist + seg_all);
    unsigned long long* fcursor = reinterpret_cast<unsigned long long*>(flist + lcap);       // of the one list
    uint32_t* how = reinterpret_cast<uint32_t*>(fcursor + 1);            // [1 .. L]: how each hop is walked
    int64_t* mirror = ctx->h_pinned + kHopMirror;
    float* ycur = ctx->y0.as<float>();
    float* ynext = ctx->y1.as<float>();
    double* tot = ctx->tot.as<double>();
    const int include0 = (flags & SPP_VIP_INCLUDE_HOP0) ? 1 : 0;
    double p0 = (double)B / (double)nT;
    if (p0 > 1.0) p0 = 1.0;

    {
        ScopedTimer tt(ctx, SPP_T_VIP_TOTAL, st);
        double* acc = ctx->acc.as<double>();
        HopPlan plan{1, g->M, slots, how, fcursor, mirror, {flist, binned ? nullptr : seg_count, per_group(nT), tgrid}};
        // the bins of a pushed hop (entries, counts, offsets), where a pulled one keeps its values
        uint2* bins = binned ? ctx->xvals.as<uint2>() : nullptr;
        uint32_t* off = binned ? reinterpret_cast<uint32_t*>(bins + bin_entries) : nullptr;
        uint32_t* total = binned ? off + (size_t)kPushGroups * (size_t)g->nrb : nullptr;
        uint32_t* bin_base = binned ? total + g->nrb : nullptr;
        vip_clear_kernel<<<vgrid, kBlock, 0, st>>>(ycur, include0 ? tot : nullptr, binned ? nullptr : acc, N);
        vip_init_kernel<<<tgrid, kBlock, 0, st>>>(d_T, nT, N, p0, (double)fanouts[0], g->rowptr, ycur, tot, include0, d_bad, plan);
        for (int h = 1; h <= L; ++h) {
            ScopedTimer th(ctx, SPP_T_VIP_HOP_FIRST + h - 1, st);
            const HopList walked = plan.l;
            plan.h = h + 1;
            plan.l.seg_cap = per_group(N); plan.l.nseg = vgrid;
            VipHop a;
            a.rowptr = g->rowptr;
            a.y_next = ynext; a.tot = tot;
            a.p_hop = d_p_hop ? d_p_hop + (int64_t)(h - 1) * N : nullptr;
            a.p_total = d_p_total;
            a.f_next = h < L ? (double)fanouts[h] : 0.0;
            a.first = (h == 1 && !include0) ? 1 : 0;
            a.last = (h == L) ? 1 : 0;
            a.next = plan;
            a.bad = h == 1 ? d_bad : nullptr;
            a.bad_mirror = mirror + 2 * SPP_MAX_L;
            const uint32_t* how_h = how + h;
            if (binned) {
                launch_frontier_list(most, st, ycur, g->rowptr, N, flist, fcursor, how_h);
                vip_bin_count_kernel<<<kPushGroups, kBinBlock, bin_lds, st>>>(flist, fcursor, ycur, g->rowptr, g->col, (int)g->nrb, off, how_h);
                vip_bin_offsets_kernel<<<(unsigned)((g->nrb + kOffBins - 1) / kOffBins), 1024, 0, st>>>(off, (int)g->nrb, total, how_h);
                vip_bin_fill_kernel<<<kPushGroups, kBinBlock, bin_lds, st>>>(flist, fcursor, ycur, g->rowptr, g->col, (int)g->nrb, off,
                                                                            total, bin_base, bins, how_h);
            } else {
                // as many workgroups as there are shares of row blocks, and one per CU at least for a push
                const int64_t shares = g->has_x ? 0 : g->nrb * parts;
                vip_hop_kernel<<<(unsigned)(shares > ctx->num_cu ? shares : ctx->num_cu), kTileBlock, hop_lds, st>>>(
                    walked, h, g->rowptr, g->col, g->t_edge, g->tile_first, g->nch, g->nrb, parts, g->tile_rbits, (uint32_t)N, ycur, acc,
                    part_stride, how_h);
            }
            int fused = 0;
            if (g->has_x) {
                const int64_t evec = g->x_entries / 4, eshare = evec / kExpandShare + 1;
                const int egrid = eshare < ctx->num_cu ? (int)eshare : ctx->num_cu;
                vip_expand_kernel<<<egrid, kXBlock, x_lds_expand, st>>>(g->x_src, g->x_chunk_first, g->x_nch, N, ycur,
                                                                        ctx->xvals.as<float>(), how_h);
                const ReduceArgs x{ctx->xvals.as<float>(), g->x_row, g->x_start, g->x_prefix, g->x_nch};
                if (binned) vip_bin_finish_kernel<<<(unsigned)g->nrb, kTileBlock, bin_finish_lds, st>>>(a, bins, bin_base, N, x, how_h);
                else vip_reduce_kernel<<<(unsigned)(g->nrb * parts), kXBlock, x_lds_reduce, st>>>(x, parts, N, acc, part_stride, a, how_h);
                fused = parts == 1;
            }
            if (!binned) vip_finish_kernel<<<vgrid, kBlock, 0, st>>>(a, how_h, fused, acc, parts, part_stride, N);
            float* t = ycur; ycur = ynext; ynext = t;
        }
    }
    SPP_HIP(hipGetLastError());
    ctx->vip_state_clean = left_clean;
    ctx->vip_hops = L;
    // training ids are checked on the device; the flag is read when the caller asks to wait
    if (flags & SPP_SYNC) {
        SPP_HIP(hipStreamSynchronize(st));
        SPP_CHECK(mirror[2 * SPP_MAX_L] == 0, SPP_E_ARG, "spp_vip_propagate: a training vertex id lies outside [0, N)");
    }
    return SPP_OK;
}
