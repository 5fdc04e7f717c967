// Node-wise fanout sampling into per-layer message-flow graphs (Sec. 2.3; the process of Sec. 3.1).
//
// Up to 64 minibatches are sampled by one set of launches: every kernel has a second grid dimension
// that names the minibatch, and each minibatch has its own workspace and counts, so the minibatches
// never interact.  Every count is kept on the device; all work is on the context's stream.  Per hop h,
// whatever the form:
//   1. prefix sums of c_i = min(f_h, d(S_{h-1}[i]))          -> indptr of MFG h, e_h
//   2. every target draws its subset (Philox words numbered by slot, Floyd's rule) and reads the ids
//   3. for every sampled id the position of its first appearance among S_{h-1} followed by the hop's
//      edges (an index below n_{h-1} means the vertex is an earlier one)
//   4. the first appearances of new ids are numbered in order -> S_h, n_h, src of those edges
//   5. src of a repeated id = its index in S_{h-1}, or the src of its first appearance
// Step 3 is where the ids meet.  With fanouts they meet in LDS (the hop_* kernels below: three
// launches per hop, one after the last hop).  The other form keeps a table in global memory (open
// addressing, 64-bit entries, six launches per hop: two per prefix sum), as do fanout sampling's hops above
// kHopLdsKeys ids; it is bound by the rate of global atomics, about 16 G/s, and serves the sampler with given probabilities, whose sizes no
// fanout bounds, calls that ask for it (SPP_SAMPLE_GLOBAL_TABLE) and calls whose edge bounds would make
// the LDS form's workspace the larger one by far.  Its table is right-sized per hop on the device: once
// e_h is known, the hop uses the first 2^k >= 2 (n_{h-1} + e_h) slots of the minibatch's region, clears
// exactly those, and the sample kernel offers S_{h-1} (value = index, which is below any position
// offered at this hop, so earlier vertices keep their ids) next to the new ids with atomic minima; the
// scan's first pass then reads what each entry resolved to.
//
// The per-minibatch pointers (a table too large for an argument block) stay on the device between
// calls and are stored again only when a call brings other buffers.
//
// The sampler with given transition probabilities (Sec. 3.1, paragraph after Prop. 1): a target takes
// every entry of its row independently with the entry's probability, so step 1 is a counting pass
// with the random draws (one wavefront per target, ballots) and step 2 repeats the draws to place the
// taken entries; no fanout bounds the sizes, so the counting pass also checks the caller's capacities
// and abandons a minibatch that would exceed them.
#include "spp_common.h"
#include "spp_device.h"

#include <algorithm>

namespace spp {

constexpr int kMaxBatches = SPP_MAX_SAMPLE_BATCHES;

// What differs between the minibatches of one call (stored in device memory once per call).
struct BatchDesc {
    const int32_t* seeds;
    int32_t*       S;                   // node ids
    int32_t*       indptr[SPP_MAX_L];
    int32_t*       src[SPP_MAX_L];
    int64_t*       counts;              // n[0..MAX_L], e[0..MAX_L]
    uint32_t*      tinfo;               // [0] mask, [1] shift of the table for the current hop, [2] abandoned (workspace)
    unsigned long long* taken;          // 64-bit count of taken entries of the current hop (given probabilities only)
    int64_t        ncap;                // capacities of the caller's buffers (checked on the device
    int64_t        ecap[SPP_MAX_L];     //   only when sizes are not bounded by fanouts)
    int32_t        nseeds;
    uint32_t       batch_lo;
};
// Fanout sampling in LDS: the counts once more, written and read by the device only.  A kernel asks for them together with
// the pointers; behind the pointer `counts` they were one more trip to memory at the head of each of a call's ten launches.
struct BatchCounts {
    uint32_t n[SPP_MAX_L + 1], e[SPP_MAX_L + 1];
};
struct BatchTable {
    BatchDesc   b[kMaxBatches];
    BatchCounts c[kMaxBatches];
};
// What changes from call to call even when the caller reuses its buffers: the seeds and the number
// of the minibatch.  It rides in the argument block of the call's first launch, which stores it
// into the table; the rest of the table stays on the device between calls.
struct BatchDyn {
    const int32_t* seeds;
    int32_t        nseeds;
    uint32_t       batch_lo;
};
struct BatchDynAll {
    BatchDyn d[kMaxBatches];
};

// What the minibatches of one call share.
struct SampleArgs {
    const int64_t* rowptr;
    const int32_t* col;
    int64_t        N;
    unsigned long long* tab;            // one region of `cap` entries per minibatch
    int64_t        cap;                 // slots per region (a power of two, sized for the bound on |S_L|)
    int32_t*       flat;                // one region of `flat_stride` entries per minibatch, in flat (edge) order: what
                                        // every sampled id of the current hop resolved to (an index into S_{h-1}, or
                                        // n_{h-1} + the flat position of the id's first appearance); with the table in
                                        // global memory, until the scan's first pass, the table slot of the id
    int32_t*       gids;                // the same shape: the sampled ids themselves
    int64_t        flat_stride;
    int64_t*       row0;                // one region of `node_stride` entries per minibatch: where the row of the i-th
    int32_t*       deg;                 // vertex of S starts in col[], and its length (fanout sampling: read from rowptr
    int64_t        node_stride;         // once, when the vertex joins S; every later pass reads these in order)
    unsigned long long* totals;         // context-wide running sums: [0] batches, [1] |S_L|, [2] edges
    int*           bad;
    int*           bad_next;            // the next call's flags: cleared by this call's last kernel
    int            L;
    int            h;                   // hop, 1-based
    int            f;                   // fanout of this hop
    uint64_t       seed;
    const float*   t;                   // this hop's transition probabilities (aligned with col), or null: fanout sampling
    int32_t*       cnt;                 // one region of `cnt_stride` per-target counts per minibatch (given probabilities)
    int64_t        cnt_stride;
    int*           ovf;                 // set when a minibatch was abandoned for lack of capacity
};

// Most members that S_h can have: S_L has the caller's room, the sets before it N, for which the workspaces and
// the later hops' buffers are sized (the bounds of spp_mfg_bound follow from n_h <= N hop by hop).  Distinct seeds
// never exceed it; repeated ones do (bad seeds too, which all become vertex 0) once a minibatch reaches nearly the
// whole graph: what lies beyond is then dropped, so that nothing is written or read out of range, and reported.
// (With given probabilities every hop has the caller's room, which ids_overflow() has checked.)
__device__ __forceinline__ int64_t vertex_cap(const BatchDesc& b, int64_t N, int h, int L) {
    return h < L ? N : (b.ncap < 0x7FFFFFFF ? b.ncap : 0x7FFFFFFF);
}

__device__ __forceinline__ unsigned long long* tab_of(const SampleArgs& a, int j) { return a.tab + (int64_t)j * a.cap; }
__device__ __forceinline__ int32_t* flat_of(const SampleArgs& a, int j) { return a.flat + (int64_t)j * a.flat_stride; }
__device__ __forceinline__ int32_t* gids_of(const SampleArgs& a, int j) { return a.gids + (int64_t)j * a.flat_stride; }
__device__ __forceinline__ int64_t* row0_of(const SampleArgs& a, int j) { return a.row0 + (int64_t)j * a.node_stride; }
__device__ __forceinline__ int32_t* deg_of(const SampleArgs& a, int j) { return a.deg + (int64_t)j * a.node_stride; }
__device__ __forceinline__ int32_t* cnt_of(const SampleArgs& a, int j) { return a.cnt + (int64_t)j * a.cnt_stride; }
constexpr int kE = SPP_MAX_L + 1;      // offset of e[] inside counts

// Zeroes the counts of the new minibatches, stores what this call brings (seeds, minibatch number)
// into the table and copies the seeds into S_0.  x-th of gx workgroups of minibatch j.
__device__ __forceinline__ void seeds_rows(const SampleArgs& a, BatchTable* t, const BatchDyn& dyn, int j, unsigned x,
                                           unsigned gx) {
    BatchDesc& b = t->b[j];
    if (x == 0 && threadIdx.x == 0) {
        int64_t* c = b.counts;
        for (int k = 1; k <= SPP_MAX_L; ++k) c[k] = 0;
        for (int k = 0; k <= SPP_MAX_L; ++k) c[kE + k] = 0;
        c[0] = dyn.nseeds;
        b.seeds = dyn.seeds; b.nseeds = dyn.nseeds; b.batch_lo = dyn.batch_lo;
        b.tinfo[2] = 0;
        if (b.taken) *b.taken = 0ull;
    }
    for (int64_t i = (int64_t)x * kBlock + threadIdx.x; i < dyn.nseeds; i += (int64_t)gx * kBlock) {
        int32_t v = dyn.seeds[i];
        if (v < 0 || v >= a.N) { v = 0; atomicOr(a.bad, 1); }       // reported; keeps later row reads in range
        b.S[i] = v;
        if (!a.t && i < a.node_stride) {
            const int64_t r0 = a.rowptr[v];
            row0_of(a, j)[i] = r0;
            deg_of(a, j)[i] = (int32_t)(a.rowptr[v + 1] - r0);
        }
    }
}
__global__ void __launch_bounds__(kBlock) seeds_kernel(SampleArgs a, BatchTable* t, BatchDynAll dyn) {
    const BatchBlock bb = batch_block();
    seeds_rows(a, t, dyn.d[bb.j], bb.j, bb.x, gridDim.x);
}

// ---- step 1 ----
// With given probabilities sizes are not bounded by fanouts: the 64-bit count of the counting pass
// decides whether the caller's buffers (and the table region laid out for them) hold this hop.
// The count stays as it is until the hop's last scan resets it, so every workgroup of a launch
// reads the same decision.
__device__ __forceinline__ bool hop_overflows(const SampleArgs& a, const BatchDesc& b) {
    return a.t != nullptr && *b.taken > (unsigned long long)b.ecap[a.h - 1];
}
// The flag tinfo[2] ("this minibatch was abandoned") is set by the Fin step of a scan, i.e. by one
// thread of a launch whose other workgroups read it.  Every reader in such a launch therefore ORs
// the flag with the condition under which that launch's Fin sets it, a condition that does not
// change during the launch (the hop's count of taken entries against the edge capacity in the
// offsets' scan; the scan's total against the vertex capacity in the scan that numbers the new
// vertices): whichever value of the flag a workgroup happens to see, the outcome is the same.
struct CountIn {
    SampleArgs a; const BatchTable* t;
    __device__ int64_t n(int j) const { return t->b[j].tinfo[2] || hop_overflows(a, t->b[j]) ? 0 : t->b[j].counts[a.h - 1]; }
    __device__ int64_t n(int j, int) const { return n(j); }
    __device__ int operator()(int j, int64_t i) const {
        if (a.t) return cnt_of(a, j)[i];
        const int d = deg_of(a, j)[i];
        return d < a.f ? d : a.f;
    }
};
struct CountOut {
    SampleArgs a; const BatchTable* t;
    __device__ void operator()(int j, int64_t i, int ex, int, int) const { t->b[j].indptr[a.h - 1][i] = ex; }
};
// This hop's table: the smallest power of two >= 2 (n_{h-1} + e_h), at least 1024 slots, never more
// than the region's `cap` slots (the host sized it for the bound, which dominates).
__device__ __forceinline__ void hop_table(int64_t cap, int64_t n_prev, int e_h, uint32_t& capj, int& shift) {
    const uint64_t want = 2ull * (uint64_t)(n_prev + (int64_t)(uint32_t)e_h);
    capj = 1024;
    shift = 22;
    while (capj < want && (int64_t)capj < cap) { capj <<= 1; --shift; }
}
struct CountFin {
    SampleArgs a; const BatchTable* t;
    __device__ void operator()(int j, int total) const {
        int64_t* c = t->b[j].counts;
        if (t->b[j].tinfo[2]) return;                        // abandoned at an earlier hop
        if (hop_overflows(a, t->b[j])) {
            t->b[j].tinfo[2] = 1;
            atomicOr(a.ovf, 1);
            return;
        }
        t->b[j].indptr[a.h - 1][c[a.h - 1]] = total;
        c[kE + a.h] = total;
        atomicAdd(&a.totals[2], (unsigned long long)(uint32_t)total);
        uint32_t capj;
        int shift;
        hop_table(a.cap, c[a.h - 1], total, capj, shift);
        t->b[j].tinfo[0] = capj - 1;
        t->b[j].tinfo[1] = (uint32_t)shift;
    }
};

// ---- step 2 ----
// Empties the part of the region that this hop's table occupies.  Rides at the end of the launch
// that writes the hop's offsets; the table's size follows from the scan's total, which every
// workgroup of that launch has.
struct TableClear {
    SampleArgs a; const BatchTable* t;
    __device__ void operator()(int j, unsigned x, unsigned gx, int total) const {
        if (t->b[j].tinfo[2] || hop_overflows(a, t->b[j])) return;
        unsigned long long* tab = tab_of(a, j);
        uint32_t capj;
        int shift;
        hop_table(a.cap, t->b[j].counts[a.h - 1], total, capj, shift);
        const int64_t stride = (int64_t)gx * kBlock;
        for (int64_t i = (int64_t)x * kBlock + threadIdx.x; i < (int64_t)capj; i += stride) tab[i] = ~0ull;
    }
};

template <int G>
__global__ void __launch_bounds__(kBlock) sample_kernel(SampleArgs a, const BatchTable* __restrict__ t) {
    const BatchBlock bb = batch_block();
    const int jb = bb.j;
    const int lane = lane_id();
    const int j = lane & (G - 1);                  // slot handled by this lane
    const int gbase = lane - j;                    // first lane of the group inside the wavefront
    const uint64_t gmask = (G == 64) ? ~0ull : (((1ull << (G & 63)) - 1ull) << gbase);
    constexpr int kGroupsPerWave = kWave / G;
    const int64_t n_prev = t->b[jb].counts[a.h - 1];
    const uint32_t batch_lo = t->b[jb].batch_lo;
    const int64_t wave = ((int64_t)bb.x * kBlock + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * kBlock) >> 6;
    const int f = a.f;
    const int32_t* __restrict__ S = t->b[jb].S;
    const int32_t* __restrict__ indptr = t->b[jb].indptr[a.h - 1];
    int32_t* __restrict__ flat = flat_of(a, jb);
    int32_t* __restrict__ gids = gids_of(a, jb);
    const int64_t* __restrict__ row0 = row0_of(a, jb);
    const int32_t* __restrict__ deg = deg_of(a, jb);
    unsigned long long* tab = tab_of(a, jb);
    const uint32_t mask = t->b[jb].tinfo[0];
    const int shift = (int)t->b[jb].tinfo[1];

    for (int64_t first = wave * kGroupsPerWave; first < n_prev; first += nwaves * kGroupsPerWave) {
        const int64_t i = first + (lane / G);
        const bool valid = i < n_prev;
        int64_t r0 = 0, d = 0;
        int32_t off = 0, v = 0;
        if (valid) {
            v = S[i];
            r0 = row0[i];
            d = deg[i];
            off = indptr[i];
        }
        const bool floyd = d > f;
        const int c = floyd ? f : (int)d;
        int64_t pos = j;                           // d <= f: the whole row, in row order
        if (floyd) {
            // Floyd's subset algorithm, one draw per slot: m = d - f + j, t uniform on [0, m]
            const uint64_t m = (uint64_t)(d - f + j);
            uint64_t tt = 0;
            if (j < f) {
                const uint32_t r = rand32(a.seed, batch_lo, (uint32_t)a.h, (uint32_t)v, (uint32_t)j);
                tt = ((uint64_t)r * (m + 1ull)) >> 32;
            }
            pos = (int64_t)tt;
            // slot jj takes t_jj unless an earlier slot already holds it, else m_jj (never held before)
            for (int jj = 1; jj < f; ++jj) {
                const int64_t tj = __shfl((long long)tt, gbase + jj, kWave);
                const bool hit = (j < jj) && (pos == tj);
                const uint64_t b = __ballot(hit) & gmask;
                if (j == jj && b != 0ull) pos = (int64_t)m;
            }
        }
        const bool mine = valid && j < c;
        int32_t gid = 0;
        int64_t e = -1;                            // flat position of this lane's sampled id, if it has one
        if (mine) {
            gid = a.col[r0 + pos];
            e = (int64_t)off + j;
            gids[e] = gid;
        }
        // the table was emptied for this hop, so the target is offered again with its index; the
        // group's last lane does it when it has no neighbour of its own (c < G), else lane 0 after
        // its neighbour
        const bool spare = c < G;
        uint32_t key = 0, val = 0;
        bool ins = false;
        if (mine) {
            key = (uint32_t)gid; val = (uint32_t)(n_prev + e); ins = true;
        } else if (valid && spare && j == G - 1) {
            key = (uint32_t)v; val = (uint32_t)i; ins = true;
        }
        if (ins) {
            const uint32_t slot = table_insert_min(tab, mask, shift, key, val);
            if (e >= 0) flat[e] = (int32_t)slot;
        }
        if (valid && !spare && j == 0) table_insert_min(tab, mask, shift, (uint32_t)v, (uint32_t)i);
    }
}

// ---- fanout sampling, three launches per hop ----
// The ids of a hop are deduplicated in LDS, partition by partition: an id belongs to the partition
// named by the top k bits of a multiplicative hash, and one workgroup of hop_dedup_kernel keeps a
// table for one partition.  What used to bound the hop was everything around that: each partition's
// workgroup read the whole hop's ids twice (half of a call of one minibatch), two launches per prefix
// sum, and hops above 131072 ids went through a table in global memory at the rate of global atomics.
// Here
//   hop_sample_kernel  draws a tile's subsets and leaves the tile's ids already dealt to the
//                      partitions: a run of (id, position) entries per tile, ordered by partition;
//   hop_dedup_kernel   walks only the runs of its own partition and marks the entries that repeat an id in
//                      place (nothing is scattered by edge); above kHopLdsKeys ids it offers the entries to a
//                      table in global memory instead, and hop_resolve_kernel marks the repeats;
//   hop_number_kernel  puts a tile's entries back in edge order in LDS and numbers the first appearances.
// No launch is spent on prefix sums and nothing ever waits for another workgroup: the sums that a
// workgroup needs (edges of the targets before its tile, new vertices before its tile) are kept per 256
// targets / per tile by the launches before it (one atomic add per tile), and the workgroup adds up
// the few hundred sums before its own itself.
// Per call, 3 hops: one minibatch of 1024 seeds on 2.4M vertices 0.21 -> 0.105 ms (waited for), 64 of
// them on 12M vertices 0.385 -> 0.256 ms, 8 of 4096 seeds with fanouts 20/15/10 on a 4M-vertex RMAT
// graph (hops of a million ids) 0.86 -> 0.45 ms.
constexpr int kHopTargets = 256;                 // most targets of a tile, and targets per kept edge sum
constexpr int kHopEdges = 4096;                  // most edges of a tile
constexpr int kHopSlots = 8192;                  // slots of a partition's table (64 KB of LDS)
constexpr int kHopSlotBits = 13;
constexpr int kHopPartKeys = 7168;               // ids a partition may hold on average, by the hop's bound
constexpr int kHopMaxPartsLog2 = 8;
constexpr int kHopGranules = 1024;               // most granules (runs of tiles, one tile as a rule) per hop
constexpr uint32_t kRepeat = 0x80000000u;        // marks a repeat in an entry's upper half, above the position it repeats
// Hops above this many ids meet in a table in global memory after all: a partition then has more entries than a
// workgroup's lanes keep in registers and would be walked twice, 2^(r + 1) times where its ids have to be taken in 2^r
// parts.  One hop in one minibatch, us in LDS / through the table: 0.5M ids 50 / 83, 1M 64 / 116, 2M 251 / 197,
// 4M 672 / 359, 8M 1818 / 684, 32M 8704 / 2767.
constexpr int64_t kHopLdsKeys = (int64_t)kHopPartKeys << kHopMaxPartsLog2;
constexpr int kDedupBlock = 1024;
constexpr int kDirectSeeds = 4096;               // up to this many seeds, hop 1 sums the seeds before a tile itself

// What the hop's kernels share.
struct HopArgs {
    const int64_t* rowptr;
    const int32_t* col;
    int64_t        N;
    uint64_t*      ent;                 // per minibatch `ent_stride` entries (id << 32 | position), tile after tile, by partition
    int64_t        ent_stride;          //   inside a tile; position: an index into S_{h-1}, or n_{h-1} + edge.  The upper half
                                        //   of an edge whose id appeared before becomes kRepeat | the first position of the id
    uint32_t*      seg;                 // per minibatch: [partition][tile] the run's start in the tile << 16 | its length
    int64_t        seg_stride;
    int64_t*       row0;                // per minibatch, per member of S_{L-1}: where its row starts in col[], its length
    int32_t*       deg;
    int64_t        node_stride;
    uint32_t*      csum;                // per minibatch two arrays of `csum_stride`, used by odd and even hops: edges of the
    int64_t        csum_stride;         //   hop per 256 targets; all zero between calls
    uint32_t*      fsum;                // per minibatch kHopGranules: first appearances per granule of tiles; all zero between calls
    unsigned long long* tab;            // per minibatch `tab_cap` slots of the id table of hops above kHopLdsKeys ids, all ones
    int64_t        tab_cap;             //   between such hops; null where the hop's bound is not above
    unsigned long long* totals;
    int*           bad;
    int*           bad_next;
    int64_t*       mirror;              // pinned host memory for the counts and flags of a call that is waited for, or null: 2 * kE counts per
                                        //   minibatch, the call's two flags, one more per minibatch
    int            n_items;
    int            L, h, f, f_next;     // f_next: fanout of hop h + 1 (0 at the last hop)
    uint64_t       seed;
};
__device__ __forceinline__ uint32_t* csum_of(const HopArgs& a, int j, int h) {
    return a.csum + ((int64_t)j * 2 + (h & 1)) * a.csum_stride;
}
// Targets per tile: 256 where the call fills the chip with such tiles (about two per CU), fewer below
// that, so that a single minibatch spreads over the CUs; the edges of a tile fit its LDS array.
__host__ __device__ __forceinline__ int hop_tile_cap(int f) { return f <= 16 ? 256 : f <= 32 ? 128 : 64; }
__host__ __device__ __forceinline__ int hop_tile_targets(int64_t n_prev, int n_items, int f) {
    const int cap = hop_tile_cap(f);
    int T = 16;
    while (T < cap && (int64_t)T * 1024 <= n_prev * n_items) T <<= 1;
    return T;
}
// log2 of the partitions: few enough ids per partition for its table, and (small calls) enough
// partitions for half the CUs while each keeps 2048 ids by the bound.
__host__ __device__ __forceinline__ int hop_parts_log2(int64_t n_prev, int n_items, int f) {
    const int64_t keys = n_prev * (1 + f);
    int k = 0;
    while (k < kHopMaxPartsLog2 && (keys >> k) > kHopPartKeys) ++k;
    while (k < kHopMaxPartsLog2 && ((int64_t)n_items << k) < 128 && (keys >> k) > 2048) ++k;
    return k;
}
// log2 of the tiles per granule.
__host__ __device__ __forceinline__ int hop_granule_log2(uint32_t ntiles) {
    int g = 0;
    while ((ntiles >> g) >= (uint32_t)kHopGranules) ++g;
    return g;
}

// The hop's table in global memory, if that is where its ids meet.
struct HopTable {
    unsigned long long* tab = nullptr;
    uint32_t slots = 0;
    int      shift = 0;
};
__device__ __forceinline__ HopTable hop_table_of(const HopArgs& a, int j, uint32_t n_prev, uint32_t e_h) {
    HopTable t;
    if (a.tab == nullptr || (int64_t)n_prev + e_h <= kHopLdsKeys) return t;
    t.tab = a.tab + (int64_t)j * a.tab_cap;
    hop_table(a.tab_cap, n_prev, (int)e_h, t.slots, t.shift);
    return t;
}

// The seeds of a call: hop 1 takes them from its argument block.
struct SeedsArg {
    BatchDynAll dyn;
    __device__ __forceinline__ int64_t n(const BatchCounts&, int j, int) const { return dyn.d[j].nseeds; }
    __device__ __forceinline__ uint32_t batch_lo(const BatchDesc&, int j) const { return dyn.d[j].batch_lo; }
};
struct NoSeedsArg {
    __device__ __forceinline__ int64_t n(const BatchCounts& c, int, int h) const { return c.n[h - 1]; }
    __device__ __forceinline__ uint32_t batch_lo(const BatchDesc& b, int) const { return b.batch_lo; }
};
__device__ __forceinline__ int32_t checked_seed(const HopArgs& a, int32_t v) {
    if (v >= 0 && v < a.N) return v;
    atomicOr(a.bad, 1);                          // reported; vertex 0 keeps later row reads in range
    return 0;
}
__device__ __forceinline__ void start_counts(BatchDesc& b, BatchCounts& k, const BatchDyn& dyn) {
    int64_t* c = b.counts;
    for (int i = 1; i <= SPP_MAX_L; ++i) c[i] = 0;
    for (int i = 0; i <= SPP_MAX_L; ++i)
        if (i != 1) c[kE + i] = 0;               // e_1 is written by the tile that ends hop 1
    c[0] = dyn.nseeds;
    k.n[0] = (uint32_t)dyn.nseeds;
    b.batch_lo = dyn.batch_lo;
}

// More seeds than hop 1 sums by itself: S_0, its rows and the edge sums of hop 1 in a launch before it.
__global__ void __launch_bounds__(kBlock) hop_seeds_kernel(HopArgs a, BatchTable* t, BatchDynAll dyn) {
    __shared__ int lds[4];
    const BatchBlock bb = batch_block();
    const int j = bb.j;
    const BatchDyn& d = dyn.d[j];
    if (bb.x == 0 && threadIdx.x == 0) start_counts(t->b[j], t->c[j], d);
    for (int64_t base = (int64_t)bb.x * kHopTargets; base < d.nseeds; base += (int64_t)gridDim.x * kHopTargets) {
        const int64_t i = base + threadIdx.x;
        int c = 0;
        if (i < d.nseeds) {
            const int32_t v = checked_seed(a, d.seeds[i]);
            const int64_t r0 = a.rowptr[v], len = a.rowptr[v + 1] - r0;
            t->b[j].S[i] = v;
            a.row0[(int64_t)j * a.node_stride + i] = r0;
            a.deg[(int64_t)j * a.node_stride + i] = (int32_t)len;
            c = len < a.f ? (int)len : a.f;
        }
        const int sum = block_reduce_sum(c, lds);
        if (threadIdx.x == 0) csum_of(a, j, 1)[base / kHopTargets] = (uint32_t)sum;
    }
}

// A repeated id takes the local id of its first appearance (an earlier edge of the same hop, final
// since the launch that numbered it), which the numbering left as a negative edge index.
__device__ __forceinline__ void relabel_repeats(const BatchDesc& b, const BatchCounts& c, int h, unsigned x, unsigned gx) {
    const int64_t e_h = c.e[h];
    int32_t* src = b.src[h - 1];
    for (int64_t e = (int64_t)x * kBlock + threadIdx.x; e < e_h; e += (int64_t)gx * kBlock) {
        const int32_t v = src[e];
        if (v < 0) src[e] = src[~v];
    }
}

// Floyd's subset algorithm for one target, one draw per slot: m = d - f + j, t uniform on [0, m]; slot j
// takes t unless an earlier slot already holds it, else m (which none holds).  A lane draws a whole
// subset: the four words of a Philox block serve four slots (a lane per slot computed the block for
// each of them and spent seven times the instructions).
template <int F>
__device__ __forceinline__ void floyd_positions(uint64_t seed, uint32_t batch_lo, uint32_t hop, uint32_t v, int32_t d, int f,
                                                uint32_t (&pos)[F]) {
#pragma unroll
    for (int q = 0; q < F / 4; ++q) {
        if (4 * q >= f) continue;
        const Philox4 r = philox4x32_10(v, (uint32_t)q, hop, batch_lo, (uint32_t)seed, (uint32_t)(seed >> 32));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t m = (uint32_t)(d - f + 4 * q + i);
            uint32_t t = __umulhi(r.w[i], m + 1u);
            bool held = false;
#pragma unroll
            for (int p = 0; p < 4 * q + i; ++p) held |= pos[p] == t;
            pos[4 * q + i] = held ? m : t;
        }
    }
}

// One tile of T consecutive targets at a time.  With F <= 16 slots (F >= f) a lane draws a target's
// subset, else a group of F lanes does (the comparisons of 64 slots do not belong in one lane).  The
// ids meet in an LDS array in edge order, from which the tile's entries are dealt to the partitions: a
// wavefront ranks 64 entries at a time among those of the same partition with ballots over the
// partition's bits, so the deal needs no LDS atomics (a handful of partitions made them collide) and
// keeps the order.  Bound by the latency of the random reads of col[].
template <int F, class Seeds>
__global__ void __launch_bounds__(kBlock, 4) hop_sample_kernel(HopArgs a, BatchTable* __restrict__ t, Seeds seeds) {
    constexpr bool kFirst = !__is_same(Seeds, NoSeedsArg);
    constexpr int kEdges = F <= 16 ? kHopTargets * F : kHopEdges;       // T * f, at most
    static_assert(kEdges <= kHopEdges, "a tile's edges");
    __shared__ int32_t gid_lds[kEdges];
    __shared__ uint16_t rank_lds[kEdges + kHopTargets];
    __shared__ int32_t tv[kHopTargets], toff[kHopTargets], tdeg[kHopTargets];
    __shared__ int64_t trow[kHopTargets];
    __shared__ uint32_t cnt[kBlock / kWave][1 << kHopMaxPartsLog2];      // entries, then first place, per wavefront and partition
    __shared__ int scan_lds[4];
    static_assert((1 << kHopMaxPartsLog2) <= kBlock && kHopTargets <= kBlock, "one partition and one target per thread");
    const BatchBlock bb = batch_block();
    const int jb = bb.j;
    BatchDesc& b = t->b[jb];
    const int64_t n_prev = seeds.n(t->c[jb], jb, a.h);
    const uint32_t batch_lo = seeds.batch_lo(b, jb);
    const int f = a.f;
    const int T = hop_tile_targets(n_prev, a.n_items, f);
    const int k = hop_parts_log2(n_prev, a.n_items, f);
    const int64_t ntiles = n_prev > 0 ? (n_prev + T - 1) / T : 1;
    int64_t* __restrict__ row0 = a.row0 + (int64_t)jb * a.node_stride;
    int32_t* __restrict__ deg = a.deg + (int64_t)jb * a.node_stride;
    int32_t* __restrict__ S = b.S;
    int32_t* __restrict__ indptr = b.indptr[a.h - 1];
    uint64_t* __restrict__ ent = a.ent + (int64_t)jb * a.ent_stride;
    uint32_t* __restrict__ seg = a.seg + (int64_t)jb * a.seg_stride;
    const uint32_t* __restrict__ csum = csum_of(a, jb, a.h);
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const uint64_t lt_mask = (1ull << lane) - 1ull;

    if constexpr (kFirst) {
        if (bb.x == 0 && threadIdx.x == 0) start_counts(b, t->c[jb], seeds.dyn.d[jb]);
    }
    for (int64_t tile = bb.x; tile < ntiles; tile += gridDim.x) {
        const int64_t i0 = tile * T;
        const int nt = n_prev - i0 < T ? (int)(n_prev - i0) : T;
        // edges of the targets before the tile
        int before = 0;
        if constexpr (kFirst) {
            for (int64_t i = threadIdx.x; i < i0; i += kBlock) {
                const int32_t v = checked_seed(a, seeds.dyn.d[jb].seeds[i]);
                const int64_t d = a.rowptr[v + 1] - a.rowptr[v];
                before += d < f ? (int)d : f;
            }
        } else {
            const int64_t g0 = i0 / kHopTargets;
            for (int64_t g = threadIdx.x; g < g0; g += kBlock) before = uadd(before, (int)csum[g]);
            const int64_t i = g0 * kHopTargets + threadIdx.x;
            if (i < i0) { const int d = deg[i]; before += d < f ? d : f; }
        }
        int c = 0, c_next = 0;
        if ((int)threadIdx.x < nt) {
            const int64_t i = i0 + threadIdx.x;
            int32_t v, d;
            int64_t r0;
            if constexpr (kFirst) {
                v = checked_seed(a, seeds.dyn.d[jb].seeds[i]);
                r0 = a.rowptr[v];
                d = (int32_t)(a.rowptr[v + 1] - r0);
                S[i] = v; row0[i] = r0; deg[i] = d;
            } else {
                v = S[i]; r0 = row0[i]; d = deg[i];
            }
            tv[threadIdx.x] = v; trow[threadIdx.x] = r0; tdeg[threadIdx.x] = d;
            c = d < f ? d : f;
            c_next = d < a.f_next ? d : a.f_next;
        }
        if (threadIdx.x < (1u << k))
            for (int w = 0; w < kBlock / kWave; ++w) cnt[w][threadIdx.x] = 0;
        int n_e;
        const int off = block_exclusive_scan(c, scan_lds, n_e);
        if ((int)threadIdx.x < nt) toff[threadIdx.x] = off;
        const int64_t ebase = (int64_t)(uint32_t)block_reduce_sum(before, scan_lds);      // its barriers publish the targets
        if (a.f_next) {                          // the targets are targets of the next hop too
            const int s = block_reduce_sum(c_next, scan_lds);
            if (threadIdx.x == 0 && s) atomicAdd(&csum_of(a, jb, a.h + 1)[i0 / kHopTargets], (uint32_t)s);
        }
        if ((int)threadIdx.x < nt) indptr[i0 + threadIdx.x] = (int32_t)(ebase + off);
        if (tile == ntiles - 1 && threadIdx.x == 0) {
            indptr[n_prev] = (int32_t)(ebase + n_e);
            b.counts[kE + a.h] = ebase + n_e;
            t->c[jb].e[a.h] = (uint32_t)(ebase + n_e);
            atomicAdd(&a.totals[2], (unsigned long long)(ebase + n_e));
        }
        // the draws
        if constexpr (F <= 16) {
            if ((int)threadIdx.x < nt) {
                const int32_t d = tdeg[threadIdx.x];
                const int n = d < f ? d : f;
                uint32_t pos[F];
#pragma unroll
                for (int u = 0; u < F; ++u) pos[u] = (uint32_t)u;        // d <= f: the whole row, in row order
                if (d > f) floyd_positions<F>(a.seed, batch_lo, (uint32_t)a.h, (uint32_t)tv[threadIdx.x], d, f, pos);
                const int64_t r0 = trow[threadIdx.x];
                int32_t gid[F];
#pragma unroll
                for (int u = 0; u < F; ++u) if (u < n) gid[u] = a.col[r0 + pos[u]];
#pragma unroll
                for (int u = 0; u < F; ++u) if (u < n) gid_lds[off + u] = gid[u];
            }
        } else {
            constexpr int kGroups = kBlock / F;
            const int jl = lane & (F - 1);           // slot handled by this lane
            const int gbase = lane - jl;             // first lane of the group inside the wavefront
            const uint64_t gmask = (F == 64) ? ~0ull : (((1ull << (F & 63)) - 1ull) << gbase);
            for (int q0 = 0; q0 < nt; q0 += kGroups) {
                const int q = q0 + (int)threadIdx.x / F;
                const bool valid = q < nt;
                const int d = valid ? tdeg[q] : 0;
                const bool floyd = d > f;
                uint32_t pos = (uint32_t)jl;
                if (__any(floyd)) {
                    const uint32_t m = (uint32_t)(d - f + jl);
                    uint32_t tt = 0;
                    if (floyd && jl < f) {
                        const uint32_t r = rand32(a.seed, batch_lo, (uint32_t)a.h, (uint32_t)tv[q], (uint32_t)jl);
                        tt = __umulhi(r, m + 1u);
                        pos = tt;
                    }
                    for (int jj = 1; jj < f; ++jj) {
                        const uint32_t tj = (uint32_t)__shfl((int)tt, gbase + jj, kWave);
                        const uint64_t hit = __ballot(floyd && jl < jj && pos == tj) & gmask;
                        if (jl == jj && hit != 0ull) pos = m;
                    }
                }
                if (valid && jl < (floyd ? f : d)) gid_lds[toff[q] + jl] = a.col[trow[q] + (int64_t)pos];
            }
        }
        __syncthreads();
        // the tile's entries (its edges, then its targets), dealt to the partitions; a wavefront takes 64
        // consecutive entries of every 256
        const int n_ent = n_e + nt;
        auto key_of = [&](int x) { return (uint32_t)(x < n_e ? gid_lds[x] : tv[x - n_e]); };
        auto part_of = [&](uint32_t key) { return k == 0 ? 0u : (key * 0x9E3779B1u) >> (32 - k); };
        for (int x0 = 0; x0 < n_ent; x0 += kBlock) {
            const int x = x0 + (int)threadIdx.x;
            const bool has = x < n_ent;
            const uint32_t p = has ? part_of(key_of(x)) : 0u;
            uint64_t same = __ballot(has);
            for (int bit = 0; bit < k; ++bit) {
                const bool one = (p >> bit) & 1u;
                const uint64_t bm = __ballot(one);
                same &= one ? bm : ~bm;
            }
            const uint32_t below = (uint32_t)__popcll(same & lt_mask);
            const uint32_t prior = cnt[wave][p];
            wave_lds_order();
            if (has && below == 0) cnt[wave][p] = prior + (uint32_t)__popcll(same);
            wave_lds_order();
            if (has) rank_lds[x] = (uint16_t)(prior + below);
        }
        __syncthreads();
        {
            uint32_t c4[kBlock / kWave], mine = 0;
            if (threadIdx.x < (1u << k))
#pragma unroll
                for (int w = 0; w < kBlock / kWave; ++w) { c4[w] = cnt[w][threadIdx.x]; mine += c4[w]; }
            int all;
            uint32_t st = (uint32_t)block_exclusive_scan((int)mine, scan_lds, all);
            if (threadIdx.x < (1u << k)) {
                seg[(int64_t)threadIdx.x * ntiles + tile] = (st << 16) | mine;
#pragma unroll
                for (int w = 0; w < kBlock / kWave; ++w) { cnt[w][threadIdx.x] = st; st += c4[w]; }
            }
        }
        __syncthreads();
        const int64_t ent0 = ebase + i0;
        for (int x = threadIdx.x; x < n_ent; x += kBlock) {      // the same entries as above: a wavefront's own places
            const uint32_t key = key_of(x);
            const uint32_t value = x < n_e ? (uint32_t)(n_prev + ebase + x) : (uint32_t)(i0 + x - n_e);
            ent[ent0 + cnt[wave][part_of(key)] + rank_lds[x]] = ((uint64_t)key << 32) | value;
        }
        __syncthreads();                         // the next tile overwrites the LDS arrays
    }
    if constexpr (!kFirst) {
        // what the hop before left: its granules' sums, and the repeats of its ids
        if (bb.x == 0)
            for (int g = threadIdx.x; g < kHopGranules; g += kBlock) a.fsum[(int64_t)jb * kHopGranules + g] = 0u;
        if (a.h > 1) relabel_repeats(b, t->c[jb], a.h - 1, bb.x, gridDim.x);
    }
}

// A partition's table: ids and smallest positions in two arrays (all ones: empty), buckets of four slots.
// An insertion reads a bucket's ids at once, claims an empty slot with a 32-bit compare-and-swap if the
// id is not there, and offers its position with an atomic minimum that returns nothing.  (64-bit
// entries probed slot by slot took a 64-bit compare-and-swap, the dearest LDS instruction, at each of the
// five or six probes of a wavefront's unluckiest lane.)  Returns the slot, or -1: no room.
constexpr uint32_t kNoId = 0xFFFFFFFFu;
__device__ __forceinline__ int hop_insert(uint32_t* ids, uint32_t* first, uint32_t home, uint32_t key, uint32_t pos) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    uint32_t bucket = home >> 2;
    for (int probes = 0; probes < 128;) {
        const u32x4 w = *reinterpret_cast<const u32x4*>(ids + 4 * bucket);
        int hit = w.x == key ? 0 : w.y == key ? 1 : w.z == key ? 2 : w.w == key ? 3 : -1;
        if (hit < 0) {
            const int empty = w.x == kNoId ? 0 : w.y == kNoId ? 1 : w.z == kNoId ? 2 : w.w == kNoId ? 3 : -1;
            if (empty < 0) { bucket = (bucket + 1) & (kHopSlots / 4 - 1); ++probes; continue; }
            const uint32_t old = atomicCAS(&ids[4 * bucket + empty], kNoId, key);
            if (old != kNoId && old != key) continue;          // another id took the slot: the bucket again
            hit = empty;
        }
        const int slot = (int)(4 * bucket) + hit;
        atomicMin(&first[slot], pos);
        return slot;
    }
    return -1;
}
__device__ __forceinline__ int hop_find(const uint32_t* ids, uint32_t home, uint32_t key) {
    uint32_t bucket = home >> 2;
    for (int probes = 0; probes < 128; ++probes) {
        for (int i = 0; i < 4; ++i) if (ids[4 * bucket + i] == key) return (int)(4 * bucket) + i;
        bucket = (bucket + 1) & (kHopSlots / 4 - 1);
    }
    return 0;                                    // not reached for an id that was inserted
}

// One workgroup per partition (or several partitions in turn).  The runs of up to 1024 tiles are laid
// end to end (a scan of their lengths in LDS), so that every lane has an entry whatever the length of
// a run; a lane finds its run by bisection.  Entries go into the table, and after a barrier every edge
// takes the smallest position of its id.  Up to 8192 entries a lane keeps its own in registers between
// the two; beyond that they are walked twice.  A partition whose ids do not fit the table (ids that share their
// hash's top bits, or a hop above kHopLdsKeys ids without the memory for its table) is taken in 2^r parts by the next
// r bits of the hash; at 19 bits in all at most four ids of a part share a bucket, because the hash is
// a bijection of 32-bit ids: any input fits.
// kLarge: the hop's bound allows more than kHopLdsKeys ids.
template <bool kLarge>
__global__ void __launch_bounds__(kDedupBlock) hop_dedup_kernel(HopArgs a, const BatchTable* __restrict__ t) {
    extern __shared__ __align__(16) uint32_t dedup_lds[];
    uint32_t* ids = dedup_lds;                                          // [kHopSlots]
    uint32_t* firsts = ids + kHopSlots;                                 // [kHopSlots]
    uint32_t* hist = firsts + kHopSlots;                                // [kHopGranules]
    uint32_t* pre = hist + kHopGranules;                                // [kDedupBlock] entries before run i
    uint32_t* adr = pre + kDedupBlock;                                  // [kDedupBlock] where run i lies, less pre[i]
    uint32_t* wsum = adr + kDedupBlock;                                 // [kDedupBlock / kWave]
    const int jb = blockIdx.x;                   // partitions are the slow index: workgroups without one come last
    const BatchDesc& b = t->b[jb];
    const uint32_t n_prev = t->c[jb].n[a.h - 1], e_h = t->c[jb].e[a.h];      // below 2^30 each
    const int T = hop_tile_targets(n_prev, a.n_items, a.f);
    const int k = hop_parts_log2(n_prev, a.n_items, a.f);
    const uint32_t ntiles = n_prev > 0 ? (n_prev + T - 1) / T : 1;
    if (blockIdx.y == 0) {                       // this hop's edge sums have been read: empty them
        uint32_t* cs = csum_of(a, jb, a.h);
        for (uint32_t g = threadIdx.x; g * kHopTargets < n_prev; g += kDedupBlock) cs[g] = 0u;
    }
    const int gshift = hop_granule_log2(ntiles);
    const int32_t* __restrict__ indptr = b.indptr[a.h - 1];
    uint64_t* ent = a.ent + (int64_t)jb * a.ent_stride;
    if constexpr (kLarge) {
        const HopTable ht = hop_table_of(a, jb, n_prev, e_h);
        if (ht.tab) {                            // resolved by the launch that follows
            for (uint32_t i = blockIdx.y * kDedupBlock + threadIdx.x; i < n_prev + e_h; i += gridDim.y * kDedupBlock)
                (void)table_insert_min(ht.tab, ht.slots - 1, ht.shift, (uint32_t)(ent[i] >> 32), (uint32_t)ent[i]);
            return;
        }
    }
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    auto resolve = [&](uint32_t at, uint32_t tile, uint32_t pos, int slot) {
        if (pos < n_prev) return;
        const uint32_t first = firsts[slot];
        if (first == pos) atomicAdd(&hist[tile >> gshift], 1u);
        else reinterpret_cast<uint32_t*>(ent + at)[1] = kRepeat | first;
    };
    const bool one_layout = ntiles <= (uint32_t)kDedupBlock;
    const uint32_t top = 1u << (31 - __clz((int)(one_layout ? ntiles : (uint32_t)kDedupBlock)));

    for (int part = blockIdx.y; part < (1 << k); part += gridDim.y) {
        const uint32_t* __restrict__ seg = a.seg + (int64_t)jb * a.seg_stride + (int64_t)part * ntiles;
        uint32_t total = 0;                      // entries of the runs laid out at present
        auto lay_out = [&](uint32_t c0) {
            __syncthreads();                     // the runs before are no longer read
            uint32_t len = 0, at = 0;
            const uint32_t tile = c0 + threadIdx.x;
            if (tile < ntiles) {
                const uint32_t s = seg[tile];
                len = s & 0xFFFFu;
                at = (uint32_t)indptr[tile * T] + tile * T + (s >> 16);
            }
            const uint32_t inc = (uint32_t)wave_inclusive_scan((int)len);
            if (lane == kWave - 1) wsum[wave] = inc;
            __syncthreads();
            uint32_t base = 0, all = 0;
            for (int w = 0; w < kDedupBlock / kWave; ++w) { const uint32_t v = wsum[w]; all += v; if (w < wave) base += v; }
            const uint32_t ex = base + inc - len;
            pre[threadIdx.x] = ex;
            adr[threadIdx.x] = at - ex;
            total = all;
            __syncthreads();
        };
        auto run_of = [&](uint32_t x, uint32_t n) {  // the run of entry x of the n runs laid out: last one with pre[r] <= x
            uint32_t r = 0;
            for (uint32_t s = top; s > 0; s >>= 1)
                if (r + s < n && pre[r + s] <= x) r += s;
            return r;
        };
        // all entries of the partition, for the partitions that do not fit a lane's registers
        auto walk = [&](auto&& fn) {
            for (uint32_t c0 = 0; c0 < ntiles; c0 += kDedupBlock) {
                if (!one_layout) lay_out(c0);
                const uint32_t n = ntiles - c0 < (uint32_t)kDedupBlock ? ntiles - c0 : kDedupBlock;
                for (uint32_t x = threadIdx.x; x < total; x += kDedupBlock) {
                    const uint32_t r = run_of(x, n), at = adr[r] + x;
                    fn(ent[at], at, c0 + r);
                }
            }
        };
        auto empty_table = [&]() {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 ones = {kNoId, kNoId, kNoId, kNoId};
            for (int i = threadIdx.x; i < 2 * kHopSlots / 4; i += kDedupBlock) reinterpret_cast<u32x4*>(ids)[i] = ones;
        };
        auto hash_of = [](uint32_t key) { return key * 0x9E3779B1u; };
        bool done = false;
        int rbits = 0;
        if (threadIdx.x < kHopGranules) hist[threadIdx.x] = 0u;
        empty_table();
        if (one_layout) lay_out(0); else __syncthreads();
        constexpr int R = 8;
        if (one_layout && total <= R * kDedupBlock) {
            uint32_t pos[R], slot_run[R];        // slot << 16 | run (a run is one of 1024 at most)
            bool ok = true;
#pragma unroll
            for (int u0 = 0; u0 < R; u0 += 4) {
                unsigned long long e[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (threadIdx.x + (u0 + u) * kDedupBlock < total) {
                        slot_run[u0 + u] = run_of(threadIdx.x + (u0 + u) * kDedupBlock, ntiles);
                        e[u] = ent[adr[slot_run[u0 + u]] + threadIdx.x + (u0 + u) * kDedupBlock];
                    }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (threadIdx.x + (u0 + u) * kDedupBlock < total) {
                        const uint32_t key = (uint32_t)(e[u] >> 32);
                        pos[u0 + u] = (uint32_t)e[u];
                        const int slot = hop_insert(ids, firsts, (hash_of(key) << k) >> (32 - kHopSlotBits), key, pos[u0 + u]);
                        slot_run[u0 + u] |= (uint32_t)slot << 16;
                        ok = ok && slot >= 0;
                    }
            }
            if (!__syncthreads_or(!ok)) {
#pragma unroll
                for (int u = 0; u < R; ++u)
                    if (threadIdx.x + u * kDedupBlock < total) {
                        const uint32_t r = slot_run[u] & 0xFFFFu;
                        resolve(adr[r] + threadIdx.x + u * kDedupBlock, r, pos[u], (int)(slot_run[u] >> 16));
                    }
                done = true;
            } else {
                rbits = 1;
            }
        } else {
            while (k + rbits < 32 - kHopSlotBits && ((n_prev + e_h) >> (k + rbits)) > (uint32_t)kHopSlots) ++rbits;
        }
        while (!done) {
            done = true;
            __syncthreads();
            if (threadIdx.x < kHopGranules) hist[threadIdx.x] = 0u;
            for (uint32_t r = 0; r < (1u << rbits) && done; ++r) {
                empty_table();
                __syncthreads();
                auto in_part = [&](uint32_t key) { return rbits == 0 || ((hash_of(key) << k) >> (32 - rbits)) == r; };
                auto home_of = [&](uint32_t key) { return (hash_of(key) << (k + rbits)) >> (32 - kHopSlotBits); };
                bool ok = true;
                walk([&](uint64_t e, uint32_t, uint32_t) {
                    const uint32_t key = (uint32_t)(e >> 32);
                    // an entry that an earlier attempt has marked repeats an id whose first entry is still there
                    if (!(key & kRepeat) && in_part(key)) ok = hop_insert(ids, firsts, home_of(key), key, (uint32_t)e) >= 0 && ok;
                });
                if (__syncthreads_or(!ok)) { ++rbits; done = false; break; }
                walk([&](uint64_t e, uint32_t at, uint32_t tile) {
                    const uint32_t key = (uint32_t)(e >> 32);
                    if ((uint32_t)e >= n_prev && !(key & kRepeat) && in_part(key))
                        resolve(at, tile, (uint32_t)e, hop_find(ids, home_of(key), key));
                });
                __syncthreads();
            }
        }
        __syncthreads();
        if (threadIdx.x < kHopGranules && hist[threadIdx.x])
            atomicAdd(&a.fsum[(int64_t)jb * kHopGranules + threadIdx.x], hist[threadIdx.x]);
        __syncthreads();
    }
}
static_assert(kHopGranules <= kDedupBlock, "one granule per thread");

// The hops whose ids met in the table in global memory: every edge takes the smallest position of its id, a granule of
// tiles at a time.  Launched only where the hop's bound allows such a hop; leaves at once where it is none.
__global__ void __launch_bounds__(kBlock) hop_resolve_kernel(HopArgs a, const BatchTable* __restrict__ t) {
    __shared__ int lds[4];
    const BatchBlock bb = batch_block();
    const int jb = bb.j;
    const BatchDesc& b = t->b[jb];
    const uint32_t n_prev = t->c[jb].n[a.h - 1], e_h = t->c[jb].e[a.h];
    const HopTable ht = hop_table_of(a, jb, n_prev, e_h);
    if (ht.tab == nullptr) return;
    const uint32_t T = (uint32_t)hop_tile_targets(n_prev, a.n_items, a.f), ntiles = (n_prev + T - 1) / T;      // n_prev > 0 here
    const int gshift = hop_granule_log2(ntiles);
    const uint32_t ngran = (ntiles + (1u << gshift) - 1) >> gshift;
    const int32_t* __restrict__ indptr = b.indptr[a.h - 1];
    uint64_t* ent = a.ent + (int64_t)jb * a.ent_stride;
    for (uint32_t g = bb.x; g < ngran; g += gridDim.x) {
        // the entries of consecutive tiles lie end to end
        const uint32_t i0 = (g << gshift) * T, i1 = (uint64_t)((g + 1) << gshift) * T < n_prev ? ((g + 1) << gshift) * T : n_prev;
        const uint32_t x0 = (uint32_t)indptr[i0] + i0, x1 = (uint32_t)indptr[i1] + i1;
        int firsts = 0;
        for (uint32_t x = x0 + threadIdx.x; x < x1; x += kBlock) {
            const uint64_t e = ent[x];
            uint32_t first = 0;
            if ((uint32_t)e < n_prev) continue;
            (void)table_find(ht.tab, ht.slots - 1, ht.shift, (uint32_t)(e >> 32), first);      // it is there
            if (first == (uint32_t)e) ++firsts;
            else reinterpret_cast<uint32_t*>(ent + x)[1] = kRepeat | first;
        }
        const int all = block_reduce_sum(firsts, lds);
        if (threadIdx.x == 0) a.fsum[(int64_t)jb * kHopGranules + g] = (uint32_t)all;
    }
}

// Numbers the first appearances, a granule of tiles at a time: a tile's entries go back to edge order
// through LDS, the new vertices are appended to S_h in order, and the row of a vertex that will be a
// target of the next hop is looked up here, once.
template <bool kLarge>
__global__ void __launch_bounds__(kBlock) hop_number_kernel(HopArgs a, BatchTable* __restrict__ t) {
    __shared__ uint32_t what[kHopEdges];         // per edge of the tile: the upper half of its entry
    __shared__ int scan_lds[4];
    __shared__ uint32_t next_sum[1024 / kHopTargets + 2];
    const BatchBlock bb = batch_block();
    const int jb = bb.j;
    const BatchDesc& b = t->b[jb];
    const uint32_t n_prev = t->c[jb].n[a.h - 1];
    const int T = hop_tile_targets(n_prev, a.n_items, a.f);
    const uint32_t ntiles = n_prev > 0 ? (n_prev + T - 1) / T : 1;
    const int gshift = hop_granule_log2(ntiles);
    const uint32_t ngran = (ntiles + (1u << gshift) - 1) >> gshift;
    const int32_t* __restrict__ indptr = b.indptr[a.h - 1];
    const uint64_t* __restrict__ ent = a.ent + (int64_t)jb * a.ent_stride;
    const uint32_t* __restrict__ fsum = a.fsum + (int64_t)jb * kHopGranules;
    const uint32_t id_cap = (uint32_t)vertex_cap(b, a.N, a.h, a.L);
    int32_t* __restrict__ src = b.src[a.h - 1];
    int64_t* __restrict__ row0 = a.row0 + (int64_t)jb * a.node_stride;
    int32_t* __restrict__ deg = a.deg + (int64_t)jb * a.node_stride;
    if constexpr (kLarge) {
        const HopTable ht = hop_table_of(a, jb, n_prev, t->c[jb].e[a.h]);  // has served
        typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
        for (uint32_t i = bb.x * kBlock + threadIdx.x; i < ht.slots / 2; i += gridDim.x * kBlock)
            reinterpret_cast<u64x2*>(ht.tab)[i] = u64x2{~0ull, ~0ull};
    }
    for (uint32_t g = bb.x; g < ngran; g += gridDim.x) {
        int before = 0;
        for (uint32_t i = threadIdx.x; i < g; i += kBlock) before = uadd(before, (int)fsum[i]);
        uint32_t id0 = n_prev + (uint32_t)block_reduce_sum(before, scan_lds);      // the next new vertex
        const uint32_t tend = ((g + 1) << gshift) < ntiles ? (g + 1) << gshift : ntiles;
        for (uint32_t tile = g << gshift; tile < tend; ++tile) {
            const uint32_t i0 = tile * T, i1 = i0 + T < n_prev ? i0 + T : n_prev;
            const uint32_t ebase = (uint32_t)indptr[i0], n_e = (uint32_t)indptr[i1] - ebase;
            const uint32_t n_ent = n_e + (i1 - i0);
            for (uint32_t x = threadIdx.x; x < n_ent; x += kBlock) {
                const uint64_t e = ent[ebase + i0 + x];
                if ((uint32_t)e >= n_prev) what[(uint32_t)e - n_prev - ebase] = (uint32_t)(e >> 32);
            }
            __syncthreads();
            for (uint32_t e0 = 0; e0 < n_e; e0 += kBlock * 4) {
                const uint32_t e = e0 + threadIdx.x * 4;       // four consecutive edges
                uint32_t w[4];
                int mine = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    w[u] = e + u < n_e ? what[e + u] : kRepeat;
                    mine += w[u] < kRepeat ? 1 : 0;
                }
                if (threadIdx.x < sizeof(next_sum) / sizeof(next_sum[0])) next_sum[threadIdx.x] = 0u;
                int total;
                uint32_t id = id0 + (uint32_t)block_exclusive_scan(mine, scan_lds, total);
                int64_t r0[4];
                int32_t rlen[4];
                if (a.f_next) {                  // all four rows' bounds are in flight together
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (w[u] < kRepeat) {
                            r0[u] = a.rowptr[w[u]];
                            rlen[u] = (int32_t)(a.rowptr[w[u] + 1] - r0[u]);
                        }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (e + u >= n_e) continue;
                    int32_t out;
                    if (w[u] < kRepeat) {
                        if (id < id_cap) {
                            b.S[id] = (int32_t)w[u];
                            if (a.f_next) {
                                row0[id] = r0[u];
                                deg[id] = rlen[u];
                                atomicAdd(&next_sum[id / kHopTargets - id0 / kHopTargets], (uint32_t)(rlen[u] < a.f_next ? rlen[u] : a.f_next));
                            }
                        }
                        out = (int32_t)(id < id_cap ? id : id_cap - 1);
                        ++id;
                    } else {
                        // an earlier vertex, or (left for the relabel) a first appearance earlier in this hop
                        const uint32_t first = w[u] & ~kRepeat;
                        out = first < n_prev ? (int32_t)first : ~(int32_t)(first - n_prev);
                    }
                    src[ebase + e + u] = out;
                }
                if (a.f_next) {
                    __syncthreads();
                    if (threadIdx.x < sizeof(next_sum) / sizeof(next_sum[0]) && next_sum[threadIdx.x])
                        atomicAdd(&csum_of(a, jb, a.h + 1)[id0 / kHopTargets + threadIdx.x], next_sum[threadIdx.x]);
                    __syncthreads();
                }
                id0 += (uint32_t)total;
            }
            __syncthreads();                     // the next tile overwrites what[]
        }
        if (g == ngran - 1 && threadIdx.x == 0) {
            const bool over = id0 > id_cap;
            if (over) { atomicOr(a.bad, 4); id0 = id_cap; }
            b.counts[a.h] = id0;
            t->c[jb].n[a.h] = id0;
            if (a.h == a.L) {
                atomicAdd(&a.totals[1], (unsigned long long)id0);
                atomicAdd(&a.totals[0], 1ull);
                if (a.mirror) {
                    int64_t* m = a.mirror + (int64_t)jb * 2 * kE;
                    for (int q = 0; q < 2 * kE; ++q) m[q] = q == a.h ? (int64_t)id0 : b.counts[q];
                    // the flags so far, and this minibatch's own of the last hop (another's may come later)
                    int* fl = reinterpret_cast<int*>(a.mirror + (int64_t)kMaxBatches * 2 * kE);
                    if (jb == 0) { fl[0] = *a.bad; fl[1] = 0; }
                    fl[2 + jb] = over ? 4 : 0;
                }
            }
        }
    }
}

// After the last hop: its repeats, and what the next call expects empty.
__global__ void __launch_bounds__(kBlock) hop_last_kernel(HopArgs a, const BatchTable* __restrict__ t) {
    const BatchBlock bb = batch_block();
    if (bb.x == 0)
        for (int g = threadIdx.x; g < kHopGranules; g += kBlock) a.fsum[(int64_t)bb.j * kHopGranules + g] = 0u;
    relabel_repeats(t->b[bb.j], t->c[bb.j], a.h, bb.x, gridDim.x);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 2) a.bad_next[threadIdx.x] = 0;
}

// ---- steps 1 and 2 with given transition probabilities ----
// Entry k of v's row is taken iff rand32(seed, batch, hop, v, k) < floor(t * 2^32); a probability
// outside [0, 1] counts as 0 and is reported.  A lane decides four consecutive entries at a time:
// their draws are the four words of one Philox block (that is how rand32 numbers them).
// Returns the 4-bit mask of the taken ones among entries k4 .. k4+3 (k4 a multiple of 4) of a row of d.
__device__ __forceinline__ uint32_t general_take4(const SampleArgs& a, uint32_t batch_lo, int64_t v, int64_t r0, int64_t k4,
                                                  int64_t d) {
    if (k4 >= d) return 0u;
    const Philox4 p = philox4x32_10((uint32_t)v, (uint32_t)(k4 >> 2), (uint32_t)a.h, batch_lo, (uint32_t)a.seed,
                                    (uint32_t)(a.seed >> 32));
    uint32_t m = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (k4 + i < d) {
            const float tt = a.t[r0 + k4 + i];
            if (!(tt >= 0.0f && tt <= 1.0f)) { atomicOr(a.bad, 2); continue; }
            const uint64_t thr = (uint64_t)((double)tt * 4294967296.0);
            if ((uint64_t)p.w[i] < thr) m |= 1u << i;
        }
    }
    return m;
}
// A row is walked by a group of G lanes (G = 16: four targets per wavefront; G = 64: one), 4 G
// entries per step.  Most rows hold a handful of entries, a few tens of thousands: rows of at most
// kShortRow entries are taken four per wavefront in a first sweep over the targets, longer ones by
// a whole wavefront in a second sweep.
constexpr int kShortRow = 256;
constexpr int kShortGroup = 16;

// Taken entries among the 4 G entries a group decides in one step: in all of the group's lanes, and
// in its lanes below this one.  gmask = the group's lanes, lt_mask = the wavefront's lanes below this one.
__device__ __forceinline__ int taken_in_group(uint32_t m, uint64_t gmask, uint64_t lt_mask, int& below) {
    int all = 0;
    below = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint64_t b = __ballot((m >> i) & 1u) & gmask;
        all += __popcll(b);
        below += __popcll(b & lt_mask);
    }
    return all;
}

// Which target a lane group works on in sweep `longer` (0: short rows, G = kShortGroup; 1: long rows, G = 64).
struct GroupWalk {
    int64_t first, stride;      // first target of this group and the step to its next one
    uint32_t glane;             // lane inside the group
    uint64_t gmask;             // the group's lanes
};
template <int G>
__device__ __forceinline__ GroupWalk group_walk(const BatchBlock& bb) {
    const int lane = lane_id();
    const int64_t wave = ((int64_t)bb.x * kBlock + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * kBlock) >> 6;
    GroupWalk w;
    w.first = wave * (kWave / G) + lane / G;
    w.stride = nwaves * (kWave / G);
    w.glane = (uint32_t)(lane % G);
    w.gmask = G == kWave ? ~0ull : ((1ull << (G & 63)) - 1ull) << (lane - lane % G);
    return w;
}

template <int G>
__device__ __forceinline__ void general_count_rows(const SampleArgs& a, const BatchDesc& b, const BatchBlock& bb,
                                                   int32_t* __restrict__ cnt, unsigned long long& mine) {
    const GroupWalk w = group_walk<G>(bb);
    const int64_t n_prev = b.counts[a.h - 1];
    const int64_t rounds = (n_prev + w.stride - 1) / w.stride;           // whole wavefronts reach the ballots
    for (int64_t it = 0; it < rounds; ++it) {
        const int64_t i = w.first + it * w.stride;
        int64_t v = 0, r0 = 0, d = 0;
        if (i < n_prev) {
            v = b.S[i];
            r0 = a.rowptr[v];
            d = a.rowptr[v + 1] - r0;
            if ((d > kShortRow) != (G == kWave)) d = 0;                  // the other sweep's row
        }
        int64_t c = 0;
        // groups of one wavefront walk rows of different lengths: all step until the longest is done
        for (int64_t k0 = 0; __any(k0 < d); k0 += 4 * G) {
            int below;
            c += taken_in_group(k0 < d ? general_take4(a, b.batch_lo, v, r0, k0 + 4 * w.glane, d) : 0u, w.gmask, 0ull, below);
        }
        // a count beyond any capacity is stored saturated; the 64-bit total decides
        if (i < n_prev && w.glane == 0 && ((a.rowptr[v + 1] - a.rowptr[v] > kShortRow) == (G == kWave))) {
            cnt[i] = (int32_t)(c < 0x7FFFFFFFll ? c : 0x7FFFFFFFll);
            mine += (unsigned long long)c;
        }
    }
}

__global__ void __launch_bounds__(kBlock) general_count_kernel(SampleArgs a, const BatchTable* __restrict__ t) {
    __shared__ unsigned long long red[kBlock];
    const BatchBlock bb = batch_block();
    const int jb = bb.j;
    if (t->b[jb].tinfo[2]) return;
    unsigned long long mine = 0;
    general_count_rows<kShortGroup>(a, t->b[jb], bb, cnt_of(a, jb), mine);
    general_count_rows<kWave>(a, t->b[jb], bb, cnt_of(a, jb), mine);
    red[threadIdx.x] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long s = 0;
        for (int k = 0; k < kBlock; ++k) s += red[k];
        if (s) atomicAdd(t->b[jb].taken, s);
    }
}

template <int G>
__device__ __forceinline__ void general_sample_rows(const SampleArgs& a, const BatchDesc& b, const BatchBlock& bb,
                                                    int32_t* __restrict__ flat, int32_t* __restrict__ gids,
                                                    unsigned long long* tab) {
    const GroupWalk w = group_walk<G>(bb);
    const int lane = lane_id();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t n_prev = b.counts[a.h - 1];
    const int32_t* __restrict__ indptr = b.indptr[a.h - 1];
    const uint32_t mask = b.tinfo[0];
    const int shift = (int)b.tinfo[1];
    const int64_t rounds = (n_prev + w.stride - 1) / w.stride;
    for (int64_t it = 0; it < rounds; ++it) {
        const int64_t i = w.first + it * w.stride;
        int64_t v = 0, r0 = 0, d = 0, e = 0;
        if (i < n_prev) {
            v = b.S[i];
            r0 = a.rowptr[v];
            d = a.rowptr[v + 1] - r0;
            if ((d > kShortRow) != (G == kWave)) d = 0;
            else {
                e = indptr[i];
                // the table was emptied for this hop, so the target is offered again with its index
                if (w.glane == 0) table_insert_min(tab, mask, shift, (uint32_t)v, (uint32_t)i);
            }
        }
        for (int64_t k0 = 0; __any(k0 < d); k0 += 4 * G) {
            const int64_t k4 = k0 + 4 * w.glane;
            const uint32_t m = k0 < d ? general_take4(a, b.batch_lo, v, r0, k4, d) : 0u;
            int below;
            const int all = taken_in_group(m, w.gmask, lt_mask, below);
            int64_t pos = e + below;                   // entries ascend with the lane, then inside the lane
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if ((m >> q) & 1u) {
                    const int32_t gid = a.col[r0 + k4 + q];
                    gids[pos] = gid;
                    flat[pos] = (int32_t)table_insert_min(tab, mask, shift, (uint32_t)gid, (uint32_t)(n_prev + pos));
                    ++pos;
                }
            }
            e += all;
        }
    }
}

__global__ void __launch_bounds__(kBlock) general_sample_kernel(SampleArgs a, const BatchTable* __restrict__ t) {
    const BatchBlock bb = batch_block();
    const int jb = bb.j;
    if (t->b[jb].tinfo[2]) return;
    general_sample_rows<kShortGroup>(a, t->b[jb], bb, flat_of(a, jb), gids_of(a, jb), tab_of(a, jb));
    general_sample_rows<kWave>(a, t->b[jb], bb, flat_of(a, jb), gids_of(a, jb), tab_of(a, jb));
}

// ---- step 4 ----
struct NewIn {
    SampleArgs a; const BatchTable* t;
    __device__ int64_t n(int j) const { return t->b[j].tinfo[2] ? 0 : t->b[j].counts[kE + a.h]; }
    // What the entry resolved to is read from its slot here (a random 8-byte read that moves a whole
    // line) and kept in the slot's place; the outcome is left in the entry's place in the hop's src
    // array (-2 first appearance, -1 repeat) for the second pass.
    __device__ int operator()(int j, int64_t e) const {
        int32_t* __restrict__ flat = flat_of(a, j);
        const uint32_t val = (uint32_t)tab_of(a, j)[(uint32_t)flat[e]];
        flat[e] = (int32_t)val;
        const int first = (int64_t)val == t->b[j].counts[a.h - 1] + e ? 1 : 0;
        t->b[j].src[a.h - 1][e] = first ? -2 : -1;
        return first;
    }
};
// Whether the scan's total of new vertices exceeds the caller's vertex capacity (given probabilities only).
__device__ __forceinline__ bool ids_overflow(const SampleArgs& a, const BatchDesc& b, int total) {
    return a.t != nullptr && b.counts[a.h - 1] + (int64_t)(uint32_t)total > b.ncap;
}
struct NewInKept {
    SampleArgs a; const BatchTable* t;
    // second launch of the scan: NewFin of this launch abandons the minibatch exactly when ids_overflow()
    __device__ int64_t n(int j, int total) const {
        return t->b[j].tinfo[2] || ids_overflow(a, t->b[j], total) ? 0 : t->b[j].counts[kE + a.h];
    }
    __device__ int operator()(int j, int64_t e) const { return t->b[j].src[a.h - 1][e] == -2 ? 1 : 0; }
};
struct NewOut {
    SampleArgs a; const BatchTable* t;
    __device__ void operator()(int j, int64_t e, int ex, int v, int total) const {
        if (!v || t->b[j].tinfo[2] || ids_overflow(a, t->b[j], total)) return;    // NewFin abandons the minibatch
        // A first appearance gets its local id here; the relabel pass fills in the repeats.
        const int64_t n_prev = t->b[j].counts[a.h - 1];
        const int64_t id = n_prev + (int64_t)(uint32_t)ex, cap = vertex_cap(t->b[j], a.N, a.h, a.t ? a.h : a.L);
        const int32_t gid = gids_of(a, j)[e];
        t->b[j].src[a.h - 1][e] = (int32_t)(id < cap ? id : cap - 1);
        if (id >= cap) return;                             // NewFin reports it
        t->b[j].S[id] = gid;
        // a vertex that will be a target of the next hop: its row is looked up here, once
        if (!a.t && a.h < a.L && id < a.node_stride) {
            const int64_t r0 = a.rowptr[gid];
            row0_of(a, j)[id] = r0;
            deg_of(a, j)[id] = (int32_t)(a.rowptr[gid + 1] - r0);
        }
    }
};
struct NewFin {
    SampleArgs a; const BatchTable* t;
    __device__ void operator()(int j, int total) const {
        int64_t* c = t->b[j].counts;
        if (a.t) *t->b[j].taken = 0ull;                    // the next hop counts from zero
        if (t->b[j].tinfo[2]) return;
        int64_t n = c[a.h - 1] + (int64_t)(uint32_t)total;
        if (ids_overflow(a, t->b[j], total)) {             // the new ids do not fit the caller's buffer
            t->b[j].tinfo[2] = 1;
            atomicOr(a.ovf, 1);
            c[kE + a.h] = 0;
            return;
        }
        const int64_t cap = vertex_cap(t->b[j], a.N, a.h, a.t ? a.h : a.L);
        if (n > cap) { atomicOr(a.bad, 4); n = cap; }
        c[a.h] = n;
        if (a.h == a.L) { atomicAdd(&a.totals[1], (unsigned long long)n); atomicAdd(&a.totals[0], 1ull); }
    }
};

// ---- step 5 ----
// A repeated id takes the index of the earlier vertex it resolved to, or the local id that the scan
// gave to its first appearance (an entry before it in the same list, final since the launch before).
__device__ __forceinline__ void relabel_rows(const SampleArgs& a, const BatchTable* __restrict__ t, int j, unsigned x,
                                             unsigned gx) {
    if (t->b[j].tinfo[2]) return;
    const int64_t e_h = t->b[j].counts[kE + a.h];
    const int64_t n_prev = t->b[j].counts[a.h - 1];
    const int32_t* __restrict__ flat = flat_of(a, j);
    int32_t* src = t->b[j].src[a.h - 1];
    const int64_t stride = (int64_t)gx * kBlock;
    for (int64_t e = (int64_t)x * kBlock + threadIdx.x; e < e_h; e += stride)
        if (src[e] < 0) {
            const int64_t fp = (uint32_t)flat[e];
            src[e] = fp < n_prev ? (int32_t)fp : src[fp - n_prev];
        }
}
__global__ void __launch_bounds__(kBlock) relabel_kernel(SampleArgs a, const BatchTable* __restrict__ t) {
    const BatchBlock bb = batch_block();
    relabel_rows(a, t, bb.j, bb.x, gridDim.x);
    // the call's last launch: nothing of this call touches the other set of flags
    if (a.h == a.L && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 2) a.bad_next[threadIdx.x] = 0;
}
// Stores a table of per-minibatch pointers in device memory, sixteen entries per launch (a launch's
// argument block holds 4 KB).  Only needed when a call brings buffers that no slot holds.
constexpr int kStoreChunk = 16;
struct BatchTableChunk { BatchDesc b[kStoreChunk]; };
__global__ void __launch_bounds__(kBlock) batch_table_store_kernel(BatchTableChunk src, BatchTable* dst, int first) {
    const uint64_t* s = reinterpret_cast<const uint64_t*>(&src);
    uint64_t* d = reinterpret_cast<uint64_t*>(&dst->b[first]);
    for (unsigned i = threadIdx.x; i < sizeof(BatchTableChunk) / sizeof(uint64_t); i += kBlock) d[i] = s[i];
}
__global__ void __launch_bounds__(kBlock) hop_fill_kernel(uint32_t* p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) p[i] = v;
}
// [0] error flag, [1] capacity flag of a call
__global__ void sample_flags_clear_kernel(int* bad) {
    if (threadIdx.x < 2) bad[threadIdx.x] = 0;
}
static_assert(sizeof(BatchTableChunk) % sizeof(uint64_t) == 0, "copied as 64-bit words");
static_assert(sizeof(BatchTableChunk) <= 4000, "must fit a launch's argument block");
static_assert(kMaxBatches % kStoreChunk == 0, "the table is stored in whole chunks");

}  // namespace spp

extern "C" int spp_mfg_bound(int32_t nseeds, const int32_t* fanouts, int32_t L, int64_t N,
                             int64_t* n_bound, int64_t* e_bound) {
    SPP_CHECK(fanouts && n_bound && e_bound, SPP_E_ARG, "spp_mfg_bound: null argument");
    SPP_CHECK(L >= 1 && L <= SPP_MAX_L && nseeds >= 0 && N > 0, SPP_E_ARG, "spp_mfg_bound: L = %d, nseeds = %d", L, nseeds);
    n_bound[0] = nseeds < N ? nseeds : N;
    e_bound[0] = 0;
    for (int h = 1; h <= L; ++h) {
        const int64_t f = fanouts[h - 1];
        SPP_CHECK(f >= 1 && f <= SPP_MAX_FANOUT, SPP_E_ARG, "spp_mfg_bound: fanout %lld of hop %d not in [1, %d]",
                  (long long)f, h, SPP_MAX_FANOUT);
        e_bound[h] = n_bound[h - 1] * f;
        const int64_t n = n_bound[h - 1] + e_bound[h];
        n_bound[h] = n < N ? n : N;
    }
    return SPP_OK;
}

// Most ids that hop h and S_{h-1} can have.
static int64_t hop_bound(const int64_t* nb, const int64_t* eb, int h, int64_t g_edges) {
    return nb[h - 1] + (eb[h] < g_edges ? eb[h] : g_edges);
}

// The launches of a fanout-sampling call: three per hop (a fourth where a hop's bound exceeds kHopLdsKeys ids) and one after the last (the call on hops of a few
// thousand edges takes 0.09 ms instead of 0.14 with six per hop).
// `g_edges`: edges of the graph, which a hop's distinct targets cannot exceed.
static void launch_hops(spp_ctx* ctx, spp::HopArgs a, int64_t g_edges, spp::BatchTable* dt, const spp::BatchDynAll& dyn, const int32_t* fanouts,
                        const int64_t* nb, const int64_t* eb, int max_seeds, size_t dedup_lds, hipStream_t st) {
    using namespace spp;
    // workgroups per minibatch: what the bound needs, eight per CU in the whole call at most (they take
    // several tiles then); multiples of 8: see batch_block()
    const int64_t share = std::max<int64_t>(8, (int64_t)ctx->num_cu * 8 / a.n_items);
    auto grid = [&](int64_t need) {
        const int64_t g = need < 1 ? 1 : (need < share ? need : share);
        return dim3((unsigned)((g + 7) & ~(int64_t)7), (unsigned)a.n_items);
    };
    const bool direct = max_seeds <= kDirectSeeds;
    unsigned long long* const tab = a.tab;
    for (int h = 1; h <= a.L; ++h) {
        a.tab = hop_bound(nb, eb, h, g_edges) > kHopLdsKeys ? tab : nullptr;
        a.h = h; a.f = fanouts[h - 1]; a.f_next = h < a.L ? fanouts[h] : 0;
        if (h == 1 && !direct) hop_seeds_kernel<<<grid((max_seeds + kHopTargets - 1) / kHopTargets), kBlock, 0, st>>>(a, dt, dyn);
        const int64_t tiles = std::max<int64_t>(std::min<int64_t>(1024 / a.n_items, nb[h - 1] / 16), nb[h - 1] / hop_tile_cap(a.f)) + 1;
        const int G = a.f <= 8 ? 8 : a.f <= 16 ? 16 : a.f <= 32 ? 32 : 64;
        auto sample = [&](auto seeds) {
            using Seeds = decltype(seeds);
            switch (G) {
                case 8:  hop_sample_kernel<8, Seeds><<<grid(tiles), kBlock, 0, st>>>(a, dt, seeds); break;
                case 16: hop_sample_kernel<16, Seeds><<<grid(tiles), kBlock, 0, st>>>(a, dt, seeds); break;
                case 32: hop_sample_kernel<32, Seeds><<<grid(tiles), kBlock, 0, st>>>(a, dt, seeds); break;
                default: hop_sample_kernel<64, Seeds><<<grid(tiles), kBlock, 0, st>>>(a, dt, seeds); break;
            }
        };
        if (h == 1 && direct) sample(SeedsArg{dyn}); else sample(NoSeedsArg{});
        // as many partitions as the bound has, four workgroups per CU in the whole call at most
        const int64_t parts = (int64_t)1 << hop_parts_log2(nb[h - 1], a.n_items, a.f);
        const int64_t most = std::max<int64_t>(1, (int64_t)ctx->num_cu * 4 / a.n_items);
        const dim3 dgrid((unsigned)a.n_items, (unsigned)std::min(parts, most)), ngrid = grid(std::min<int64_t>(tiles, kHopGranules));
        if (a.tab) {
            hop_dedup_kernel<true><<<dgrid, kDedupBlock, dedup_lds, st>>>(a, dt);
            hop_resolve_kernel<<<ngrid, kBlock, 0, st>>>(a, dt);
            hop_number_kernel<true><<<ngrid, kBlock, 0, st>>>(a, dt);
        } else {
            hop_dedup_kernel<false><<<dgrid, kDedupBlock, dedup_lds, st>>>(a, dt);
            hop_number_kernel<false><<<ngrid, kBlock, 0, st>>>(a, dt);
        }
    }
    hop_last_kernel<<<grid((eb[a.L] + kBlock - 1) / kBlock), kBlock, 0, st>>>(a, dt);
}

// Both samplers: sizes bounded by `fanouts`, or (d_t given) every entry of a row taken with its
// own probability and sizes checked against the caller's capacities on the device.
static int sample_batches(spp_ctx* ctx, const spp_graph* g, const spp_sample_item* items, int32_t n_items,
                          const int32_t* fanouts, const float* const* d_t, int32_t L, uint64_t seed, uint32_t flags) {
    using namespace spp;
    const bool general = d_t != nullptr;
    SPP_CHECK(ctx && g && (fanouts || general) && (items || n_items == 0), SPP_E_ARG, "spp_sample_mfg: null argument");
    SPP_CHECK(n_items >= 0 && n_items <= SPP_MAX_SAMPLE_BATCHES, SPP_E_ARG, "spp_sample_mfg: %d minibatches (at most %d)",
              n_items, SPP_MAX_SAMPLE_BATCHES);
    SPP_CHECK(L >= 1 && L <= SPP_MAX_L, SPP_E_ARG, "spp_sample_mfg: L = %d not in [1, %d]", L, SPP_MAX_L);
    if (general)
        for (int h = 0; h < L; ++h)
            SPP_CHECK(d_t[h] || g->M == 0, SPP_E_ARG, "spp_sample_mfg_general: no transition probabilities for hop %d", h + 1);
    if (n_items == 0) return SPP_OK;
    BatchTable ht = {};             // what stays the same while the caller reuses its buffers
    BatchDynAll dyn = {};           // what every call brings
    int64_t nb[SPP_MAX_L + 1] = {0}, eb[SPP_MAX_L + 1] = {0};       // bounds (capacities) of the largest minibatch
    int max_seeds = 0;
    for (int j = 0; j < n_items; ++j) {
        const spp_sample_item& it = items[j];
        spp_mfg* io = it.io;
        SPP_CHECK(io, SPP_E_ARG, "spp_sample_mfg: minibatch %d has no output struct", j);
        SPP_CHECK(it.nseeds >= 0 && (it.d_seeds || it.nseeds == 0), SPP_E_ARG, "spp_sample_mfg: seeds of minibatch %d", j);
        SPP_CHECK(it.nseeds <= g->N, SPP_E_ARG, "spp_sample_mfg: more seeds than vertices");
        SPP_CHECK(io->d_node_ids && io->d_counts, SPP_E_ARG, "spp_sample_mfg: null output buffer");
        int64_t nbj[SPP_MAX_L + 1], ebj[SPP_MAX_L + 1];
        if (general) {
            // no fanout bounds the sizes: the capacities are the bounds, enforced on the device
            SPP_CHECK(io->n_nodes_cap >= it.nseeds && io->n_nodes_cap >= 1, SPP_E_CAPACITY,
                      "spp_sample_mfg_general: d_node_ids holds %lld entries, the minibatch has %d seeds",
                      (long long)io->n_nodes_cap, it.nseeds);
            ebj[0] = 0;
            for (int h = 0; h <= L; ++h) nbj[h] = io->n_nodes_cap;
            for (int h = 1; h <= L; ++h) {
                SPP_CHECK(io->n_edges_cap[h - 1] >= 0, SPP_E_ARG, "spp_sample_mfg_general: negative capacity of hop %d", h);
                ebj[h] = io->n_edges_cap[h - 1];
            }
        } else {
            SPP_TRY(spp_mfg_bound(it.nseeds, fanouts, L, g->N, nbj, ebj));
            SPP_CHECK(io->n_nodes_cap >= nbj[L] && io->n_nodes_cap >= 1, SPP_E_CAPACITY,
                      "spp_sample_mfg: d_node_ids holds %lld entries, the bound is %lld", (long long)io->n_nodes_cap, (long long)nbj[L]);
        }
        ht.b[j].ncap = io->n_nodes_cap;
        for (int h = 1; h <= L; ++h) {
            SPP_CHECK(io->d_indptr[h - 1] && io->d_src[h - 1], SPP_E_ARG, "spp_sample_mfg: null buffer of hop %d", h);
            SPP_CHECK(io->n_edges_cap[h - 1] >= ebj[h], SPP_E_CAPACITY,
                      "spp_sample_mfg: d_src of hop %d holds %lld entries, the bound is %lld", h,
                      (long long)io->n_edges_cap[h - 1], (long long)ebj[h]);
            SPP_CHECK(ebj[h] < 0x3FFFFFFFll && nbj[h] + ebj[h] < 0x3FFFFFFFll, SPP_E_ARG, "spp_sample_mfg: hop %d exceeds 30-bit sizes", h);
            ht.b[j].indptr[h - 1] = io->d_indptr[h - 1];
            ht.b[j].src[h - 1] = io->d_src[h - 1];
            ht.b[j].ecap[h - 1] = io->n_edges_cap[h - 1];
        }
        for (int h = 0; h <= L; ++h) { if (nbj[h] > nb[h]) nb[h] = nbj[h]; if (ebj[h] > eb[h]) eb[h] = ebj[h]; }
        dyn.d[j].seeds = it.d_seeds; dyn.d[j].nseeds = it.nseeds; dyn.d[j].batch_lo = (uint32_t)it.batch_index;
        ht.b[j].S = io->d_node_ids; ht.b[j].counts = io->d_counts;
        if (it.nseeds > max_seeds) max_seeds = it.nseeds;
    }
    int64_t emax = 1;
    for (int h = 1; h <= L; ++h) if (eb[h] > emax) emax = eb[h];
    SPP_HIP(hipSetDevice(ctx->device));
    hipStream_t st = ctx->stream;

    // Fanout sampling deduplicates in LDS (hop_* kernels).  Its workspace grows with the edge bounds, the id
    // table of the other form with the vertex bounds: where wide fanouts on a small graph make the first by
    // far the larger one, the call keeps the table, so that what fitted a GPU's memory still does.
    int64_t ent_stride = 0, seg_stride = 0;
    for (int h = 1; h <= L && !general; ++h) {
        const int64_t ents = eb[h] + nb[h - 1];
        const int64_t tiles = std::max<int64_t>(1024 / n_items, nb[h - 1] / hop_tile_cap(fanouts[h - 1])) + 2;
        const int64_t segs = std::min(tiles, nb[h - 1] / 16 + 2) << hop_parts_log2(nb[h - 1], n_items, fanouts[h - 1]);
        if (ents > ent_stride) ent_stride = ents;
        if (segs > seg_stride) seg_stride = segs;
    }
    // table region per minibatch: twice the most keys a hop can hold (all ids so far plus the hop's entries)
    const int64_t max_keys = general ? nb[L] + emax : nb[L];
    const uint32_t cap = next_pow2((uint64_t)(2 * max_keys > 1024 ? 2 * max_keys : 1024));
    const size_t hop_bytes = (size_t)n_items * (size_t)(ent_stride * 8 + seg_stride * 4);
    const size_t tab_bytes = (size_t)n_items * ((size_t)cap * 8 + (size_t)emax * 8);
    const bool in_lds = !general && !(flags & SPP_SAMPLE_GLOBAL_TABLE) && hop_bytes <= tab_bytes + ((size_t)1 << 30);
    // workgroups per minibatch in the scans and the table clear: the whole call gets about 4 per CU
    const int per_batch = (ctx->num_cu * 4 + n_items - 1) / n_items;
    const int scan_grid = ((per_batch < 32 ? 32 : per_batch) + 7) & ~7;     // multiples of 8: see batch_block()
    if (in_lds) {
        SPP_TRY(ctx->table.reserve((size_t)ent_stride * sizeof(uint64_t) * n_items));
        SPP_TRY(ctx->flat.reserve((size_t)seg_stride * sizeof(uint32_t) * n_items));
    } else {
        SPP_TRY(ctx->table.reserve((size_t)cap * sizeof(uint64_t) * n_items));
        SPP_TRY(ctx->flat.reserve((size_t)emax * sizeof(int32_t) * n_items * 2));        // what the ids resolve to, and the ids
    }
    SPP_TRY(ctx->slots.reserve((size_t)(4 * sizeof(uint32_t) + sizeof(unsigned long long)) * kMaxBatches + 64 +
                               (general ? (size_t)nb[L] * sizeof(int32_t) * n_items : 0)));
    unsigned long long* taken = ctx->slots.as<unsigned long long>();
    uint32_t* tinfo = reinterpret_cast<uint32_t*>(taken + kMaxBatches);
    for (int j = 0; j < n_items; ++j) {
        ht.b[j].tinfo = tinfo + 4 * j;
        ht.b[j].taken = general ? taken + j : nullptr;
    }
    SPP_TRY(ctx->partials.reserve((size_t)scan_grid * n_items * sizeof(int) + 64));
    int* partial = ctx->partials.as<int>();
    // The table of per-minibatch pointers is too large to ride in the argument block of every kernel, so it
    // lives in device memory: in one of a few slots, found again by content when a later call brings the same
    // buffers (then nothing is stored), else stored over the slot used longest ago.
    constexpr int kSlots = spp_ctx::kBatchSlots;
    if (!ctx->btab.ptr) {
        SPP_TRY(ctx->btab.reserve(kSlots * sizeof(BatchTable) + 256));
        for (int k = 0; k < kSlots; ++k) ctx->btab_n[k] = 0;
        ctx->sample_flags_clean = 0;
    }
    if (!ctx->btab_mirror) {
        ctx->btab_mirror = calloc(kSlots, sizeof(BatchTable));
        SPP_CHECK(ctx->btab_mirror, SPP_E_OOM, "spp_sample_mfg: out of host memory");
    }
    BatchTable* mirror = static_cast<BatchTable*>(ctx->btab_mirror);
    int slot = -1;
    for (int k = 0; k < kSlots && slot < 0; ++k)
        if (ctx->btab_n[k] == n_items && memcmp(&mirror[k], &ht, (size_t)n_items * sizeof(BatchDesc)) == 0) slot = k;
    const bool stored = slot >= 0;
    if (!stored) {
        slot = 0;
        for (int k = 1; k < kSlots; ++k)
            if (ctx->btab_stamp[k] < ctx->btab_stamp[slot]) slot = k;
        ctx->btab_n[slot] = 0;          // until its launches are enqueued
    }
    ctx->btab_stamp[slot] = ++ctx->sample_calls;
    BatchTable* dt = ctx->btab.as<BatchTable>() + slot;
    // two sets of flags, used alternately: this call's were cleared by the last kernel of the call before
    int* flags2 = reinterpret_cast<int*>(ctx->btab.as<BatchTable>() + kSlots);
    int* d_bad = flags2 + 2 * (ctx->sample_calls & 1);
    int* d_bad_next = flags2 + 2 * ((ctx->sample_calls + 1) & 1);
    const bool flags_clean = ctx->sample_flags_clean != 0;
    ctx->sample_flags_clean = 0;        // set again once this call's last kernel is enqueued

    SampleArgs a;
    a.rowptr = g->rowptr; a.col = g->col; a.N = g->N;
    a.tab = ctx->table.as<unsigned long long>(); a.cap = cap;
    a.flat = ctx->flat.as<int32_t>(); a.flat_stride = emax;
    a.gids = a.flat + (size_t)emax * n_items;
    // row start and length of every vertex that can be a target: the members of S_{L-1}
    a.node_stride = general ? 0 : nb[L - 1];
    SPP_TRY(ctx->nodeinfo.reserve((size_t)a.node_stride * n_items * (sizeof(int64_t) + sizeof(int32_t)) + 64));
    a.row0 = ctx->nodeinfo.as<int64_t>();
    a.deg = reinterpret_cast<int32_t*>(a.row0 + (size_t)a.node_stride * n_items);
    constexpr size_t dedup_lds = sizeof(uint32_t) * (2 * kHopSlots + kHopGranules + 2 * kDedupBlock + kDedupBlock / kWave);
    HopArgs ha;
    if (in_lds) {
        if (!ctx->dedup_lds_set) {
            for (const void* k : {reinterpret_cast<const void*>(&hop_dedup_kernel<false>), reinterpret_cast<const void*>(&hop_dedup_kernel<true>)})
                SPP_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dedup_lds));
            ctx->dedup_lds_set = 1;
        }
        ha.rowptr = g->rowptr; ha.col = g->col; ha.N = g->N;
        ha.ent = ctx->table.as<uint64_t>(); ha.ent_stride = ent_stride;
        ha.seg = ctx->flat.as<uint32_t>(); ha.seg_stride = seg_stride;
        ha.row0 = a.row0; ha.deg = a.deg; ha.node_stride = a.node_stride;
        ha.csum_stride = nb[L - 1] / kHopTargets + 2;
        const size_t sum_words = (size_t)n_items * (2 * (size_t)ha.csum_stride + kHopGranules);
        if (ctx->hopsums.bytes < sum_words * sizeof(uint32_t)) ctx->hopsums_clean = 0;
        SPP_TRY(ctx->hopsums.reserve(sum_words * sizeof(uint32_t)));
        ha.csum = ctx->hopsums.as<uint32_t>();
        ha.fsum = ha.csum + 2 * (size_t)ha.csum_stride * n_items;
        ha.totals = reinterpret_cast<unsigned long long*>(ctx->totals); ha.bad = d_bad; ha.bad_next = d_bad_next;
        ha.mirror = (flags & SPP_SYNC) ? ctx->h_pinned + 64 : nullptr;       // kMaxBatches x 18 counts, then the flags
        ha.n_items = n_items; ha.L = L; ha.seed = seed;
        // The table of the hops above kHopLdsKeys ids, where a bound allows one: as large as the other form's.  Without the
        // memory for it such hops take their partitions in parts.
        ha.tab = nullptr; ha.tab_cap = cap;
        bool wide = false;
        for (int h = 1; h <= L; ++h) wide = wide || hop_bound(nb, eb, h, g->M) > kHopLdsKeys;
        if (wide) {
            const size_t bytes = (size_t)cap * sizeof(uint64_t) * n_items;
            if (ctx->hoptab.bytes < bytes) ctx->hoptab_clean = 0;
            if (ctx->hoptab.reserve(bytes) == SPP_OK) ha.tab = ctx->hoptab.as<unsigned long long>();
            else (void)hipGetLastError();
        }
    }
    a.totals = reinterpret_cast<unsigned long long*>(ctx->totals); a.bad = d_bad; a.ovf = d_bad + 1; a.bad_next = d_bad_next;
    a.L = L; a.h = 0; a.f = 0; a.seed = seed;
    a.t = nullptr;
    a.cnt = reinterpret_cast<int32_t*>(tinfo + 4 * kMaxBatches + 16); a.cnt_stride = nb[L];

    auto capped = [&](int64_t need, int64_t lim) {
        const int64_t g = need < 1 ? 1 : (need < lim ? need : lim);
        return (unsigned)((g + 7) & ~(int64_t)7);
    };
    const int64_t share = (int64_t)ctx->num_cu * 64 / n_items + 1;    // workgroups per minibatch in the wide kernels
    {
        ScopedTimer tt(ctx, SPP_T_SAMPLE, st);
        if (!flags_clean) sample_flags_clear_kernel<<<1, 64, 0, st>>>(d_bad);
        if (!stored) {
            for (int first = 0; first < n_items; first += kStoreChunk) {
                BatchTableChunk chunk;
                memcpy(&chunk, &ht.b[first], sizeof(chunk));
                batch_table_store_kernel<<<1, kBlock, 0, st>>>(chunk, dt, first);
            }
            memcpy(&mirror[slot], &ht, sizeof(BatchTable));
        }
        if (in_lds) {
            if (!ctx->hopsums_clean)
                hop_fill_kernel<<<ctx->num_cu, kBlock, 0, st>>>(ctx->hopsums.as<uint32_t>(), (int64_t)(ctx->hopsums.bytes / sizeof(uint32_t)), 0u);
            if (ha.tab && !ctx->hoptab_clean)
                hop_fill_kernel<<<ctx->num_cu * 8, kBlock, 0, st>>>(ctx->hoptab.as<uint32_t>(), (int64_t)(ctx->hoptab.bytes / sizeof(uint32_t)), ~0u);
            ctx->hopsums_clean = 0;         // set again once this call's last kernel is enqueued
            if (ha.tab) ctx->hoptab_clean = 0;
            launch_hops(ctx, ha, g->M, dt, dyn, fanouts, nb, eb, max_seeds, dedup_lds, st);
        } else {
            seeds_kernel<<<dim3(capped((max_seeds + kBlock - 1) / kBlock, 1 << 20), n_items), kBlock, 0, st>>>(a, dt, dyn);
        }
        for (int h = 1; h <= L && !in_lds; ++h) {
            a.h = h; a.f = general ? 0 : fanouts[h - 1]; a.t = general ? d_t[h - 1] : nullptr;
            const dim3 wgrid(capped((nb[h - 1] * kWave + kBlock - 1) / kBlock, share), n_items);   // a wavefront per target
            if (general) general_count_kernel<<<wgrid, kBlock, 0, st>>>(a, dt);
            // the emptying of this hop's table rides in the scan's second launch
            grid_scan_batched(st, scan_grid, n_items, CountIn{a, dt}, CountOut{a, dt}, CountFin{a, dt}, partial, TableClear{a, dt});
            if (general) {
                general_sample_kernel<<<wgrid, kBlock, 0, st>>>(a, dt);
            } else {
                const int G = a.f <= 8 ? 8 : a.f <= 16 ? 16 : a.f <= 32 ? 32 : 64;
                const dim3 sgrid(capped((nb[h - 1] * G + kBlock - 1) / kBlock, share), n_items);
                switch (G) {
                    case 8:  sample_kernel<8><<<sgrid, kBlock, 0, st>>>(a, dt); break;
                    case 16: sample_kernel<16><<<sgrid, kBlock, 0, st>>>(a, dt); break;
                    case 32: sample_kernel<32><<<sgrid, kBlock, 0, st>>>(a, dt); break;
                    default: sample_kernel<64><<<sgrid, kBlock, 0, st>>>(a, dt); break;
                }
            }
            grid_scan_batched_two(st, scan_grid, n_items, NewIn{a, dt}, NewInKept{a, dt}, NewOut{a, dt}, NewFin{a, dt}, partial);
            relabel_kernel<<<dim3(capped((eb[h] + kBlock - 1) / kBlock, share), n_items), kBlock, 0, st>>>(a, dt);
        }
    }
    SPP_HIP(hipGetLastError());
    // what the launches leave behind for the next call, now that all of them have been accepted
    ctx->btab_n[slot] = n_items;
    ctx->sample_flags_clean = 1;
    if (in_lds) ctx->hopsums_clean = 1;
    if (in_lds && ha.tab) ctx->hoptab_clean = 1;
    if (flags & SPP_SYNC) {
        int64_t* hp = ctx->h_pinned + 64;            // kMaxBatches x 18 counts, then the flags
        if (!in_lds) {                               // else the last hop's numbering has stored them there
            for (int j = 0; j < n_items; ++j)
                SPP_HIP(hipMemcpyAsync(hp + j * 2 * kE, items[j].io->d_counts, 2 * kE * sizeof(int64_t), hipMemcpyDeviceToHost, st));
            SPP_HIP(hipMemcpyAsync(hp + kMaxBatches * 2 * kE, d_bad, 2 * sizeof(int), hipMemcpyDeviceToHost, st));
        }
        SPP_HIP(hipStreamSynchronize(st));
        for (int j = 0; j < n_items; ++j)
            for (int k = 0; k <= SPP_MAX_L; ++k) {
                items[j].io->n[k] = hp[j * 2 * kE + k];
                items[j].io->e[k] = hp[j * 2 * kE + kE + k];
            }
        int* fl = reinterpret_cast<int*>(hp + kMaxBatches * 2 * kE);
        for (int j = 0; in_lds && j < n_items; ++j) fl[0] |= fl[2 + j];
        SPP_CHECK((fl[0] & 1) == 0, SPP_E_ARG, "spp_sample_mfg: a seed lies outside [0, N)");
        SPP_CHECK((fl[0] & 4) == 0, SPP_E_ARG, "spp_sample_mfg: a minibatch reached more vertices than its bound: its seeds are not distinct");
        SPP_CHECK((fl[0] & 2) == 0, SPP_E_ARG, "spp_sample_mfg_general: a transition probability lies outside [0, 1]; it was taken as 0");
        SPP_CHECK(fl[1] == 0, SPP_E_CAPACITY, "spp_sample_mfg_general: a minibatch exceeded the capacity of its buffers and was abandoned");
    }
    return SPP_OK;
}

extern "C" int spp_sample_mfg_multi(spp_ctx* ctx, const spp_graph* g, const spp_sample_item* items, int32_t n_items,
                                    const int32_t* fanouts, int32_t L, uint64_t seed, uint32_t flags) {
    SPP_CHECK(fanouts, SPP_E_ARG, "spp_sample_mfg: null argument");
    return sample_batches(ctx, g, items, n_items, fanouts, nullptr, L, seed, flags);
}

extern "C" int spp_sample_mfg_general(spp_ctx* ctx, const spp_graph* g, const float* const* d_t,
                                      const spp_sample_item* items, int32_t n_items, int32_t L, uint64_t seed,
                                      uint32_t flags) {
    SPP_CHECK(d_t, SPP_E_ARG, "spp_sample_mfg_general: null argument");
    return sample_batches(ctx, g, items, n_items, nullptr, d_t, L, seed, flags);
}

extern "C" int spp_sample_mfg(spp_ctx* ctx, const spp_graph* g, const int32_t* d_seeds, int32_t nseeds,
                              const int32_t* fanouts, int32_t L, uint64_t seed, uint64_t batch_index,
                              spp_mfg* io, uint32_t flags) {
    SPP_CHECK(io, SPP_E_ARG, "spp_sample_mfg: null argument");
    spp_sample_item one;
    one.d_seeds = d_seeds; one.nseeds = nseeds; one.batch_index = batch_index; one.io = io;
    return spp_sample_mfg_multi(ctx, g, &one, 1, fanouts, L, seed, flags);
}
