// Graph handle: wraps the caller's CSR and, on request, builds the transposed structure that the
// pull form of Proposition 1, eq. (2), walks, in one of two layouts.
//   Row blocks (graphs up to 2^23 vertices, whose per-vertex vector y stays in the caches): the edges
//   v -> u grouped by blocks of 2^14 destination rows u and, inside a block, sorted by source v,
//   4 bytes per edge (the low 18 bits of the source and the row inside the block; a table says where
//   each run of 2^18 sources starts in each block).
//   Chunked (larger graphs): the edges sorted by (chunk of 2^15 sources, row block, source), every
//   (chunk, row block) piece padded to a multiple of four entries, 2 + 2 bytes per entry (source
//   inside the chunk, row inside the block), with tables for both walks: where every chunk starts,
//   and per row block where each chunk's piece lies and how many vectors precede it.
// The row blocks are one stable partition of the CSR's edges by the block of their destination: the CSR
// is sorted by source already.  The chunked layout is built by a radix sort of packed edge keys.  Either
// is built once per graph, then read back and compared with the edges of the CSR before anything walks it.
#include "spp_common.h"
#include "spp_device.h"

#include <stddef.h>

#include <new>
#include <type_traits>

namespace spp {

// Every kernel of the library indexes with these arrays, so they are checked once here: offsets
// monotone inside [0, M], column ids inside [0, N).  Nothing is read of col[] unless the CSR says that it has M entries.
struct CsrFound { int64_t first, last, bad; };   // rowptr[0], rowptr[N], whether something is wrong (zero before)
__device__ __forceinline__ bool csr_ends(int64_t N, int64_t M, const int64_t* __restrict__ rowptr, CsrFound* __restrict__ found) {
    const int64_t first = rowptr[0], last = rowptr[N];
    if (blockIdx.x == 0 && threadIdx.x == 0) { found->first = first; found->last = last; }
    return first == 0 && last == M;
}
__global__ void __launch_bounds__(kBlock) validate_csr_kernel(int64_t N, int64_t M, const int64_t* __restrict__ rowptr,
                                                              const int32_t* __restrict__ col, CsrFound* __restrict__ found) {
    if (!csr_ends(N, M, rowptr, found)) return;
    int64_t* __restrict__ bad = &found->bad;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    for (int64_t v = t; v < N; v += stride) {
        const int64_t b = rowptr[v], e = rowptr[v + 1];
        if (b < 0 || e > M || b > e) *bad = 1;
    }
    for (int64_t i = t; i < M; i += stride) {
        const int32_t u = col[i];
        if (u < 0 || u >= N) *bad = 1;
    }
}

__global__ void fill_i64_kernel(int64_t* p, int64_t n, int64_t v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// ---- the row-block layout ----------------------------------------------------------------------
// A workgroup takes tiles of 4096 consecutive edges; a wavefront walks its sixteenth of a tile 64 edges at
// a time and ranks them among those of the same block with ballots over the block's bits, which keeps
// the edges of a block in CSR order, that is sorted by source.  One counting pass, one scan of the
// (block, tile) counts, one pass that places a tile's edge words in LDS by block and writes them as
// runs.  (A radix sort of 64-bit keys (block, source, row) took four passes over 16 bytes per edge, and
// 16 bytes per edge of temporary memory whose allocation cost more than the sort.)  2.4M vertices, 121M
// edges: the kernels of a build 9.2 -> 0.81 ms: 0.35 in the placing pass, most of it vector instructions,
// 0.11 in the counting pass, 0.15 in the read-back and 0.175 in the sum over the CSR that it is compared with.
constexpr int kPartBlock = 1024;
constexpr int kPartWaves = kPartBlock / kWave;
constexpr int kPartPer = kPartTile / kPartBlock;         // 64-edge batches per wavefront
constexpr int kPartRows = 4;                             // most rows that begin among 64 edges to be looked at one by one
constexpr int kPartMaxBlocks = 512;                      // 2^23 vertices in blocks of 2^14 rows

__device__ __forceinline__ void add_mix(unsigned long long mine, unsigned long long* sum) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_down(mine, off, kWave);
    if (lane_id() == 0 && mine) atomicAdd(sum, mine);
}

// The passes that build the row blocks validate the CSR on the way: this one its offsets, the counting pass its ids, each
// before it uses them; the passes after those two do nothing if either found something wrong.  (A pass of its own cost a
// build of 121M edges 141 us.)
__device__ __forceinline__ bool csr_bad(const CsrFound* found, int64_t M) { return found->first != 0 || found->last != M || found->bad != 0; }

// tile_row[t] = the vertex whose row holds the first edge of tile t; tile_row[ntiles] = the last one with edges.
__global__ void __launch_bounds__(kBlock) part_rows_kernel(int64_t N, int64_t M, int64_t ntiles, const int64_t* __restrict__ rowptr,
                                                           int32_t* __restrict__ tile_row, CsrFound* __restrict__ found) {
    if (!csr_ends(N, M, rowptr, found)) return;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x; v < N; v += stride) {
        const int64_t b = rowptr[v], e = rowptr[v + 1];
        if (b < 0 || e > M || b > e) { found->bad = 1; continue; }
        for (int64_t t = (b + kPartTile - 1) / kPartTile; t * kPartTile < e; ++t) tile_row[t] = (int32_t)v;
        if (b < e && e == M) tile_row[ntiles] = (int32_t)v;
    }
}

// hist[block * ntiles + tile] = edges of the tile that end in the block.
__global__ void __launch_bounds__(kPartBlock) part_count_kernel(int64_t N, int64_t M, const int64_t* __restrict__ rowptr,
                                                                const int32_t* __restrict__ col, int rbits,
                                                                int nrb, int64_t ntiles,
                                                                uint32_t* __restrict__ hist, CsrFound* __restrict__ found) {
    if (rowptr[0] != 0 || rowptr[N] != M) return;        // then col[] need not hold M ids
    bool wrong = false;
    constexpr int kCopies = 8;                   // a lane adds to one of eight copies: most edges of a tile end in few blocks
    __shared__ uint32_t cnt[kPartMaxBlocks][kCopies];
    uint32_t u[kPartPer], next[kPartPer];        // the next tile's ids are asked for before this one's are counted
    auto load = [&](uint32_t (&v)[kPartPer], int64_t tile) {
#pragma unroll
        for (int k = 0; k < kPartPer; ++k) {
            const int64_t e = tile * kPartTile + threadIdx.x + k * kPartBlock;
            v[k] = (uint32_t)__builtin_nontemporal_load(col + (e < M ? e : M - 1));
        }
    };
    load(u, blockIdx.x);
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        for (int i = threadIdx.x; i < nrb * kCopies; i += kPartBlock) (&cnt[0][0])[i] = 0u;
        const int64_t e0 = tile * kPartTile + threadIdx.x;
        load(next, tile + gridDim.x);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPartPer; ++k)
            if (e0 + k * kPartBlock < M) {
                if (u[k] < (uint32_t)N) atomicAdd(&cnt[u[k] >> rbits][threadIdx.x & (kCopies - 1)], 1u);
                else wrong = true;
            }
        __syncthreads();
        if ((int)threadIdx.x < nrb) {
            uint32_t c = 0;
#pragma unroll
            for (int w = 0; w < kCopies; ++w) c += cnt[threadIdx.x][w];
            hist[(int64_t)threadIdx.x * ntiles + tile] = c;
        }
#pragma unroll
        for (int k = 0; k < kPartPer; ++k) u[k] = next[k];
        __syncthreads();
    }
    if (wrong) found->bad = 1;
}

// Places a tile's edge words by block, in CSR order, and stores them as runs.  How many edges of each block the tile has follows
// from the offsets, so that the blocks' places in the tile are known before an edge is looked at; left to find are an
// edge's source (the rows leave their numbers at their first edges; an edge takes the last one before it among its 64, or the
// last row to start in the 64s before) and its rank among its wavefront's edges of the block.  Four barriers per tile: (1) sources
// and ranks; (2) per block, the wavefronts' places; (3) the words; (4) they are stored while the next tile's rows are marked.  All
// loads of a tile are asked for before the stores of the tile before, unconditionally: a load that is waited for after stores waits
// for those too.
// 2.4M vertices, 121M edges: 352 us, 1.04 GB.  It took 554: a lane wrote a long row's number at every 64th of its edges one
// by one and the first wavefront scanned the blocks' counts by shuffles (half of a tile's time, the other wavefronts waiting), values
// kept over the loop went to memory and back (see here()), and a ballot's bit cost six instructions (four: 427 -> 368).  What
// bounds it now: the ranks' vector instructions, a third of the time, and the four barriers.  (Ranks by LDS atomics, row by row
// as the lanes of one row may come in any order: 513, they wait for each other.)
struct PlaceLds {
    uint32_t words[kPartTile];           // the tile's words by block
    uint16_t blk_of[kPartTile];
    uint32_t mark[2][kPartTile];         // per edge: the row that starts there, less the tile's first
    uint32_t last[2][kPartTile / kWave]; // per 64 edges: the last row that starts among them, less the tile's first, plus one
    uint32_t num[kPartMaxBlocks], off[kPartMaxBlocks];        // of the next tile: edges per block and where they go
    uint32_t start[kPartMaxBlocks];      // where a block's words start among the tile's
    uint32_t shift[2][kPartMaxBlocks];   // where they go in t_edge, less that
    uint4    cnt[1];                     // per block 16 numbers of 16 bits: edges, then first place, per wavefront
};
template <int BITS>
__global__ void __launch_bounds__(kPartBlock, 8) part_place_kernel(int64_t N, int64_t M, const int64_t* __restrict__ rowptr,
                                                                const int32_t* __restrict__ col, int rbits,
                                                                int nrb, int ntiles, const int32_t* __restrict__ tile_row,
                                                                const uint32_t* __restrict__ offs,
                                                                uint32_t* __restrict__ t_edge, const CsrFound* __restrict__ found) {
    extern __shared__ __align__(16) char place_lds[];
    if (csr_bad(found, M)) return;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    PlaceLds& l = *reinterpret_cast<PlaceLds*>(place_lds);
    uint16_t* cnt = reinterpret_cast<uint16_t*>(l.cnt);
    static_assert(kPartWaves == 16, "a block's counts are two 128-bit words");
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    const int lane = lane_id();
    const uint32_t tid = threadIdx.x, wave = tid >> 6, rmask = (1u << rbits) - 1u;
    const uint32_t wave_u = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave);
    const uint32_t we0 = wave * (kPartTile / kPartWaves) + lane;
    const uint32_t off0 = ((int)tid < nrb ? tid : 0u) * (uint32_t)ntiles;      // below 2^30
    const uint32_t* __restrict__ row32 = reinterpret_cast<const uint32_t*>(rowptr);      // the lower halves: offsets are below 2^32, like M
    // a tile's rows (the first kPartBlock of them, one per thread; threads beyond take the last one once more) and offsets
    struct { int32_t v0, v1; uint32_t b, e, off, off_n; } r;
    auto load_row = [&](uint32_t v) { r.b = row32[2u * v]; r.e = row32[2u * v + 2u]; };
    // where a tile's rows begin and end, in even and odd lanes, is asked for a tile before they are: by a vector load, as a scalar
    // one is waited for at the next read of LDS
    int32_t ends;
    auto load_ends = [&](int tile) { ends = tile_row[tile + (lane & 1)]; };
    auto load_rows = [&](int tile) {
        r.v0 = __builtin_amdgcn_readlane(ends, 0); r.v1 = __builtin_amdgcn_readlane(ends, 1);
        load_row((uint32_t)(r.v1 - r.v0 > (int32_t)tid ? r.v0 + (int32_t)tid : r.v1));
        const uint32_t at = off0 + (uint32_t)tile;
        r.off = offs[at];
        r.off_n = offs[at + 1u];                 // behind the last one stands M
    };
    uint32_t u[kPartPer];
    auto load_edges = [&](int tile) {            // of a full tile
        const int32_t* __restrict__ c = col + (int64_t)tile * kPartTile;
#pragma unroll
        for (int k = 0; k < kPartPer; ++k) u[k] = (uint32_t)__builtin_nontemporal_load(c + (we0 + k * kWave));
    };
    auto mark_rows = [&](int tile, uint32_t n, uint32_t* mark, uint32_t* last) {
        const uint32_t base = (uint32_t)tile * (uint32_t)kPartTile, stop = base + n;       // at most M
        auto one = [&](int32_t v) {
            const uint32_t b = (r.b > base ? (r.b < stop ? r.b : stop) : base) - base, e = (r.e > base ? (r.e < stop ? r.e : stop) : base) - base;
            if (b < e) {
                mark[b] = (uint32_t)(v - r.v0);
                atomicMax(&last[b / kWave], (uint32_t)(v - r.v0) + 1u);
            }
        };
        if (r.v1 - r.v0 > kTileManyRows) {       // the same for all threads
#pragma unroll 1
            for (int k = 0; k < kPartPer; ++k)
                if (we0 + k * kWave < n) mark[we0 + k * kWave] = (uint32_t)(row_of_edge(rowptr, r.v0, r.v1, base + we0 + k * kWave) - r.v0);
            return;
        }
        if (r.v1 - r.v0 >= (int32_t)tid) one(r.v0 + (int32_t)tid);
        for (int64_t v = (int64_t)r.v0 + kPartBlock + tid; v <= r.v1; v += kPartBlock) { load_row((uint32_t)v); one((int32_t)v); }
    };
    auto clear_marks = [&](uint32_t* mark, uint32_t* last) {
        const uint32_t none = here(kNone);
        reinterpret_cast<u32x4*>(mark)[here(tid)] = u32x4{none, none, none, none};
        if (tid < kPartTile / kWave) last[tid] = 0u;
    };
    auto clear_counts = [&]() { const uint32_t z = here(0u); for (int i = here(tid); i < 2 * nrb; i += kPartBlock) l.cnt[i] = uint4{z, z, z, z}; };
    auto keep_offsets = [&]() { if ((int)tid < nrb) { l.num[tid] = r.off_n - r.off; l.off[tid] = r.off; } };
    auto set_starts = [&](uint32_t* shift) {     // 64 blocks to a wavefront, from the third on: the first ones have the rows to mark,
                                                 // the last ones are the last to get through what all do
        const int b0 = ((int)wave_u - 2) * kWave, b = b0 + lane;
        if (b0 < 0 || b0 >= nrb) return;
        uint32_t before = 0;
        for (int q = lane; q < b0; q += kWave) before += l.num[q];
        const uint32_t c = b < nrb ? l.num[b] : 0u, inc = (uint32_t)wave_inclusive_scan((int)c), st = (uint32_t)wave_sum((int)before) + inc - c;
        if (b < nrb) { l.start[b] = st; shift[b] = l.off[b] - st; }
    };
    uint32_t place[kPartPer];                    // block << 16 | rank among the wavefront's edges of the block
    auto rank = [&](const uint32_t* mark, const uint32_t* last, int32_t v0, auto full, uint32_t n) {
        // the row that an edge of a 64 lies in, if none starts at or before it there: the last one to start in those before
        const uint32_t rows_before = wave_inclusive_max(last[lane]);
#pragma unroll
        for (int k = 0; k < kPartPer; ++k) {
            const uint32_t e = here(we0) + k * kWave;
            const bool has = full || e < n;
            const uint32_t m = mark[e];
            const uint64_t starts = __ballot(m != kNone);
            const int batch = (int)(wave_u * kPartPer) + k;      // the first edge of a tile is marked
            uint32_t src = (uint32_t)__builtin_amdgcn_readlane((int)rows_before, batch > 0 ? batch - 1 : 0) - 1u;
            if (__popcll(starts) <= kPartRows) { // one after the other: two instructions each, where looking back takes eleven
                for (uint64_t rest = starts; rest; rest &= rest - 1) {
                    const int at = __builtin_ctzll(rest);
                    src = __builtin_amdgcn_inverse_ballot_w64(~0ull << at) ? (uint32_t)__builtin_amdgcn_readlane((int)m, at) : src;
                }
            } else {
                const uint64_t upto = starts & ((2ull << here(lane)) - 1ull);
                const uint32_t found = (uint32_t)__shfl((int)m, 63 - __clzll((long long)(upto | 1ull)), kWave);
                src = upto ? found : src;
            }
            src += (uint32_t)v0;
            const uint32_t blk = u[k] >> rbits;
            const uint64_t same = lanes_alike<BITS>(has, blk);
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
            uint16_t* c = cnt + (has ? blk * kPartWaves + wave : 0u);
            const uint32_t prior = *c;
            wave_lds_order();                    // the lanes alike have read it
            if (has && below == 0) *c = (uint16_t)(prior + (uint32_t)__popcll(same));
            wave_lds_order();                    // before the next 64 read it
            place[k] = (blk << 16) | (prior + below);
            u[k] = ((src & ((1u << kTileSrcLoBits) - 1u)) << kTileRowBits) | (u[k] & rmask);
        }
    };
    auto wave_places = [&]() {
        if ((int)tid >= nrb) return;
        uint32_t run = l.start[tid];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint4 c = l.cnt[2 * tid + h];
            uint32_t x[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t mid = run + (x[q] & 0xFFFFu), next = mid + (x[q] >> 16);
                x[q] = run | (mid << 16);        // places are below 4097
                run = next;
            }
            l.cnt[2 * tid + h] = uint4{x[0], x[1], x[2], x[3]};
        }
    };
    auto put = [&](auto full, uint32_t n) {
#pragma unroll
        for (int k = 0; k < kPartPer; ++k)
            if (full || we0 + k * kWave < n) {
                const uint32_t at = cnt[(place[k] >> 16) * kPartWaves + wave] + (place[k] & 0xFFFFu);
                l.words[at] = u[k];
                l.blk_of[at] = (uint16_t)(place[k] >> 16);
            }
    };
    auto store = [&](const uint32_t* shift, auto full, uint32_t n) {
#pragma unroll
        for (int k = 0; k < kPartPer; ++k) {
            const uint32_t i = here(tid) + k * kPartBlock;
            if (full || i < n) t_edge[shift[l.blk_of[i]] + i] = l.words[i];
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
        clear_marks(l.mark[0], l.last[0]);
        clear_counts();
        keep_offsets();
        __syncthreads();
        mark_rows(tile, kPartTile, l.mark[0], l.last[0]);
        set_starts(l.shift[0]);
        int32_t v0 = r.v0;
        load_rows(at(tile + step));
        load_ends(at(tile + 2 * step));
        __syncthreads();
        for (int k = 0; tile < end; tile += step, k ^= 1) {      // k: which of the two marks and shifts
            rank(l.mark[k], l.last[k], v0, std::true_type{}, kPartTile);
            clear_marks(l.mark[k ^ 1], l.last[k ^ 1]);
            __syncthreads();
            wave_places();
            __syncthreads();
            put(std::true_type{}, kPartTile);
            keep_offsets();
            v0 = r.v0;
            load_edges(at(tile + step));
            __syncthreads();
            clear_counts();
            mark_rows(at(tile + step), kPartTile, l.mark[k ^ 1], l.last[k ^ 1]);
            set_starts(l.shift[k ^ 1]);
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
        for (int k = 0; k < kPartPer; ++k) u[k] = we0 + k * kWave < n ? (uint32_t)col[(int64_t)nfull * kPartTile + we0 + k * kWave] : 0u;
        clear_marks(l.mark[0], l.last[0]);
        clear_counts();
        keep_offsets();
        __syncthreads();
        mark_rows(nfull, n, l.mark[0], l.last[0]);
        set_starts(l.shift[0]);
        __syncthreads();
        rank(l.mark[0], l.last[0], r.v0, std::false_type{}, n);
        __syncthreads();
        wave_places();
        __syncthreads();
        put(std::false_type{}, n);
        __syncthreads();
        store(l.shift[0], std::false_type{}, n);
    }
}
static_assert(kPartMaxBlocks <= kPartBlock, "one block per thread");

// first[block * nch + c] = first edge of the block whose source is in chunk c (of 2^kTileSrcLoBits sources)
// or a later one: where the tile that holds the chunk's first edge starts in the block, and the edges of
// that tile before it.  One workgroup per chunk.
__global__ void __launch_bounds__(kPartBlock) part_first_kernel(int64_t M, const int64_t* __restrict__ rowptr,
                                                                const int32_t* __restrict__ col, int rbits, int nrb, int nch,
                                                                int64_t ntiles, const uint32_t* __restrict__ offs,
                                                                int64_t* __restrict__ first, const CsrFound* __restrict__ found) {
    if (csr_bad(found, M)) return;
    __shared__ uint32_t cnt[kPartMaxBlocks];
    const int c = blockIdx.x;
    const int64_t at = rowptr[(int64_t)c << kTileSrcLoBits];             // at most M
    const int64_t tile = at / kPartTile < ntiles ? at / kPartTile : ntiles - 1;
    if (threadIdx.x < kPartMaxBlocks) cnt[threadIdx.x] = 0u;
    __syncthreads();
    for (int64_t e = tile * kPartTile + threadIdx.x; e < at; e += kPartBlock) atomicAdd(&cnt[(uint32_t)col[e] >> rbits], 1u);
    __syncthreads();
    if ((int)threadIdx.x < nrb) first[(int64_t)threadIdx.x * nch + c] = (int64_t)offs[(int64_t)threadIdx.x * ntiles + tile] + cnt[threadIdx.x];
    if (c == 0 && threadIdx.x == 0) first[(int64_t)nrb * nch] = M;
}

// The sum of the mixes of the CSR's edges, each with the row that holds it: what the structure is compared with, found by
// another way than the one that built it.  A wavefront takes 2^piece_bits edges at a time (a tile, or less where the
// graph has fewer tiles than the chip wavefronts) and holds the ends of 64 rows in its lanes, among which an edge finds its
// own; the first row is sought from the tile's entry in tile_row[] on and must hold the first edge (else the structure
// is bad), later ones follow or, after a long run of empty rows, are found by bisection.  The next
// edges and the next 64 rows' ends are asked for before those in hand are looked at.  2.4M vertices, 121M edges: 175 us (207 without;
// 271 with a bisection over all rows for every 2048 edges' first one and one among the 64 rows for every edge).  Vector
// instructions bound it, the two products above all: the bytes alone take 72.
__global__ void __launch_bounds__(kBlock) csr_mix_kernel(int64_t N, int64_t M, const int64_t* __restrict__ rowptr,
                                                         const int32_t* __restrict__ col, const int32_t* __restrict__ tile_row,
                                                         int piece_bits, unsigned long long* __restrict__ mix, int* __restrict__ bad,
                                                         const CsrFound* __restrict__ found) {
    if (csr_bad(found, M)) return;
    constexpr int U = 4;                         // batches of 64 edges in flight
    const int lane = lane_id();
    const int64_t wave = (int64_t)blockIdx.x * (kBlock / kWave) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t nwaves = (int64_t)gridDim.x * (kBlock / kWave);
    unsigned long long sum = 0;
    for (int64_t piece = wave; piece << piece_bits < M; piece += nwaves) {
        const int64_t base = piece << piece_bits, tile = base / kPartTile;
        const uint32_t count = M - base < (1ll << piece_bits) ? (uint32_t)(M - base) : 1u << piece_bits;
        int64_t lo = tile_row[tile], up = base == tile * kPartTile ? lo : (tile + 1) * kPartTile < M ? tile_row[tile + 1] : N - 1;
        if (lo < 0 || lo > up || up >= N) { *bad = 1; continue; }
        while (lo < up) {
            const int64_t mid = (lo + up + 1) >> 1;
            if (rowptr[mid] <= base) lo = mid; else up = mid - 1;
        }
        if (rowptr[lo] > base || rowptr[lo + 1] <= base) { *bad = 1; continue; }
        uint32_t done = 0;
        uint32_t ahead[U];                       // the ids of the edges that come next
        auto load = [&](uint32_t p0) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t p = p0 + k * kWave + lane;
                ahead[k] = (uint32_t)__builtin_nontemporal_load(col + base + (p < count ? p : count - 1));
            }
        };
        auto row_end = [&](int64_t v) { return rowptr[v + 1 + lane < N ? v + 1 + lane : N]; };       // M at N
        load(0);
        while (done < count) {
            if (done > 0) {
                // the last row that starts at or before the edge (it holds it: rows after an empty one start where that does)
                int64_t hi = N - 1;
                lo = 0;
                while (lo < hi) {
                    const int64_t mid = (lo + hi + 1) >> 1;
                    if (rowptr[mid] <= base + done) lo = mid; else hi = mid - 1;
                }
            }
            // rows lo .. lo + 63, as long as they hold edges of the piece; the next 64 rows' ends are asked for before
            int64_t ends = row_end(lo);
            for (bool more = true; more && done < count; lo += kWave) {
                const int64_t end64 = ends - base;
                ends = row_end(lo + kWave);
                const uint32_t end = end64 < (int64_t)count ? (uint32_t)end64 : count;
                const uint32_t stop = (uint32_t)__builtin_amdgcn_readlane((int)end, kWave - 1);
                more = stop > done;
                for (uint32_t p0 = done; p0 < stop; p0 += U * kWave) {
                    uint32_t u[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) u[k] = ahead[k];
                    // the batches after these, or those of the next rows
                    load(p0 + U * kWave < stop ? p0 + U * kWave : stop);
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        const uint32_t p = p0 + k * kWave + lane;
                        // the rows of the 64 that end at or before the edge: those before the batch, then the few that
                        // end inside it one by one, many by bisection
                        const int first = __popcll(__ballot(end <= p0 + k * kWave));
                        const int last = __popcll(__ballot(end <= p0 + k * kWave + (kWave - 1)));
                        int r = first;
                        if (last - first <= 6) {
                            for (int i = first; i < last; ++i) r += (uint32_t)__builtin_amdgcn_readlane((int)end, i) <= p ? 1 : 0;
                        } else {
                            r = 0;               // at most 63 for an edge of the window
#pragma unroll
                            for (int s = kWave / 2; s > 0; s >>= 1)
                                if ((uint32_t)__shfl((int)end, r + s - 1, kWave) <= p) r += s;
                        }
                        if (p < stop) edge_mix(sum, (uint32_t)(lo + r), u[k]);
                    }
                }
                done = stop;
            }
        }
    }
    add_mix(sum, mix);
}

// Reads the structure back the way the propagation kernel does: every edge must lie in range and the sources of a
// block must ascend inside a chunk (so that a kernel that gathers through the structure never sees a source, a row or a place
// in its window of y out of range), and the edges' mixes must add up to those of the CSR's.  `parts` workgroups per
// row block; the block's chunk bounds sit in LDS.
__global__ void __launch_bounds__(kBlock) tile_verify_kernel(int rbits, int nch, const uint32_t* __restrict__ t_edge,
                                                             const int64_t* __restrict__ first, int parts, int64_t N, int64_t M,
                                                             unsigned long long* __restrict__ mix, int* __restrict__ bad,
                                                             const CsrFound* __restrict__ found) {
    extern __shared__ uint32_t bound[];
    if (csr_bad(found, M)) return;
    const int64_t rb = blockIdx.x / parts;
    const int j = blockIdx.x % parts;
    const int64_t b0 = first[rb * nch], len = first[(rb + 1) * nch] - b0;
    if (b0 < 0 || len < 0 || b0 + len > M || len > 0xFFFFFFFFll) { if (threadIdx.x == 0) *bad = 1; return; }
    for (int c = threadIdx.x; c <= nch; c += kBlock) {
        const int64_t f = first[rb * nch + c] - b0;
        if (f < 0 || f > len || (c > 0 && first[rb * nch + c] < first[rb * nch + c - 1])) *bad = 1;
        bound[c] = (uint32_t)f;
    }
    __syncthreads();
    unsigned long long sum = 0;
    const uint32_t beg = (uint32_t)(len * j / parts), end = (uint32_t)(len * (j + 1) / parts);
    const uint32_t rows = N - (rb << rbits) < (1ll << rbits) ? (uint32_t)(N - (rb << rbits)) : 1u << rbits;
    const uint32_t u0 = (uint32_t)(rb << rbits);
    const uint32_t* __restrict__ words = t_edge + b0;
    bool wrong = false;
    for (int c = 0; c < nch; ++c) {              // the share's part of every chunk of sources
        const uint32_t lo = bound[c] > beg ? bound[c] : beg, hi = bound[c + 1] < end ? bound[c + 1] : end;
#pragma unroll 8
        for (uint32_t p = lo + threadIdx.x; p < hi; p += kBlock) {
            const uint32_t w = words[p], before = words[p > bound[c] ? p - 1 : p];
            wrong |= !tile_word_ok(w, before, c, (uint32_t)N, rows);
            edge_mix(sum, tile_source(w, c), u0 + (w & kTileRowMask));
        }
    }
    if (wrong) *bad = 1;
    add_mix(sum, mix);
}

struct PartIn  { const uint32_t* h; __device__ int operator()(int64_t i) const { return (int)h[i]; } };
struct PartOut { uint32_t* h; __device__ void operator()(int64_t i, int ex, int) const { h[i] = (uint32_t)ex; } };
struct PartFin { uint32_t* end; __device__ void operator()(int total) const { *end = (uint32_t)total; } };

__global__ void block_first_from_tiles_kernel(const int64_t* __restrict__ tile_first, int nch, int64_t nrb,
                                              int64_t* __restrict__ block_first) {      // copies whatever tile_first[] holds
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b <= nrb) block_first[b] = tile_first[b * nch];
}

// Says what is wrong with the CSR, if anything is.
static bool csr_error(const CsrFound& f, int64_t M) {
    if (f.first != 0 || f.last != M)
        set_error("spp_graph_create: rowptr[0] = %lld, rowptr[N] = %lld, M = %lld", (long long)f.first, (long long)f.last, (long long)M);
    else if (f.bad)
        set_error("spp_graph_create: rowptr is not monotone within [0, M] or a column id lies outside [0, N)");
    else
        return false;
    return true;
}

// The edges grouped by destination row block and sorted by source inside a block.  Validates the CSR if M > 0.
static int build_tiles(spp_ctx* ctx, spp_graph* g) {
    hipStream_t st = ctx->stream;
    const int64_t N = g->N, M = g->M;
    const int grid = ctx->num_cu * 8;
    int lds = 0;
    SPP_HIP(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, ctx->device));
    const int nch = (int)((N + ((int64_t)1 << kTileSrcLoBits) - 1) >> kTileSrcLoBits);
    // the fp64 sums of a block, the wavefronts' windows of y and the block's chunk bounds share the LDS of a workgroup
    const size_t bound_bytes = (size_t)(nch + 1) * sizeof(uint32_t);
    const size_t beside = bound_bytes + kTileWinBytes + 1024;
    const int rbits = (size_t)lds >= (sizeof(double) << kTileRowBits) + beside ? kTileRowBits : kTileRowBits - 1;
    SPP_CHECK((size_t)lds >= (sizeof(double) << rbits) + beside, SPP_E_HIP,
              "row blocks: %d bytes of LDS per workgroup do not hold a block's sums and chunk bounds", lds);
    const int64_t nrb = (N + ((int64_t)1 << rbits) - 1) >> rbits;
    SPP_CHECK(nrb <= kPartMaxBlocks, SPP_E_HIP, "row blocks: %lld blocks of 2^%d rows", (long long)nrb, rbits);
    static_assert(kPartMaxBlocks <= 512, "nine bits name a block");
    g->tile_rbits = rbits; g->nrb = nrb; g->nch = nch;
    const int64_t nfirst = nrb * nch + 1;
    SPP_HIP(pool_take(g->device, &g->tile_first, (size_t)nfirst * sizeof(int64_t)));
    SPP_HIP(pool_take(g->device, &g->t_edge, (size_t)(M > 0 ? M : 1) * sizeof(uint32_t)));
    SPP_HIP(pool_take(g->device, &g->block_first, (size_t)(nrb + 1) * sizeof(int64_t)));
    const unsigned bf_grid = (unsigned)((nrb + 1 + kBlock - 1) / kBlock);
    if (M > 0) {
        const int64_t ntiles = (M + kPartTile - 1) / kPartTile;
        const int64_t nhist = nrb * ntiles;
        const int scan_grid = 1024;
        // one allocation: the counts (then offsets) and the tiles' first rows, which the graph keeps, the scan's
        // partial sums, the sums of the edges' mixes and a flag
        struct Head { unsigned long long mix[2]; int bad, pad; CsrFound csr; } back;
        const size_t bytes = sizeof(Head) + (size_t)(nhist + 1 + scan_grid) * sizeof(int) + (size_t)(ntiles + 1) * sizeof(int32_t);
        char* tmp = nullptr;
        if (pool_take(g->device, &tmp, bytes) != hipSuccess) {
            (void)hipGetLastError();
            set_error("row blocks: out of device memory for %zu bytes of counts", bytes);
            return SPP_E_OOM;
        }
        unsigned long long* mix = reinterpret_cast<unsigned long long*>(tmp);
        int* d_bad = reinterpret_cast<int*>(mix + 2);
        CsrFound* found = &reinterpret_cast<Head*>(tmp)->csr;
        uint32_t* hist = reinterpret_cast<uint32_t*>(tmp + sizeof(Head));
        int* partial = reinterpret_cast<int*>(hist + nhist + 1);
        int32_t* tile_row = partial + scan_grid;
        int rc = SPP_OK;
        hipError_t e = hipMemsetAsync(tmp, 0, sizeof(Head), st);
        if (e == hipSuccess) {
            const int pgrid = (int)(ntiles < (int64_t)ctx->num_cu * 8 ? ntiles : (int64_t)ctx->num_cu * 8);
            part_rows_kernel<<<grid, kBlock, 0, st>>>(N, M, ntiles, g->rowptr, tile_row, found);
            part_count_kernel<<<pgrid, kPartBlock, 0, st>>>(N, M, g->rowptr, g->col, rbits, (int)nrb, ntiles, hist, found);
            grid_scan(st, scan_grid, nhist, PartIn{hist}, PartOut{hist}, PartFin{hist + nhist}, partial);
            // two workgroups per CU, fewer where there are fewer tiles; a multiple of eight
            const int64_t want_place = (ntiles + 7) / 8 * 8, most_place = ctx->num_cu * 2 / 8 * 8;
            const size_t place_lds = offsetof(PlaceLds, cnt) + (size_t)nrb * kPartWaves * sizeof(uint16_t);
            auto place = [&](auto kernel) {
                e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)place_lds);
                if (e != hipSuccess) return;
                kernel<<<(unsigned)(want_place < most_place ? want_place : most_place), kPartBlock, place_lds, st>>>(
                    N, M, g->rowptr, g->col, rbits, (int)nrb, (int)ntiles, tile_row, hist, g->t_edge, found);
            };
            if (nrb <= 256) place(part_place_kernel<8>); else place(part_place_kernel<9>);
            part_first_kernel<<<nch, kPartBlock, 0, st>>>(M, g->rowptr, g->col, rbits, (int)nrb, nch, ntiles, hist, g->tile_first, found);
            int piece_bits = 8;
            while ((1 << piece_bits) < kPartTile && (M >> piece_bits) > (int64_t)ctx->num_cu * 8 * (kBlock / kWave)) ++piece_bits;
            csr_mix_kernel<<<ctx->num_cu * 8, kBlock, 0, st>>>(N, M, g->rowptr, g->col, tile_row, piece_bits, mix, d_bad, found);
            const int64_t want = ((int64_t)ctx->num_cu * 8 + nrb - 1) / nrb;
            const int parts = (int)(want < 1 ? 1 : (want > 256 ? 256 : want));
            tile_verify_kernel<<<(unsigned)(nrb * parts), kBlock, bound_bytes, st>>>(rbits, nch, g->t_edge, g->tile_first, parts, N, M,
                                                                                     mix + 1, d_bad, found);
            block_first_from_tiles_kernel<<<bf_grid, kBlock, 0, st>>>(g->tile_first, nch, nrb, g->block_first);
            if (e == hipSuccess) e = hipMemcpyAsync(ctx->h_pinned, tmp, sizeof(back), hipMemcpyDeviceToHost, st);
        }
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        memcpy(&back, ctx->h_pinned, sizeof(back));
        if (e == hipSuccess) e = hipGetLastError();
        if (e != hipSuccess) { set_error("row blocks: %s", hipGetErrorString(e)); rc = SPP_E_HIP; }
        else if (csr_error(back.csr, M)) rc = SPP_E_ARG;
        else if (back.bad || back.mix[0] != back.mix[1]) {
            set_error("row blocks: the structure does not read back as the edges it was built from"); rc = SPP_E_HIP;
        }
        g->part_mem = tmp;               // freed with the graph, also after an error
        SPP_TRY(rc);
        g->tile_off = hist; g->tile_row = tile_row; g->part_tiles = ntiles;
    }
    if (M == 0) {
        fill_i64_kernel<<<grid, kBlock, 0, st>>>(g->tile_first, nfirst, M);
        block_first_from_tiles_kernel<<<bf_grid, kBlock, 0, st>>>(g->tile_first, nch, nrb, g->block_first);
        SPP_HIP(hipStreamSynchronize(st));
    }
    return SPP_OK;
}


// ---- the chunked layout ------------------------------------------------------------------------
// key[e] = (source chunk, row block, source inside the chunk, row inside the block) for the e-th
// edge v -> u of the CSR.
__global__ void __launch_bounds__(kBlock) x_keys_kernel(int64_t N, const int64_t* __restrict__ rowptr,
                                                        const int32_t* __restrict__ col, int bbits,
                                                        uint64_t* __restrict__ keys) {
    const int lane = lane_id();
    const int64_t wave = ((int64_t)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * kBlock) >> 6;
    constexpr int lo_bits = kXSrcBits + kTileRowBits;
    for (int64_t v = wave; v < N; v += nwaves) {
        const int64_t b = rowptr[v], e = rowptr[v + 1];
        const uint64_t vc = (uint64_t)v >> kXSrcBits, vl = (uint64_t)v & ((1u << kXSrcBits) - 1u);
        for (int64_t i = b + lane; i < e; i += kWave) {
            const uint64_t u = (uint64_t)(uint32_t)col[i];          // validated at graph creation
            keys[i] = (vc << (lo_bits + bbits)) | ((u >> kTileRowBits) << lo_bits) | (vl << kTileRowBits) | (u & kTileRowMask);
        }
    }
}

// Piece index (chunk-major) of a key.
__device__ __forceinline__ int64_t x_piece_of(uint64_t k, int bbits, int64_t nrb) {
    constexpr int lo_bits = kXSrcBits + kTileRowBits;
    return (int64_t)(k >> (lo_bits + bbits)) * nrb + (int64_t)((k >> lo_bits) & ((1ull << bbits) - 1));
}

// first[g] = first sorted edge whose piece index is >= g (entries beyond the last piece keep the M
// they were filled with).
__global__ void __launch_bounds__(kBlock) x_bounds_kernel(const uint64_t* __restrict__ keys, int64_t M, int bbits,
                                                          int64_t nrb, int64_t* __restrict__ first) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < M; e += stride) {
        const int64_t g = x_piece_of(keys[e], bbits, nrb);
        const int64_t prev = e > 0 ? x_piece_of(keys[e - 1], bbits, nrb) : -1;
        for (int64_t r = prev + 1; r <= g; ++r) first[r] = e;
    }
}

// Exclusive prefix sums of the padded piece sizes, in three steps: per 1024 pieces a sum, the sums
// scanned by one workgroup, then the pieces' own offsets.  padded[npieces] = all entries.
constexpr int kXScanPer = 4;
__device__ __forceinline__ int64_t x_padded_len(const int64_t* first, int64_t g) {
    return (first[g + 1] - first[g] + 3) & ~(int64_t)3;
}
__global__ void __launch_bounds__(kBlock) x_scan_sums_kernel(const int64_t* __restrict__ first, int64_t npieces,
                                                             int64_t* __restrict__ sums) {
    __shared__ long long red[kBlock / kWave];
    const int64_t g0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kXScanPer;
    long long acc = 0;
    for (int k = 0; k < kXScanPer; ++k)
        if (g0 + k < npieces) acc += x_padded_len(first, g0 + k);
    for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_down(acc, off, kWave);
    if (lane_id() == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}
__global__ void __launch_bounds__(kBlock) x_scan_top_kernel(int64_t* __restrict__ sums, int64_t n) {
    __shared__ long long wsum[kBlock / kWave];
    __shared__ long long carry_lds;
    if (threadIdx.x == 0) carry_lds = 0;
    __syncthreads();
    for (int64_t base = 0; base < n; base += kBlock) {
        const int64_t i = base + threadIdx.x;
        const long long v = i < n ? sums[i] : 0;
        long long inc = v;
        const int lane = lane_id(), wave = threadIdx.x >> 6;
        for (int off = 1; off < kWave; off <<= 1) {
            const long long t = __shfl_up(inc, off, kWave);
            if (lane >= off) inc += t;
        }
        if (lane == kWave - 1) wsum[wave] = inc;
        __syncthreads();
        long long before = carry_lds;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (i < n) sums[i] = before + inc - v;
        __syncthreads();
        if (threadIdx.x == kBlock - 1) carry_lds = before + inc;
        __syncthreads();
    }
}
__global__ void __launch_bounds__(kBlock) x_scan_write_kernel(const int64_t* __restrict__ first, int64_t npieces,
                                                              const int64_t* __restrict__ sums, int64_t* __restrict__ padded) {
    __shared__ long long wsum[kBlock / kWave];
    const int64_t g0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kXScanPer;
    long long len[kXScanPer], mine = 0;
    for (int k = 0; k < kXScanPer; ++k) {
        len[k] = g0 + k < npieces ? x_padded_len(first, g0 + k) : 0;
        mine += len[k];
    }
    long long inc = mine;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    for (int off = 1; off < kWave; off <<= 1) {
        const long long t = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += t;
    }
    if (lane == kWave - 1) wsum[wave] = inc;
    __syncthreads();
    long long at = sums[blockIdx.x] + inc - mine;
    for (int w = 0; w < wave; ++w) at += wsum[w];
    for (int k = 0; k < kXScanPer; ++k) {
        if (g0 + k < npieces) padded[g0 + k] = at;
        at += len[k];
        if (g0 + k == npieces - 1) padded[npieces] = at;
    }
}

// The entries: sorted edge e of piece g goes to padded[g] + (e - first[g]).
__global__ void __launch_bounds__(kBlock) x_entries_kernel(const uint64_t* __restrict__ keys, int64_t M, int bbits,
                                                           int64_t nrb, const int64_t* __restrict__ first,
                                                           const int64_t* __restrict__ padded,
                                                           uint16_t* __restrict__ x_src, uint16_t* __restrict__ x_row) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < M; e += stride) {
        const uint64_t k = keys[e];
        const int64_t g = x_piece_of(k, bbits, nrb);
        const int64_t pos = padded[g] + (e - first[g]);
        x_src[pos] = (uint16_t)((k >> kTileRowBits) & ((1u << kXSrcBits) - 1u));
        x_row[pos] = (uint16_t)(k & kTileRowMask);
    }
}
// The padding at the end of every piece.
__global__ void __launch_bounds__(kBlock) x_padding_kernel(int64_t npieces, const int64_t* __restrict__ first,
                                                           const int64_t* __restrict__ padded,
                                                           uint16_t* __restrict__ x_src, uint16_t* __restrict__ x_row) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x; g < npieces; g += stride)
        for (int64_t pos = padded[g] + (first[g + 1] - first[g]); pos < padded[g + 1]; ++pos) {
            x_src[pos] = (uint16_t)kXPad;
            x_row[pos] = 0;
        }
}
// Per row block b (one thread each; at step c the threads of a wavefront read neighbouring pieces):
// where its piece of every chunk starts, how many vectors of the block lie in earlier chunks, and
// the edges that end in the block.
__global__ void __launch_bounds__(kBlock) x_tables_kernel(int64_t nrb, int nch, const int64_t* __restrict__ first,
                                                          const int64_t* __restrict__ padded,
                                                          uint32_t* __restrict__ x_start, uint32_t* __restrict__ x_prefix,
                                                          int64_t* __restrict__ block_edges) {
    const int64_t b = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (b >= nrb) return;
    uint32_t vecs = 0;
    int64_t edges = 0;
    for (int c = 0; c < nch; ++c) {
        const int64_t g = (int64_t)c * nrb + b;
        x_start[b * nch + c] = (uint32_t)(padded[g] >> 2);
        x_prefix[b * (nch + 1) + c] = vecs;
        vecs += (uint32_t)((padded[g + 1] - padded[g]) >> 2);
        edges += first[g + 1] - first[g];
    }
    x_prefix[b * (nch + 1) + nch] = vecs;
    block_edges[b] = edges;
}
__global__ void x_chunk_first_kernel(int64_t nrb, int nch, const int64_t* __restrict__ padded, int64_t* __restrict__ chunk_first) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c <= nch) chunk_first[c] = padded[(int64_t)c * nrb];
}
// block_first[b] = sum of counts[0 .. b), b <= nrb, by one workgroup (counts sits in block_first[1 ..]).
__global__ void __launch_bounds__(kBlock) block_first_kernel(int64_t* __restrict__ block_first, int64_t nrb) {
    __shared__ long long wsum[kBlock / kWave];
    __shared__ long long carry_lds;
    if (threadIdx.x == 0) { carry_lds = 0; }
    __syncthreads();
    for (int64_t base = 0; base < nrb; base += kBlock) {
        const int64_t i = base + threadIdx.x;
        const long long v = i < nrb ? block_first[i + 1] : 0;
        long long inc = v;
        const int lane = lane_id(), wave = threadIdx.x >> 6;
        for (int off = 1; off < kWave; off <<= 1) {
            const long long t = __shfl_up(inc, off, kWave);
            if (lane >= off) inc += t;
        }
        if (lane == kWave - 1) wsum[wave] = inc;
        __syncthreads();
        long long before = carry_lds;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        __syncthreads();
        if (i < nrb) block_first[i + 1] = before + inc;          // inclusive: the prefix of b + 1
        if (threadIdx.x == kBlock - 1) carry_lds = before + inc;
        __syncthreads();
    }
    if (threadIdx.x == 0) block_first[0] = 0;
}

// Reads the arrays back the way the propagation kernels do: every entry that is not padding must
// be an edge of the CSR (found in the row of its source), lie in the piece that holds it, and the
// entries that are not padding must number M; the per-row-block tables must agree with the pieces'
// offsets.  A kernel that walks the structure afterwards never sees a source or a row out of range.
__global__ void __launch_bounds__(kBlock) x_verify_kernel(int64_t N, int64_t nrb, int nch, const int64_t* __restrict__ rowptr,
                                                          const int32_t* __restrict__ col,
                                                          const int64_t* __restrict__ padded, int64_t entries,
                                                          const uint16_t* __restrict__ x_src, const uint16_t* __restrict__ x_row,
                                                          const uint32_t* __restrict__ x_start, const uint32_t* __restrict__ x_prefix,
                                                          unsigned long long* __restrict__ real, int* __restrict__ bad) {
    __shared__ int lds[4];
    const int64_t npieces = nrb * nch;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    int mine = 0;
    for (int64_t pos = (int64_t)blockIdx.x * kBlock + threadIdx.x; pos < entries; pos += stride) {
        const uint32_t s = x_src[pos];
        if (s & kXPad) continue;
        int64_t lo = 0, hi = npieces - 1;                       // last piece g with padded[g] <= pos
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (padded[mid] <= pos) lo = mid; else hi = mid - 1;
        }
        const int64_t c = lo / nrb, b = lo - c * nrb;
        const int64_t v = (c << kXSrcBits) | s, u = (b << kTileRowBits) | x_row[pos];
        bool ok = pos < padded[lo + 1] && v < N && u < N && x_row[pos] <= kTileRowMask;
        if (ok) {
            int64_t a = rowptr[v], e = rowptr[v + 1];
            ok = false;
            while (a < e) {
                const int64_t mid = (a + e) >> 1;
                const int64_t w = col[mid];
                if (w == u) { ok = true; break; }
                if (w < u) a = mid + 1; else e = mid;
            }
        }
        if (!ok) *bad = 1;
        ++mine;
    }
    const int total = block_reduce_sum(mine, lds);
    if (threadIdx.x == 0 && total) atomicAdd(real, (unsigned long long)total);
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < npieces; t += stride) {
        const int64_t b = t / nch, c = t - b * nch, g = c * nrb + b;
        const bool ok = (int64_t)x_start[t] * 4 == padded[g] &&
                        (int64_t)(x_prefix[b * (nch + 1) + c + 1] - x_prefix[b * (nch + 1) + c]) * 4 == padded[g + 1] - padded[g] &&
                        (c > 0 || x_prefix[b * (nch + 1)] == 0) && (padded[g] & 3) == 0;
        if (!ok) *bad = 1;
    }
}

struct XBuild {               // temporaries of build_chunked, freed on every path
    uint64_t *ka = nullptr, *kb = nullptr;
    int64_t *first = nullptr, *padded = nullptr, *sums = nullptr;
    unsigned long long* real = nullptr;
    int* bad = nullptr;
    ~XBuild() {
        (void)hipFree(ka); (void)hipFree(kb); (void)hipFree(first); (void)hipFree(padded); (void)hipFree(sums);
        (void)hipFree(real); (void)hipFree(bad);
    }
};

// The edges sorted by (chunk of sources, row block) with padded pieces, and the tables of both walks.
static int build_chunked(spp_ctx* ctx, spp_graph* g) {
    hipStream_t st = ctx->stream;
    const int64_t N = g->N, M = g->M;
    const int grid = ctx->num_cu * 8;
    const int nch = (int)((N + ((int64_t)1 << kXSrcBits) - 1) >> kXSrcBits);
    const int64_t nrb = (N + ((int64_t)1 << kTileRowBits) - 1) >> kTileRowBits;
    int bbits = 1, cbits = 1;
    while (((int64_t)1 << bbits) < nrb) ++bbits;
    while (((int64_t)1 << cbits) < nch) ++cbits;
    const int64_t npieces = nrb * nch;
    SPP_CHECK(M + 3 * npieces < ((int64_t)1 << 34), SPP_E_ARG, "chunked layout: %lld edges in %lld pieces exceed 2^32 vectors",
              (long long)M, (long long)npieces);
    g->tile_rbits = kTileRowBits; g->nrb = nrb; g->x_nch = nch;
    SPP_HIP(pool_take(g->device, &g->block_first, (size_t)(nrb + 1) * sizeof(int64_t)));
    SPP_HIP(pool_take(g->device, &g->x_chunk_first, (size_t)(nch + 1) * sizeof(int64_t)));
    SPP_HIP(pool_take(g->device, &g->x_start, (size_t)npieces * sizeof(uint32_t)));
    SPP_HIP(pool_take(g->device, &g->x_prefix, (size_t)nrb * (nch + 1) * sizeof(uint32_t)));
    XBuild t;
    SPP_HIP(device_malloc(&t.first, (size_t)(npieces + 1) * sizeof(int64_t)));
    SPP_HIP(device_malloc(&t.padded, (size_t)(npieces + 1) * sizeof(int64_t)));
    const int64_t nsum = (npieces + (int64_t)kBlock * kXScanPer - 1) / ((int64_t)kBlock * kXScanPer);
    SPP_HIP(device_malloc(&t.sums, (size_t)(nsum + 1) * sizeof(int64_t)));
    SPP_HIP(device_malloc(&t.real, sizeof(unsigned long long)));
    SPP_HIP(device_malloc(&t.bad, sizeof(int)));
    SPP_HIP(device_malloc(&t.ka, (size_t)(M > 0 ? M : 1) * sizeof(uint64_t)));
    SPP_HIP(device_malloc(&t.kb, (size_t)(M > 0 ? M : 1) * sizeof(uint64_t)));
    uint64_t* sorted = t.ka;
    fill_i64_kernel<<<grid, kBlock, 0, st>>>(t.first, npieces + 1, M);
    if (M > 0) {
        x_keys_kernel<<<grid, kBlock, 0, st>>>(N, g->rowptr, g->col, bbits, t.ka);
        constexpr int lo_bits = kXSrcBits + kTileRowBits;
        SPP_TRY(radix_sort_u64(ctx, t.ka, t.kb, M, lo_bits, lo_bits + bbits + cbits, &sorted));
        x_bounds_kernel<<<grid, kBlock, 0, st>>>(sorted, M, bbits, nrb, t.first);
    }
    x_scan_sums_kernel<<<(unsigned)nsum, kBlock, 0, st>>>(t.first, npieces, t.sums);
    x_scan_top_kernel<<<1, kBlock, 0, st>>>(t.sums, nsum);
    x_scan_write_kernel<<<(unsigned)nsum, kBlock, 0, st>>>(t.first, npieces, t.sums, t.padded);
    int64_t entries = 0;
    SPP_HIP(hipMemcpyAsync(&entries, t.padded + npieces, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    SPP_HIP(hipStreamSynchronize(st));
    SPP_CHECK(entries >= M && entries <= M + 3 * npieces && (entries & 3) == 0, SPP_E_HIP,
              "chunked layout: %lld entries for %lld edges in %lld pieces", (long long)entries, (long long)M, (long long)npieces);
    g->x_entries = entries;
    SPP_HIP(pool_take(g->device, &g->x_src, (size_t)(entries > 0 ? entries : 4) * sizeof(uint16_t)));
    SPP_HIP(pool_take(g->device, &g->x_row, (size_t)(entries > 0 ? entries : 4) * sizeof(uint16_t)));
    if (M > 0) x_entries_kernel<<<grid, kBlock, 0, st>>>(sorted, M, bbits, nrb, t.first, t.padded, g->x_src, g->x_row);
    x_padding_kernel<<<grid, kBlock, 0, st>>>(npieces, t.first, t.padded, g->x_src, g->x_row);
    x_tables_kernel<<<(unsigned)((nrb + kBlock - 1) / kBlock), kBlock, 0, st>>>(nrb, nch, t.first, t.padded, g->x_start,
                                                                                g->x_prefix, g->block_first + 1);
    block_first_kernel<<<1, kBlock, 0, st>>>(g->block_first, nrb);
    x_chunk_first_kernel<<<(unsigned)((nch + 1 + kBlock - 1) / kBlock), kBlock, 0, st>>>(nrb, nch, t.padded, g->x_chunk_first);
    SPP_HIP(hipMemsetAsync(t.real, 0, sizeof(unsigned long long), st));
    SPP_HIP(hipMemsetAsync(t.bad, 0, sizeof(int), st));
    x_verify_kernel<<<grid, kBlock, 0, st>>>(N, nrb, nch, g->rowptr, g->col, t.padded, entries, g->x_src, g->x_row,
                                             g->x_start, g->x_prefix, t.real, t.bad);
    unsigned long long real = 0;
    int bad = 0;
    SPP_HIP(hipMemcpyAsync(&real, t.real, sizeof(real), hipMemcpyDeviceToHost, st));
    SPP_HIP(hipMemcpyAsync(&bad, t.bad, sizeof(bad), hipMemcpyDeviceToHost, st));
    SPP_HIP(hipStreamSynchronize(st));
    SPP_HIP(hipGetLastError());
    SPP_CHECK(bad == 0 && (int64_t)real == M, SPP_E_HIP,
              "chunked layout: the structure does not read back as the edges it was built from (%llu of %lld entries)",
              real, (long long)M);
    return SPP_OK;
}

}  // namespace spp

extern "C" int spp_graph_create(spp_ctx* ctx, int64_t N, int64_t M, const int64_t* d_rowptr,
                                const int32_t* d_col, uint32_t flags, spp_graph** out) {
    SPP_CHECK(ctx && out, SPP_E_ARG, "spp_graph_create: null argument");
    *out = nullptr;
    SPP_CHECK(N > 0 && N <= 0x7FFFFFFFll, SPP_E_ARG, "spp_graph_create: N = %lld out of range (int32 ids)", (long long)N);
    SPP_CHECK(M >= 0 && M < 0xFFFFFFFFll, SPP_E_ARG, "spp_graph_create: M = %lld out of range", (long long)M);
    SPP_CHECK(d_rowptr && (d_col || M == 0), SPP_E_ARG, "spp_graph_create: null CSR array");
    SPP_HIP(hipSetDevice(ctx->device));
    spp_graph* g = new (std::nothrow) spp_graph();
    SPP_CHECK(g != nullptr, SPP_E_OOM, "spp_graph_create: out of host memory");
    g->device = ctx->device; g->N = N; g->M = M; g->rowptr = d_rowptr; g->col = d_col;
    // which layout: gathering y per edge pays while y stays in the caches (see spp_vip.hip)
    const bool lists = (flags & SPP_GRAPH_IN_LISTS) != 0;
    const bool chunked = lists && ((flags & SPP_GRAPH_CHUNKED) != 0 || N > spp::kChunkedAboveVertices);
    // the arrays may come from the default stream, which a context's stream need not wait for
    hipError_t e = ctx->stream ? hipStreamSynchronize(nullptr) : hipSuccess;
    if (e == hipSuccess && !(lists && !chunked && M > 0)) {          // the row blocks' build does it on the way
        spp::CsrFound* d_found = nullptr;
        spp::CsrFound* found = reinterpret_cast<spp::CsrFound*>(ctx->h_pinned);
        e = spp::pool_take(g->device, &d_found, sizeof(*found));
        if (e == hipSuccess) e = hipMemsetAsync(d_found, 0, sizeof(*found), ctx->stream);
        if (e == hipSuccess) {
            spp::validate_csr_kernel<<<ctx->num_cu * 8, spp::kBlock, 0, ctx->stream>>>(N, M, d_rowptr, d_col, d_found);
            e = hipMemcpyAsync(found, d_found, sizeof(*found), hipMemcpyDeviceToHost, ctx->stream);
        }
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        if (e == hipSuccess) spp::pool_give(g->device, d_found); else spp::pool_retire(g->device, {d_found});
        if (e == hipSuccess && spp::csr_error(*found, M)) { delete g; return SPP_E_ARG; }
    }
    if (e != hipSuccess) { spp::set_error("spp_graph_create: %s", hipGetErrorString(e)); delete g; return SPP_E_HIP; }
    if (flags & SPP_GRAPH_IN_LISTS) {
        int rc = chunked ? spp::build_chunked(ctx, g) : spp::build_tiles(ctx, g);
        if (rc != SPP_OK) { spp_graph_destroy(g); return rc; }
        g->has_in = true;
        g->has_x = chunked;
    }
    *out = g;
    return SPP_OK;
}

extern "C" void spp_graph_destroy(spp_graph* g) {
    if (!g) return;
    if (hipSetDevice(g->device) != hipSuccess) { (void)hipGetLastError(); delete g; return; }   // runtime already shut down
    // work that still reads the row blocks may be in flight
    spp::pool_retire(g->device, {g->t_edge, g->tile_first, g->part_mem, g->block_first, g->x_src, g->x_row, g->x_chunk_first, g->x_start,
                                 g->x_prefix});
    delete g;
}
