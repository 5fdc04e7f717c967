// VIP-ranked replica cache (Secs. 3.2, 4.2): rank the remote vertices by decreasing score, keep
// the first floor(alpha*N/K), build the id -> slot table, copy their rows from the remote store.
//
// Of all candidates (remote, score > 0) only those that can be kept are ranked: positive floats order
// like their bit patterns, so three histogram passes over the scores (11, 10 and 10 bits) find the C-th
// largest score exactly.  The candidates at or above it are compacted in ascending id order (one launch counts
// a workgroup's, one places them), packed as (~score bits) << 32 | id, and sorted: in one workgroup up to 4096 of them, else
// stably by radix on the score bits only (the complement turns ascending into descending score, and
// stability keeps ascending id among equal scores).  Before, all candidates were sorted, in buffers of
// 16 bytes per candidate that each call allocated.  A call with 8-byte rows in device memory, 320k kept of 8M scores: 280 -> 173 us
// with a workgroup per CU in the passes over the scores and two launches per pass of the sort; 60k of 1M 196 -> 121, 10k of 60k
// 162 -> 104, 1.5M of 8M 456 -> 378.  Rows from the host add what the link takes: 8M scores, 320k rows of 256 bytes 1.70 ms, 1.53 of it.
#include "spp_common.h"
#include "spp_device.h"
#include "spp_rowcopy.h"

#include <math.h>
#include <new>

namespace spp {

// The histograms of a ranking, one after the other, and what they decide.
constexpr int kRankBins[3] = {2048, 1024, 1024}, kRankShift[3] = {20, 10, 0};
constexpr int kRankHistWords = 2048 + 1024 + 1024;
struct RankArgs {
    const float* score;
    int64_t      N, lo, hi;
    uint64_t     C;                  // candidates wanted
    uint32_t*    hist;               // kRankHistWords counts
};
__device__ __forceinline__ uint32_t candidate_bits(const RankArgs& a, int64_t u) {      // 0: not a candidate, or beyond the last id
    const float s = a.score[u < a.N ? u : a.N - 1];              // whatever u: a load under a condition is waited for by itself
    return s > 0.0f && u < a.N && !(u >= a.lo && u < a.hi) ? __float_as_uint(s) : 0u;
}
// The smallest score bits that are kept, as far as the first `passes` histograms decide them: the digit of
// each pass is the largest bin from which on upward there are enough candidates.  kTooFew if all candidates
// together are.  All threads of a workgroup of kRankBlock; after all three passes `kept` is how many candidates
// reach them, ties at the threshold included.
constexpr uint32_t kTooFew = 0xFFFFFFFFu;            // not the bits of a positive score
constexpr int kRankBlock = 1024, kRankWaves = kRankBlock / kWave;
struct RankLds { uint32_t sums[kRankWaves]; unsigned long long bin, want, holds; };
__device__ __forceinline__ uint32_t kept_from(const RankArgs& a, int passes, RankLds& l, uint64_t& kept) {
    uint64_t want = a.C;
    uint32_t bits = 0;
    const uint32_t* h = a.hist;
    const int wave = threadIdx.x >> 6;
    kept = 0;
    for (int p = 0; p < passes; ++p) {
        const int nb = kRankBins[p], per = nb / kRankBlock;
        // thread t adds up the t-th run of bins from the top, modulo 2^32, which the at most 2^31 candidates fit
        uint32_t mine = 0;
        for (int i = 0; i < per; ++i) mine += h[nb - 1 - (int)threadIdx.x * per - i];
        const uint32_t inc = (uint32_t)wave_inclusive_scan((int)mine);
        if (lane_id() == kWave - 1) l.sums[wave] = inc;
        __syncthreads();
        uint32_t above = inc - mine, all = 0;
        for (int w = 0; w < kRankWaves; ++w) {
            const uint32_t x = l.sums[w];
            above += w < wave ? x : 0u;
            all += x;
        }
        if ((uint64_t)all < want) { kept = all; return kTooFew; }        // only possible at the first pass
        if (above < want && above + (uint64_t)mine >= want)      // one thread
            for (int i = 0; i < per; ++i) {
                const int bin = nb - 1 - (int)threadIdx.x * per - i;
                const uint32_t c = h[bin];
                if (above + (uint64_t)c >= want) { l.bin = (unsigned long long)bin; l.want = want - above; l.holds = c; break; }
                above += c;
            }
        __syncthreads();
        bits |= (uint32_t)l.bin << kRankShift[p];
        want = l.want;
        kept = a.C - want + l.holds;
        __syncthreads();
        h += nb;
    }
    return bits;
}
// One workgroup per CU: each adds what it has counted to the same few bins (scores cluster), at 15 ns an add.  8M scores, the three
// passes: 31, 17 and 15 us with four workgroups of 256 threads per CU.
__global__ void __launch_bounds__(kRankBlock) rank_hist_kernel(RankArgs a, int pass) {
    constexpr int kCopies = 4, U = 8;            // scores in flight per thread
    __shared__ uint32_t h[kCopies][2048];
    __shared__ RankLds l;
    const int nb = kRankBins[pass], shift = kRankShift[pass];
    for (int i = threadIdx.x; i < kCopies * 2048; i += kRankBlock) (&h[0][0])[i] = 0u;
    uint64_t kept;
    const uint32_t from = kept_from(a, pass, l, kept);
    if (pass > 0 && from == kTooFew) return;          // every candidate is kept: nothing to narrow down
    __syncthreads();
    const int above = pass == 0 ? 32 : kRankShift[pass - 1];     // the bits decided so far must agree
    for (int64_t base = (int64_t)blockIdx.x * (U * kRankBlock); base < a.N; base += (int64_t)gridDim.x * (U * kRankBlock)) {
        uint32_t b[U];
#pragma unroll
        for (int k = 0; k < U; ++k) b[k] = candidate_bits(a, base + k * kRankBlock + threadIdx.x);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (b[k] != 0u && (pass == 0 || (b[k] >> above) == (from >> above)))
                atomicAdd(&h[threadIdx.x % kCopies][(b[k] >> shift) & (uint32_t)(nb - 1)], 1u);
    }
    __syncthreads();
    uint32_t* out = a.hist + (pass == 0 ? 0 : pass == 1 ? 2048 : 3072);
    for (int i = threadIdx.x; i < nb; i += kRankBlock) {
        uint32_t c = 0;
#pragma unroll
        for (int k = 0; k < kCopies; ++k) c += h[k][i];
        if (c) atomicAdd(&out[i], c);
    }
}

// The candidates that are kept, in ascending id order: a workgroup takes a run of whole tiles of kRankTile ids, first to count
// its own (and to leave the threshold, and for the host their number), then to place them behind those of the workgroups before it.
// 8M scores, 320k of them kept: 14 + 4 + 24 us as a scan by a general grid scan, which asked for one score per thread at a time.
constexpr int kRankPer = 8, kRankTile = kRankPer * kRankBlock, kRankGroups = 256;
struct RankRun {
    int64_t beg, end;
    __device__ __forceinline__ explicit RankRun(int64_t N) {
        const int64_t tiles = (N + kRankTile - 1) / kRankTile, per = (tiles + gridDim.x - 1) / gridDim.x * kRankTile;
        beg = (int64_t)blockIdx.x * per;
        end = beg + per < N ? beg + per : N;
    }
};
__global__ void __launch_bounds__(kRankBlock) rank_count_kernel(RankArgs a, uint32_t* __restrict__ from, uint32_t* __restrict__ count,
                                                                int64_t* __restrict__ total) {
    __shared__ RankLds l;
    uint64_t kept;
    uint32_t bits = kept_from(a, 3, l, kept);
    if (bits == kTooFew) bits = 1u;
    if (blockIdx.x == 0 && threadIdx.x == 0) { *from = bits; *total = (int64_t)kept; }
    const RankRun run(a.N);
    uint32_t mine = 0;
    for (int64_t base = run.beg; base < run.end; base += kRankTile) {
        uint32_t b[kRankPer];
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) b[k] = candidate_bits(a, base + k * kRankBlock + threadIdx.x);
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) mine += b[k] >= bits ? 1u : 0u;
    }
    mine = (uint32_t)wave_sum((int)mine);
    __syncthreads();
    if (lane_id() == 0) l.sums[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kRankWaves; ++w) mine += l.sums[w];
        count[blockIdx.x] = mine;
    }
}
__global__ void __launch_bounds__(kRankBlock) rank_place_kernel(RankArgs a, const uint32_t* __restrict__ from,
                                                                const uint32_t* __restrict__ count, uint64_t* __restrict__ keys) {
    __shared__ uint32_t sums[2][kRankWaves];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const uint32_t bits = *from;
    uint32_t at = 0;                             // where the workgroup's next one goes
    {
        const uint32_t x = (int)threadIdx.x < (int)blockIdx.x ? count[threadIdx.x] : 0u;     // at most kRankGroups of them
        const uint32_t s = (uint32_t)wave_sum((int)x);
        if (lane == 0) sums[0][wave] = s;
        __syncthreads();
        for (int w = 0; w < kRankWaves; ++w) at += sums[0][w];
    }
    const RankRun run(a.N);
    for (int64_t base = run.beg; base < run.end; base += kRankTile) {
        // a wavefront takes kRankPer times 64 consecutive ids
        const int64_t u0 = base + wave * (kWave * kRankPer) + lane;
        uint32_t b[kRankPer];
        uint64_t has[kRankPer];
        uint32_t mine = 0;
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) b[k] = candidate_bits(a, u0 + k * kWave);
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) {
            has[k] = __ballot(b[k] >= bits);
            mine += (uint32_t)__popcll(has[k]);
        }
        __syncthreads();                         // the sums of the tile before have been read
        if (lane == 0) sums[1][wave] = mine;
        __syncthreads();
        uint32_t to = at;
        for (int w = 0; w < kRankWaves; ++w) {
            const uint32_t x = sums[1][w];
            to += w < wave ? x : 0u;
            at += x;
        }
#pragma unroll
        for (int k = 0; k < kRankPer; ++k) {
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(has[k] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has[k], 0u));
            if (b[k] >= bits) keys[to + below] = ((uint64_t)~b[k] << 32) | (uint32_t)(u0 + k * kWave);
            to += (uint32_t)__popcll(has[k]);
        }
    }
}

// Up to kSmallRank keys in one workgroup: a bitonic network in LDS over the whole keys (ids make them
// distinct), padded with all ones.  A ranking of 4000 keys out of 20k 105 us, as by the eight launches of the radix sort; of 8000
// out of 40k 148, and 101 by radix.
constexpr int kSmallRank = 4096;
constexpr int kSmallBlock = 1024;
__global__ void __launch_bounds__(kSmallBlock) rank_small_kernel(uint64_t* __restrict__ keys, int n, int size) {
    extern __shared__ unsigned long long small_keys[];
    for (int i = threadIdx.x; i < size; i += kSmallBlock) small_keys[i] = i < n ? keys[i] : ~0ull;
    __syncthreads();
    for (int k = 2; k <= size; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < size / 2; t += kSmallBlock) {
                const int i = 2 * t - (t & (j - 1)), o = i + j;      // the t-th pair at distance j
                const unsigned long long x = small_keys[i], y = small_keys[o];
                if ((x > y) == ((i & k) == 0)) { small_keys[i] = y; small_keys[o] = x; }
            }
            __syncthreads();
        }
    for (int i = threadIdx.x; i < n; i += kSmallBlock) keys[i] = small_keys[i];
}

__global__ void __launch_bounds__(kBlock) cache_fill_kernel(const uint64_t* __restrict__ sorted, int64_t n,
                                                            int64_t lo, int64_t hi, int32_t* __restrict__ ids,
                                                            int64_t* __restrict__ rowidx,
                                                            unsigned long long* __restrict__ tab, uint32_t mask,
                                                            int shift) {
    const int64_t r = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= n) return;
    const uint32_t id = (uint32_t)sorted[r];
    ids[r] = (int32_t)id;
    rowidx[r] = (int64_t)id < lo ? (int64_t)id : (int64_t)id - (hi - lo);
    table_insert_min(tab, mask, shift, id, (uint32_t)r);
}

__global__ void fill_table_kernel(unsigned long long* p, int64_t n, unsigned long long v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

__global__ void __launch_bounds__(kBlock) cache_lookup_kernel(const unsigned long long* __restrict__ tab,
                                                              uint32_t mask, int shift, int64_t limit,
                                                              const int32_t* __restrict__ ids, int64_t n,
                                                              int32_t* __restrict__ out) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        uint32_t slot = 0;
        const int32_t g = ids[i];
        const bool found = tab && g >= 0 && table_find(tab, mask, shift, (uint32_t)g, slot) >= 0 && (int64_t)slot < limit;
        out[i] = found ? (int32_t)slot : -1;
    }
}

// Empirical access frequencies (Sec. 3.2, "sim." and "oracle" policies): one count per listed id.
// Ids of one minibatch are distinct and the lists of a call are few, so the float atomics rarely
// meet on one address.
struct CountLists {
    const int32_t* ids[SPP_MAX_GATHER_LISTS];
    int64_t        n[SPP_MAX_GATHER_LISTS];
    const int64_t* n_ptr[SPP_MAX_GATHER_LISTS];
};
__global__ void clear_flag_kernel(int* flag) { if (threadIdx.x == 0) *flag = 0; }

__global__ void __launch_bounds__(kBlock) access_count_kernel(CountLists l, int64_t N, float* __restrict__ count,
                                                              int* __restrict__ bad) {
    const int j = blockIdx.y;
    int64_t n = l.n_ptr[j] ? *l.n_ptr[j] : l.n[j];
    if (n > l.n[j]) n = l.n[j];                       // never beyond what the caller's buffer holds
    const int32_t* __restrict__ ids = l.ids[j];
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
        const int64_t g = ids[i];
        if (g < 0 || g >= N) atomicOr(bad, 1);
        else unsafeAtomicAdd(&count[g], 1.0f);
    }
}

}  // namespace spp

extern "C" int spp_access_count(spp_ctx* ctx, const spp_id_list* lists, int32_t n_lists, int64_t N, float* d_count,
                                uint32_t flags) {
    using namespace spp;
    SPP_CHECK(ctx && d_count && (lists || n_lists == 0), SPP_E_ARG, "spp_access_count: null argument");
    SPP_CHECK(n_lists >= 0 && n_lists <= SPP_MAX_GATHER_LISTS, SPP_E_ARG, "spp_access_count: %d lists (at most %d)",
              n_lists, SPP_MAX_GATHER_LISTS);
    SPP_CHECK(N > 0, SPP_E_ARG, "spp_access_count: N = %lld", (long long)N);
    if (n_lists == 0) return SPP_OK;
    CountLists l;
    memset(&l, 0, sizeof(l));
    int64_t nmax = 0;
    for (int j = 0; j < n_lists; ++j) {
        SPP_CHECK(lists[j].n >= 0 && (lists[j].d_ids || lists[j].n == 0), SPP_E_ARG, "spp_access_count: list %d", j);
        l.ids[j] = lists[j].d_ids; l.n[j] = lists[j].n; l.n_ptr[j] = lists[j].d_n;
        if (lists[j].n > nmax) nmax = lists[j].n;
    }
    if (nmax == 0) return SPP_OK;
    SPP_HIP(hipSetDevice(ctx->device));
    hipStream_t st = ctx->stream;
    SPP_TRY(ctx->partials.reserve(256));
    int* d_bad = ctx->partials.as<int>();
    clear_flag_kernel<<<1, 64, 0, st>>>(d_bad);
    const int64_t need = (nmax + kBlock - 1) / kBlock;
    const int64_t lim = (int64_t)ctx->num_cu * 8 / n_lists + 1;
    access_count_kernel<<<dim3((unsigned)(need < lim ? need : lim), n_lists), kBlock, 0, st>>>(l, N, d_count, d_bad);
    SPP_HIP(hipGetLastError());
    if (flags & SPP_SYNC) {
        int* hb = reinterpret_cast<int*>(ctx->h_pinned + 60);
        SPP_HIP(hipMemcpyAsync(hb, d_bad, sizeof(int), hipMemcpyDeviceToHost, st));
        SPP_HIP(hipStreamSynchronize(st));
        SPP_CHECK(*hb == 0, SPP_E_ARG, "spp_access_count: an id lies outside [0, N); it was skipped");
    }
    return SPP_OK;
}

extern "C" int spp_build_vip_cache(spp_ctx* ctx, const float* d_score, int64_t N, int64_t lo, int64_t hi,
                                   int32_t K, double alpha, const void* remote, int32_t D,
                                   int32_t elem_bytes, int32_t* d_cache_ids, int64_t* n_cached,
                                   spp_cache** out) {
    using namespace spp;
    SPP_CHECK(ctx && d_score && n_cached && out, SPP_E_ARG, "spp_build_vip_cache: null argument");
    *out = nullptr; *n_cached = 0;
    SPP_CHECK(N > 0 && N <= 0x7FFFFFFFll && lo >= 0 && lo <= hi && hi <= N, SPP_E_ARG,
              "spp_build_vip_cache: range [%lld, %lld) of N = %lld", (long long)lo, (long long)hi, (long long)N);
    SPP_CHECK(K >= 1 && alpha >= 0.0 && alpha == alpha, SPP_E_ARG, "spp_build_vip_cache: K = %d, alpha = %g", K, alpha);
    SPP_CHECK(D >= 1 && elem_bytes >= 1 && ((int64_t)D * elem_bytes) % 2 == 0, SPP_E_ARG,
              "spp_build_vip_cache: D = %d, elem_bytes = %d", D, elem_bytes);
    const int64_t C = (int64_t)floor(alpha * (double)N / (double)K);
    SPP_CHECK(C == 0 || d_cache_ids, SPP_E_ARG, "spp_build_vip_cache: d_cache_ids is null");
    SPP_HIP(hipSetDevice(ctx->device));
    hipStream_t st = ctx->stream;

    spp_cache* c = new (std::nothrow) spp_cache();
    SPP_CHECK(c != nullptr, SPP_E_OOM, "spp_build_vip_cache: out of host memory");
    c->device = ctx->device; c->N = N; c->lo = lo; c->hi = hi; c->row_bytes = (int64_t)D * elem_bytes;

    int rc = SPP_OK;
    uint64_t* sorted = nullptr;
    DevBuf own;                        // keys of a ranking too large to stay with the context
    const int64_t max_cand = N - (hi - lo);
    int64_t nsel = 0, keep = 0;

    auto fail = [&](int code) { rc = code; };
    do {
        if (C == 0 || max_cand == 0) break;
        // head of the workspace: histograms, threshold, the workgroups' counts; then two arrays of keys and the rows
        const size_t head = ((size_t)kRankHistWords + 2 + kRankGroups) * sizeof(uint32_t);
        rc = ctx->rankws.reserve(head);
        if (rc != SPP_OK) break;
        RankArgs ra;
        ra.score = d_score; ra.N = N; ra.lo = lo; ra.hi = hi; ra.C = (uint64_t)C;
        ra.hist = ctx->rankws.as<uint32_t>();
        uint32_t* from = ra.hist + kRankHistWords;
        uint32_t* count = from + 2;
        const int64_t tiles = (N + kRankTile - 1) / kRankTile;
        const int hgrid = (int)(tiles < (int64_t)ctx->num_cu ? tiles : (int64_t)ctx->num_cu);
        const int rgrid = hgrid < kRankGroups ? hgrid : kRankGroups;
        fill_table_kernel<<<8, kBlock, 0, st>>>(reinterpret_cast<unsigned long long*>(ra.hist), kRankHistWords / 2, 0ull);
        for (int pass = 0; pass < 3; ++pass) rank_hist_kernel<<<hgrid, kRankBlock, 0, st>>>(ra, pass);
        // how many are kept decides the room for their keys
        int64_t* hp = ctx->h_pinned + 61;
        rank_count_kernel<<<rgrid, kRankBlock, 0, st>>>(ra, from, count, hp);
        if (hipStreamSynchronize(st) != hipSuccess) { set_error("spp_build_vip_cache: candidate scan failed: %s", hipGetErrorString(hipGetLastError())); fail(SPP_E_HIP); break; }
        nsel = *hp;                    // ties at the threshold included
        if (nsel == 0) break;
        keep = nsel < C ? nsel : C;
        const size_t keys_at = (head + 255) / 256 * 256, need = keys_at + (size_t)nsel * 2 * sizeof(uint64_t) + (size_t)keep * sizeof(int64_t);
        char* base = nullptr;
        if (need <= kKeptSortBytes) {
            // grown in place of the head: its threshold and sums move along
            if (ctx->rankws.bytes < need) {
                DevBuf grown;
                rc = grown.reserve(need);
                if (rc != SPP_OK) break;
                if (hipMemcpyAsync(grown.ptr, ctx->rankws.ptr, head, hipMemcpyDeviceToDevice, st) != hipSuccess) { set_error("spp_build_vip_cache: copy failed"); grown.release(); fail(SPP_E_HIP); break; }
                ctx->rankws.release();           // waits for the copy
                ctx->rankws = grown;
                ra.hist = ctx->rankws.as<uint32_t>();
                from = ra.hist + kRankHistWords;
                count = from + 2;
            }
            base = ctx->rankws.as<char>();
        } else {
            rc = own.reserve(need);
            if (rc != SPP_OK) break;
            base = own.as<char>();
        }
        uint64_t* ka = reinterpret_cast<uint64_t*>(base + keys_at);
        uint64_t* kb = ka + nsel;
        int64_t* rowidx = reinterpret_cast<int64_t*>(kb + nsel);
        rank_place_kernel<<<rgrid, kRankBlock, 0, st>>>(ra, from, count, ka);
        if (nsel <= kSmallRank) {
            int size = 2;
            while (size < nsel) size <<= 1;
            rank_small_kernel<<<1, kSmallBlock, (size_t)size * sizeof(uint64_t), st>>>(ka, (int)nsel, size);
            sorted = ka;
        } else {
            rc = radix_sort_u64(ctx, ka, kb, nsel, 32, 64, &sorted);
            if (rc != SPP_OK) break;
        }
        const uint32_t cap = next_pow2((uint64_t)(2 * keep > 1024 ? 2 * keep : 1024));
        int shift = 32;
        for (uint32_t t = cap; t > 1; t >>= 1) --shift;
        c->table_mask = cap - 1; c->table_shift = shift;
        if (pool_take(c->device, &c->table, (size_t)cap * sizeof(uint64_t)) != hipSuccess) {
            set_error("spp_build_vip_cache: out of device memory for the id table"); fail(SPP_E_OOM); break;
        }
        fill_table_kernel<<<ctx->num_cu * 4, kBlock, 0, st>>>(reinterpret_cast<unsigned long long*>(c->table), cap, ~0ull);
        cache_fill_kernel<<<(unsigned)((keep + kBlock - 1) / kBlock), kBlock, 0, st>>>(
            sorted, keep, lo, hi, d_cache_ids, rowidx, reinterpret_cast<unsigned long long*>(c->table), c->table_mask, shift);
        if (remote) {
            if (pool_take(c->device, &c->rows, (size_t)keep * (size_t)c->row_bytes) != hipSuccess) {
                set_error("spp_build_vip_cache: out of device memory for %lld cached rows", (long long)keep); fail(SPP_E_OOM); break;
            }
            rc = copy_rows_indexed(st, remote, rowidx, keep, c->row_bytes, c->rows, ctx->num_cu);
            if (rc != SPP_OK) break;
        }
        if (hipStreamSynchronize(st) != hipSuccess) { set_error("spp_build_vip_cache: %s", hipGetErrorString(hipGetLastError())); fail(SPP_E_HIP); break; }
    } while (0);

    if (own.ptr) { (void)hipStreamSynchronize(st); own.release(); }
    if (rc != SPP_OK) { spp_cache_destroy(c); return rc; }
    c->n_rows = keep; c->limit = keep;
    *n_cached = keep;
    *out = c;
    return SPP_OK;
}

extern "C" void spp_cache_destroy(spp_cache* c) {
    if (!c) return;
    if (hipSetDevice(c->device) != hipSuccess) { (void)hipGetLastError(); delete c; return; }   // runtime already shut down
    spp::pool_retire(c->device, {c->table, c->rows});        // a gather that still reads the cache may be in flight
    delete c;
}

extern "C" int spp_cache_set_limit(spp_cache* c, int64_t n_slots) {
    SPP_CHECK(c, SPP_E_ARG, "spp_cache_set_limit: cache is null");
    SPP_CHECK(n_slots <= c->n_rows, SPP_E_ARG, "spp_cache_set_limit: %lld slots asked, %lld built", (long long)n_slots, (long long)c->n_rows);
    c->limit = n_slots < 0 ? c->n_rows : n_slots;
    return SPP_OK;
}

extern "C" int spp_cache_lookup(spp_ctx* ctx, const spp_cache* c, const int32_t* d_ids, int64_t n,
                                int32_t* d_slot_out) {
    using namespace spp;
    SPP_CHECK(ctx && c && (n == 0 || (d_ids && d_slot_out)), SPP_E_ARG, "spp_cache_lookup: null argument");
    if (n == 0) return SPP_OK;
    SPP_HIP(hipSetDevice(ctx->device));
    const int64_t need = (n + kBlock - 1) / kBlock;
    const int grid = (int)(need < (int64_t)ctx->num_cu * 8 ? need : (int64_t)ctx->num_cu * 8);
    // an empty cache has no table: every id misses
    cache_lookup_kernel<<<grid, kBlock, 0, ctx->stream>>>(reinterpret_cast<const unsigned long long*>(c->table),
                                                          c->table_mask, c->table_shift, c->limit, d_ids, n, d_slot_out);
    SPP_HIP(hipGetLastError());
    return SPP_OK;
}
