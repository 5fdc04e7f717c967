// Stable least-significant-digit radix sort of 64-bit keys, 8 bits per pass, used at set-up time:
// to build the chunked transposed edge structure and to rank cache candidates and local vertices
// (Sec. 3.2).
//
// A tile is 4096 keys (1024 where the keys do not make four tiles of 4096 per CU, so that every CU has some;
// up to 1M keys take the form with two launches per pass below) handled by one 256-thread workgroup; wavefront w owns the w-th quarter of
// the tile and walks it in order, 64 keys at a time, so a key's stable rank among equal digits is
// (count of that digit in earlier wavefronts' quarters) + (count earlier in its own quarter) +
// (count in lower lanes of its own 64), the last from ballots.  Keys are then placed in digit
// order in LDS and written out as per-digit runs.
#include "spp_common.h"
#include "spp_device.h"

namespace spp {

template <int kTile>
__global__ void __launch_bounds__(kBlock) radix_hist_kernel(const uint64_t* __restrict__ keys, int64_t n,
                                                            int shift, int64_t ntiles,
                                                            uint32_t* __restrict__ hist) {
    __shared__ uint32_t h[256];
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        h[threadIdx.x] = 0;
        __syncthreads();
        const int64_t base = tile * kTile;
        for (int k = threadIdx.x; k < kTile; k += kBlock) {
            int64_t i = base + k;
            if (i < n) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & 255u], 1u);
        }
        __syncthreads();
        hist[(int64_t)threadIdx.x * ntiles + tile] = h[threadIdx.x];
        __syncthreads();
    }
}

struct HistIn  { const uint32_t* h; __device__ int operator()(int64_t i) const { return (int)h[i]; } };
struct HistOut { uint32_t* h; __device__ void operator()(int64_t i, int ex, int) const { h[i] = (uint32_t)ex; } };
struct NoFin   { __device__ void operator()(int) const {} };

template <int kTile>
__global__ void __launch_bounds__(kBlock) radix_scatter_kernel(const uint64_t* __restrict__ keys,
                                                               uint64_t* __restrict__ out, int64_t n,
                                                               int shift, int64_t ntiles,
                                                               const uint32_t* __restrict__ offs) {
    constexpr int kPerWave = kTile / 4, kBatches = kPerWave / kWave;         // batches of 64 per wavefront
    __shared__ uint32_t cnt[4][256];
    __shared__ uint32_t dstart[256];
    __shared__ uint32_t gbase[256];
    __shared__ uint64_t sorted[kTile];
    __shared__ int scan_lds[4];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        for (int w = 0; w < 4; ++w) cnt[w][threadIdx.x] = 0;
        __syncthreads();

        uint64_t key[kBatches];
        uint16_t rnk[kBatches];
        const int64_t wbase = tile * kTile + (int64_t)wave * kPerWave;
#pragma unroll
        for (int b = 0; b < kBatches; ++b) {
            const int64_t i = wbase + b * kWave + lane;
            const bool valid = i < n;
            const uint64_t k = valid ? keys[i] : 0ull;
            const uint32_t d = (uint32_t)(k >> shift) & 255u;
            uint64_t m = __ballot(valid);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const bool one = (d >> bit) & 1u;
                const uint64_t bm = __ballot(valid && one);
                m &= one ? bm : ~bm;
            }
            const uint32_t below = (uint32_t)__popcll(m & lt_mask);
            uint32_t prior = 0;
            if (valid) prior = cnt[wave][d];
            wave_lds_order();
            if (valid && below == 0) cnt[wave][d] = prior + (uint32_t)__popcll(m);
            wave_lds_order();
            key[b] = k;
            rnk[b] = (uint16_t)(prior + below);
        }
        __syncthreads();

        {   // digit totals -> start of each digit's run in the tile, and per-wavefront offsets
            const int d = threadIdx.x;
            const uint32_t c0 = cnt[0][d], c1 = cnt[1][d], c2 = cnt[2][d], c3 = cnt[3][d];
            int total;
            const int ex = block_exclusive_scan((int)(c0 + c1 + c2 + c3), scan_lds, total);
            dstart[d] = (uint32_t)ex;
            cnt[0][d] = (uint32_t)ex;
            cnt[1][d] = (uint32_t)ex + c0;
            cnt[2][d] = (uint32_t)ex + c0 + c1;
            cnt[3][d] = (uint32_t)ex + c0 + c1 + c2;
            gbase[d] = offs[(int64_t)d * ntiles + tile];
        }
        __syncthreads();

#pragma unroll
        for (int b = 0; b < kBatches; ++b) {
            const int64_t i = wbase + b * kWave + lane;
            if (i < n) {
                const uint32_t d = (uint32_t)(key[b] >> shift) & 255u;
                sorted[cnt[wave][d] + rnk[b]] = key[b];
            }
        }
        __syncthreads();

        const int64_t left = n - tile * kTile;
        const int count = left < kTile ? (int)left : kTile;
        for (int k = threadIdx.x; k < count; k += kBlock) {
            const uint64_t v = sorted[k];
            const uint32_t d = (uint32_t)(v >> shift) & 255u;
            out[(uint64_t)gbase[d] + (uint32_t)(k - dstart[d])] = v;
        }
        __syncthreads();
    }
}

// The same with two launches per pass instead of five, for up to kMidTiles tiles: a tile's counts lie side by side, and the
// workgroup that places a tile adds up those of all tiles for itself.  What bounds it is the chain of dependent steps in a
// launch and the launches themselves, so a workgroup has 1024 threads with kBatches keys each.  320k keys, a pass: 12 us, where
// the five launches take 22 and the gaps between them; 1M keys a call of 360 us takes 249.  With more tiles than that the
// workgroups' reads of each other's counts grow with the square of their number.
constexpr int kMidBlock = 1024, kMidWaves = kMidBlock / kWave, kMidTiles = 256;
template <int kBatches>
__global__ void __launch_bounds__(kMidBlock) radix_mid_hist_kernel(const uint64_t* __restrict__ keys, int64_t n, int shift,
                                                                   uint32_t* __restrict__ hist) {
    constexpr int kCopies = kMidBlock / 256;     // neighbouring lanes add to different ones
    __shared__ uint32_t h[kCopies][256];
    (&h[0][0])[threadIdx.x] = 0u;
    const int64_t i0 = (int64_t)blockIdx.x * (kMidBlock * kBatches) + threadIdx.x;
    uint32_t d[kBatches];
#pragma unroll
    for (int b = 0; b < kBatches; ++b) d[b] = (uint32_t)(keys[i0 + b * kMidBlock < n ? i0 + b * kMidBlock : n - 1] >> shift) & 255u;
    __syncthreads();
#pragma unroll
    for (int b = 0; b < kBatches; ++b)
        if (i0 + b * kMidBlock < n) atomicAdd(&h[threadIdx.x % kCopies][d[b]], 1u);
    __syncthreads();
    if (threadIdx.x < 256) {
        uint32_t c = 0;
#pragma unroll
        for (int k = 0; k < kCopies; ++k) c += h[k][threadIdx.x];
        hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = c;
    }
}
template <int kBatches>
__global__ void __launch_bounds__(kMidBlock) radix_mid_scatter_kernel(const uint64_t* __restrict__ keys, uint64_t* __restrict__ out,
                                                                      int64_t n, int shift, const uint32_t* __restrict__ hist) {
    constexpr int kTile = kMidBlock * kBatches, kGroups = kMidBlock / 256;
    __shared__ uint32_t cnt[kMidWaves][256];
    __shared__ uint32_t all[kGroups][256], before[kGroups][256];     // per digit, from every kGroups-th tile: all of them, those before this one
    __shared__ uint32_t dstart[256], gbase[256];
    __shared__ uint32_t sums[2][256 / kWave];
    __shared__ uint64_t sorted[kTile];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = lane_id();
    const int tile = (int)blockIdx.x, ntiles = (int)gridDim.x;
    const int64_t wbase = (int64_t)tile * kTile + wave * (kWave * kBatches) + lane;
    uint64_t key[kBatches];
#pragma unroll
    for (int b = 0; b < kBatches; ++b) key[b] = keys[wbase + b * kWave < n ? wbase + b * kWave : n - 1];
    {
        const int d = threadIdx.x & 255, group = threadIdx.x >> 8;
        uint32_t a = 0, f = 0;
#pragma unroll 16
        for (int t = group; t < ntiles; t += kGroups) {
            const uint32_t c = hist[t * 256 + d];
            a += c;
            f += t < tile ? c : 0u;
        }
        all[group][d] = a;
        before[group][d] = f;
    }
#pragma unroll
    for (int k = 0; k < 256 / kWave; ++k) cnt[wave][k * kWave + lane] = 0u;      // the wavefront's own
    wave_lds_order();
    uint32_t rnk[kBatches];
#pragma unroll
    for (int b = 0; b < kBatches; ++b) {
        const bool valid = wbase + b * kWave < n;
        const uint32_t d = (uint32_t)(key[b] >> shift) & 255u;
        const uint64_t same = lanes_alike<8>(valid, d);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        const uint32_t prior = cnt[wave][d];
        wave_lds_order();                        // the lanes alike have read it
        if (valid && below == 0) cnt[wave][d] = prior + (uint32_t)__popcll(same);
        wave_lds_order();                        // before the next 64 read it
        rnk[b] = prior + below;
    }
    __syncthreads();
    // per digit: where the tile's run of it starts in the tile, every wavefront's part of that, and where it goes
    const int d = threadIdx.x & 255;
    uint32_t mine = 0, total = 0, mine_inc = 0, total_inc = 0;
    if (threadIdx.x < 256) {
#pragma unroll
        for (int w = 0; w < kMidWaves; ++w) mine += cnt[w][d];
#pragma unroll
        for (int k = 0; k < kGroups; ++k) total += all[k][d];
        mine_inc = (uint32_t)wave_inclusive_scan((int)mine);
        total_inc = (uint32_t)wave_inclusive_scan((int)total);
        if (lane == kWave - 1) { sums[0][wave] = mine_inc; sums[1][wave] = total_inc; }
    }
    __syncthreads();
    if (threadIdx.x < 256) {
        uint32_t at = mine_inc - mine, to = total_inc - total;
        for (int w = 0; w < wave; ++w) { at += sums[0][w]; to += sums[1][w]; }
#pragma unroll
        for (int k = 0; k < kGroups; ++k) to += before[k][d];
        dstart[d] = at;
        gbase[d] = to;
#pragma unroll
        for (int w = 0; w < kMidWaves; ++w) {
            const uint32_t c = cnt[w][d];
            cnt[w][d] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < kBatches; ++b)
        if (wbase + b * kWave < n) sorted[cnt[wave][(uint32_t)(key[b] >> shift) & 255u] + rnk[b]] = key[b];
    __syncthreads();
    const int64_t left = n - (int64_t)tile * kTile;
    const int count = left < kTile ? (int)left : kTile;
    for (int k = threadIdx.x; k < count; k += kMidBlock) {
        const uint64_t v = sorted[k];
        const uint32_t dv = (uint32_t)(v >> shift) & 255u;
        out[gbase[dv] + ((uint32_t)k - dstart[dv])] = v;
    }
}

template <int kBatches>
static int sort_mid(spp_ctx* ctx, uint64_t* src, uint64_t* dst, int64_t n, int bit_lo, int bit_hi, uint64_t** result) {
    hipStream_t st = ctx->stream;
    const int ntiles = (int)((n + kMidBlock * kBatches - 1) / (kMidBlock * kBatches));       // at most kMidTiles
    SPP_TRY(ctx->sortws.reserve((size_t)ntiles * 256 * sizeof(uint32_t)));
    uint32_t* hist = ctx->sortws.as<uint32_t>();
    for (int shift = bit_lo; shift < bit_hi; shift += 8) {
        radix_mid_hist_kernel<kBatches><<<ntiles, kMidBlock, 0, st>>>(src, n, shift, hist);
        radix_mid_scatter_kernel<kBatches><<<ntiles, kMidBlock, 0, st>>>(src, dst, n, shift, hist);
        uint64_t* t = src; src = dst; dst = t;
    }
    *result = src;
    SPP_HIP(hipGetLastError());
    return SPP_OK;
}

template <int kTile>
static int sort_tiles(spp_ctx* ctx, uint64_t* src, uint64_t* dst, int64_t n, int bit_lo, int bit_hi, uint64_t** result) {
    hipStream_t st = ctx->stream;
    const int64_t ntiles = (n + kTile - 1) / kTile;
    const int64_t nhist = 256 * ntiles;
    const int scan_grid = (int)(nhist / 2048 < 1 ? 1 : (nhist / 2048 < 1024 ? nhist / 2048 : 1024));
    const size_t bytes = (size_t)nhist * sizeof(uint32_t) + (size_t)scan_grid * sizeof(int);
    // the counts of a large sort are not kept
    DevBuf own;
    DevBuf& ws = bytes <= kKeptSortBytes ? ctx->sortws : own;
    SPP_TRY(ws.reserve(bytes));
    uint32_t* hist = ws.as<uint32_t>();
    int* partial = reinterpret_cast<int*>(hist + nhist);
    const int grid = (int)(ntiles < (int64_t)ctx->num_cu * 8 ? ntiles : (int64_t)ctx->num_cu * 8);
    for (int shift = bit_lo; shift < bit_hi; shift += 8) {
        radix_hist_kernel<kTile><<<grid, kBlock, 0, st>>>(src, n, shift, ntiles, hist);
        grid_scan(st, scan_grid, nhist, HistIn{hist}, HistOut{hist}, NoFin{}, partial);
        radix_scatter_kernel<kTile><<<grid, kBlock, 0, st>>>(src, dst, n, shift, ntiles, hist);
        uint64_t* t = src; src = dst; dst = t;
    }
    *result = src;
    hipError_t e = hipGetLastError();
    if (own.ptr) {
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        own.release();
    }
    if (e != hipSuccess) { set_error("radix_sort_u64: %s", hipGetErrorString(e)); return SPP_E_HIP; }
    return SPP_OK;
}

// The sorted keys are complete on the context's stream; the host has not waited for them.
int radix_sort_u64(spp_ctx* ctx, uint64_t* keys_a, uint64_t* keys_b, int64_t n, int bit_lo, int bit_hi,
                   uint64_t** result) {
    *result = keys_a;
    if (n <= 1 || bit_hi <= bit_lo) return SPP_OK;
    SPP_CHECK(n < (int64_t)0xFFFFFFFFll, SPP_E_ARG, "radix_sort_u64: %lld keys exceed the 32-bit offset range",
              (long long)n);
    if (n <= (int64_t)kMidTiles * kMidBlock * 2) return sort_mid<2>(ctx, keys_a, keys_b, n, bit_lo, bit_hi, result);
    if (n <= (int64_t)kMidTiles * kMidBlock * 4) return sort_mid<4>(ctx, keys_a, keys_b, n, bit_lo, bit_hi, result);
    return n < (int64_t)ctx->num_cu * 4 * 4096 ? sort_tiles<1024>(ctx, keys_a, keys_b, n, bit_lo, bit_hi, result)
                                               : sort_tiles<4096>(ctx, keys_a, keys_b, n, bit_lo, bit_hi, result);
}

}  // namespace spp
