// Scans and the stable LSD radix sort used for the centre-depth order and for
// bucketing (tile, surfel) pairs by tile (Sec. 3.2 "Rasterization": sort by centre
// depth, organise into tiles).
//
// Radix sort: 8-bit digits, 256 threads x 16 items = 4096 items per block.
//   hist    : per-block digit histogram in LDS -> hist[digit * nblocks + block], or per
//             segment (below)
//   scan    : exclusive scan of hist (digit-major) -> global base of (digit, block)
//   scatter : per-wave stable multisplit through a table of lane masks and counts in LDS
//             (rank_rows), then a prefix over the 4 waves places each digit's run inside the
//             block.
// Tile bucketing sorts within segments (one per view) on key minus the segment's base,
// so the number of passes follows the largest view's tile count; its last pass also
// writes each tile's [begin, end) range.
// Item counts may live in device memory (pair counts are data dependent), so grids
// are sized by capacity and blocks past the live count exit at once.
#include "ss_internal.h"
#include <algorithm>

namespace ss {

constexpr int kSortThreads = 256;
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortThreads * kSortItems;   // 4096
constexpr int kSortWaves = kSortThreads / kWave;

__device__ __forceinline__ int64_t live_count(const unsigned long long *n_dev, int64_t cap,
                                              int64_t n_host)
{
    if (!n_dev) return n_host;
    unsigned long long n = *n_dev;
    return n < (unsigned long long)cap ? (int64_t)n : cap;
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t count)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) p[i] = v;
}

hipError_t fill_u32(uint32_t *p, uint32_t value, int64_t count, hipStream_t st)
{
    if (count <= 0) return hipSuccess;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, value, count);
    return hipGetLastError();
}

__global__ void k_reset_pass(uint32_t *flag, unsigned long long *stat, unsigned long long *extra)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kStatSlots * kStatStride) stat[i] = 0ull;
    if (i == 0) {
        *flag = 0u;
        if (extra) *extra = 0ull;
    }
}

hipError_t reset_pass(uint32_t *flag, unsigned long long *stat, unsigned long long *extra, hipStream_t st)
{
    hipLaunchKernelGGL(k_reset_pass, dim3((kStatSlots * kStatStride + 255) / 256), dim3(256), 0, st, flag,
                       stat, extra);
    return hipGetLastError();
}

hipError_t fill_f32(float *p, float value, int64_t count, hipStream_t st)
{
    union { float f; uint32_t u; } cv;
    cv.f = value;
    return fill_u32(reinterpret_cast<uint32_t *>(p), cv.u, count, st);
}

// ------------------------------------------------------------- pair-count scan
// Each thread owns kSortItems consecutive entries; full groups are moved as uint4 (the
// arrays start 256-byte aligned and a group starts at a multiple of 16 entries).
__device__ __forceinline__ void load_items(const uint32_t *in, int64_t base, int64_t len,
                                           uint32_t (&v)[kSortItems])
{
    if (base + kSortItems <= len) {
        const uint4 *p = reinterpret_cast<const uint4 *>(in + base);
#pragma unroll
        for (int q = 0; q < kSortItems / 4; ++q) {
            const uint4 x = p[q];
            v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kSortItems; ++i) v[i] = base + i < len ? in[base + i] : 0u;
    }
}

__device__ __forceinline__ void store_items(uint32_t *out, int64_t base, int64_t len,
                                            const uint32_t (&v)[kSortItems])
{
    if (base + kSortItems <= len) {
        uint4 *p = reinterpret_cast<uint4 *>(out + base);
#pragma unroll
        for (int q = 0; q < kSortItems / 4; ++q)
            p[q] = make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < kSortItems; ++i)
            if (base + i < len) out[base + i] = v[i];
    }
}

__global__ void k_scan_reduce(const uint32_t *in, int64_t len, uint32_t *partials)
{
    __shared__ unsigned long long lds[kSortWaves];
    int64_t base = (int64_t)blockIdx.x * kSortTile + (int64_t)threadIdx.x * kSortItems;
    uint32_t v[kSortItems];
    load_items(in, base, len, v);
    unsigned long long s = 0;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) s += v[i];
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) lds[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kSortWaves; ++k) s += lds[k];
        partials[blockIdx.x] = (uint32_t)min(s, 0xFFFFFFFFull);
    }
}

// One block: exclusive scan in place in 64-bit (results clamped to 2^32 - 1), overflow
// detection.
constexpr int kScanPartialsThreads = 1024;
constexpr int kScanPartialsItems = 8;
constexpr int kScanOneBlock = 2 * kScanPartialsThreads * kScanPartialsItems;

__global__ __launch_bounds__(kScanPartialsThreads) void k_scan_partials(
    uint32_t *partials, int64_t nparts, uint32_t *out_total, unsigned long long *counters,
    int which, uint32_t *flags, uint64_t cap)
{
    __shared__ unsigned long long lds[kScanPartialsThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    unsigned long long carry = 0;
    for (int64_t b0 = 0; b0 < nparts; b0 += kScanPartialsThreads * kScanPartialsItems) {
        const int64_t i = b0 + (int64_t)threadIdx.x * kScanPartialsItems;
        uint32_t x[kScanPartialsItems];
        unsigned long long sum = 0;
#pragma unroll
        for (int k = 0; k < kScanPartialsItems; ++k) {
            x[k] = i + k < nparts ? partials[i + k] : 0u;
            sum += x[k];
        }
        unsigned long long inc = sum;
        for (int d = 1; d < kWave; d <<= 1) {
            unsigned long long y = __shfl_up(inc, d, kWave);
            if (lane >= d) inc += y;
        }
        if (lane == kWave - 1) lds[w] = inc;
        __syncthreads();
        unsigned long long run = carry + inc - sum;
        for (int k = 0; k < kScanPartialsThreads / kWave; ++k) {
            if (k < w) run += lds[k];
            carry += lds[k];
        }
#pragma unroll
        for (int k = 0; k < kScanPartialsItems; ++k) {
            if (i + k < nparts) partials[i + k] = (uint32_t)min(run, 0xFFFFFFFFull);
            run += x[k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        counters[which] = carry;
        *out_total = (uint32_t)min(carry, 0xFFFFFFFFull);
        if (carry > 0xFFFFFFFFull || carry > cap) flags[0] |= 1u;
    }
}

__global__ void k_scan_down(const uint32_t *in, int64_t len, const uint32_t *partials,
                            uint32_t *out)
{
    __shared__ uint32_t lds[kSortWaves];
    int64_t base = (int64_t)blockIdx.x * kSortTile + (int64_t)threadIdx.x * kSortItems;
    uint32_t v[kSortItems];
    load_items(in, base, len, v);
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) s += v[i];
    uint32_t tot;
    uint32_t run = block_exclusive_scan(s, lds, &tot) + partials[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) {
        const uint32_t x = v[i];
        v[i] = run;
        run += x;
    }
    store_items(out, base, len, v);
}

size_t scan_temp_elems(int64_t len)
{
    return (size_t)((len + kSortTile - 1) / kSortTile) + 1;
}

// Up to kScanOneBlock sums (4M (view, rank) pairs) one block scans them all: ~6 us, less
// than the two further launches of the three-kernel scan.
hipError_t scan_pair_sums(uint32_t *sums, int64_t n, int32_t nv, uint32_t *partials,
                          unsigned long long *counters, int which, uint32_t *flags, uint64_t cap,
                          hipStream_t st)
{
    const int64_t len = (int64_t)nv * rank_blocks(n);
    const bool one = len <= kScanOneBlock;
    const int64_t nb = (len + kSortTile - 1) / kSortTile;
    if (!one)
        hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kSortThreads), 0, st, sums, len,
                           partials);
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kScanPartialsThreads), 0, st, one ? sums : partials,
                       one ? len : nb, sums + len, counters, which, flags, cap);
    if (!one)
        hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(kSortThreads), 0, st, sums, len,
                           partials, sums);
    return hipGetLastError();
}

// ------------------------------------------------------------------ radix sort
// Blocks never straddle a segment: block b of segment v covers items
// [start_v + j * kSortTile, ...) with j = b - blk0_v, and its digits are taken from
// key - base_v.  The histogram of block b sits at blk0_v * 256 + digit * nblk_v + j, so
// one exclusive scan over all blocks' histograms gives every (segment, digit, block) its
// output position inside its own segment.  Blocks past the last live one write zeros at
// b * 256 + digit, after every live block's entries.
struct SegDesc {
    uint32_t start, end, blk0, base;
};

struct BlockRange {
    int64_t lo, hi;
    uint32_t base;
    int64_t hidx0;      // histogram index of digit 0
    int64_t hstride;    // histogram index step per digit
    bool live;
};

__device__ __forceinline__ BlockRange block_range(const SegDesc *segs, int nseg,
                                                  const unsigned long long *n_dev, int64_t cap,
                                                  int64_t n_host, int64_t b)
{
    BlockRange r;
    if (!segs) {
        const int64_t n = live_count(n_dev, cap, n_host);
        const int64_t nb = (n + kSortTile - 1) / kSortTile;
        r.lo = b * kSortTile;
        r.hi = min(n, r.lo + kSortTile);
        r.base = 0;
        r.live = b < nb;
        r.hidx0 = r.live ? b : b * 256;
        r.hstride = r.live ? nb : 1;
        return r;
    }
    const int64_t total = segs[nseg].blk0;
    r.live = b < total;
    if (!r.live) {
        r.lo = r.hi = 0;
        r.base = 0;
        r.hidx0 = b * 256;
        r.hstride = 1;
        return r;
    }
    // last segment whose first block is <= b (segments without blocks share blk0 with
    // the next one and are skipped by taking the last)
    int lo = 0, hi = nseg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)segs[mid].blk0 <= b) lo = mid; else hi = mid - 1;
    }
    const SegDesc sd = segs[lo];
    const int64_t j = b - sd.blk0;
    const int64_t nblk = (int64_t)segs[lo + 1].blk0 - sd.blk0;
    r.lo = (int64_t)sd.start + j * kSortTile;
    r.hi = min((int64_t)sd.end, r.lo + kSortTile);
    r.base = sd.base;
    r.hidx0 = (int64_t)sd.blk0 * 256 + j;
    r.hstride = nblk;
    return r;
}

// One block: segment table from view-major pair offsets.  Segment v holds the items
// [offs[v * stride], offs[(v + 1) * stride]) clamped to the live count; its keys are
// based at views[v].tile_off.
constexpr int kSegThreads = 1024;

__global__ __launch_bounds__(kSegThreads) void k_seg_table(
    const uint32_t *offs, int64_t stride, int32_t nseg, const ViewDesc *views,
    const unsigned long long *n_dev, int64_t cap, SegDesc *segs)
{
    __shared__ uint32_t lds_w[kSegThreads / kWave];
    __shared__ uint32_t carry;
    const int64_t n = live_count(n_dev, cap, cap);
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int32_t v0 = 0; v0 <= nseg; v0 += kSegThreads) {
        const int32_t v = v0 + (int32_t)threadIdx.x;
        uint32_t st = 0, en = 0, nblk = 0;
        if (v <= nseg) {
            st = (uint32_t)min((int64_t)offs[(int64_t)v * stride], n);
            en = v < nseg ? (uint32_t)min((int64_t)offs[(int64_t)(v + 1) * stride], n) : st;
            en = max(en, st);
            nblk = v < nseg ? (en - st + kSortTile - 1) / kSortTile : 0u;
        }
        const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
        uint32_t inc = nblk;
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(inc, d, kWave);
            if (lane >= d) inc += y;
        }
        if (lane == kWave - 1) lds_w[w] = inc;
        __syncthreads();
        uint32_t wbase = 0, tot = 0;
        for (int k = 0; k < kSegThreads / kWave; ++k) {
            if (k < w) wbase += lds_w[k];
            tot += lds_w[k];
        }
        if (v <= nseg)
            segs[v] = SegDesc{st, en, carry + wbase + inc - nblk,
                              v < nseg ? (uint32_t)views[v].tile_off : 0u};
        __syncthreads();
        if (threadIdx.x == 0) carry += tot;
        __syncthreads();
    }
}

// KT = uint16_t: tile keys local to their segment (the digit is taken from the key
// itself, the segment base only offsets the tile ranges); uint32_t: keys carry the
// segment base, which the digit subtracts.
template <typename KT>
__device__ __forceinline__ uint32_t key_digit(KT key, uint32_t base, int shift)
{
    constexpr bool kLocal = sizeof(KT) == 2;
    return (((uint32_t)key - (kLocal ? 0u : base)) >> shift) & 255u;
}

// Runs of 16 consecutive tiles on one XCD (blocks go round-robin to the 8): a digit's runs of
// neighbouring tiles meet in one L2, which then writes whole lines (those scatters 2.98 -> 2.61
// ms, the histograms 0.71 -> 0.67; runs of 32: 2.64 ms).
__device__ __forceinline__ int sort_block(int b, int nblocks)
{
    constexpr int kRun = 16;
    if (b >= nblocks - nblocks % (8 * kRun)) return b;
    const int x = b % 8, i = b / 8;
    return ((i / kRun) * 8 + x) * kRun + i % kRun;
}

template <typename KT>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(
    const KT *keys, const SegDesc *segs, int nseg, const unsigned long long *n_dev,
    int64_t cap, int64_t n_host, int shift, uint32_t *hist)
{
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const BlockRange br = block_range(segs, nseg, n_dev, cap, n_host, sort_block(blockIdx.x, gridDim.x));
    if (br.live) {
        const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
        const int64_t wbase = br.lo + (int64_t)w * (kSortItems * kWave);
        // all of the wave's keys are loaded before any is counted
        uint32_t key[kSortItems];
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) {
            const int64_t i = wbase + it * kWave + lane;
            key[it] = i < br.hi ? (uint32_t)keys[i] : 0u;
        }
        // one LDS add per key: the LDS serialises lanes that hit the same counter, which
        // costs less than finding each digit's group of lanes with ballots
#pragma unroll
        for (int it = 0; it < kSortItems; ++it) {
            if (wbase + it * kWave + lane < br.hi)
                atomicAdd(&h[key_digit<KT>((KT)key[it], br.base, shift)], 1u);
        }
    }
    __syncthreads();
    hist[br.hidx0 + (int64_t)threadIdx.x * br.hstride] = h[threadIdx.x];
}

// Exclusive scan over the histograms, single pass per block chunk using the same
// three-kernel scheme as the pair counts but on a 32-bit total.
__global__ void k_hist_scan_reduce(uint32_t *hist, int64_t len, uint32_t *partials)
{
    __shared__ uint32_t lds[kSortWaves];
    int64_t base = (int64_t)blockIdx.x * kSortTile + (int64_t)threadIdx.x * kSortItems;
    uint32_t v[kSortItems];
    load_items(hist, base, len, v);
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < kSortItems; ++i) s += v[i];
    uint32_t tot;
    block_exclusive_scan(s, lds, &tot);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kScanPartialsThreads) void k_hist_scan_partials(uint32_t *partials,
                                                                             int64_t nparts)
{
    __shared__ uint32_t lds[kScanPartialsThreads / kWave];
    __shared__ uint32_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < nparts; b0 += blockDim.x) {
        int64_t i = b0 + threadIdx.x;
        uint32_t x = i < nparts ? partials[i] : 0u;
        const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
        uint32_t inc = x;
        for (int d = 1; d < kWave; d <<= 1) {
            uint32_t y = __shfl_up(inc, d, kWave);
            if (lane >= d) inc += y;
        }
        if (lane == kWave - 1) lds[w] = inc;
        __syncthreads();
        uint32_t wbase = 0, tot = 0;
        for (int k = 0; k < (int)(blockDim.x / kWave); ++k) {
            if (k < w) wbase += lds[k];
            tot += lds[k];
        }
        if (i < nparts) partials[i] = carry + wbase + inc - x;
        __syncthreads();
        if (threadIdx.x == 0) carry += tot;
        __syncthreads();
    }
}

// Stable ranks of a wave's rows of items within their digits; entry d of the wave's table in
// LDS holds the lanes of the row in work that have digit d, and the items of digit d in the
// rows before.  Every lane sets its bit, reads the entry - its peers, so its place among them -
// and the lowest peer writes the entry back with the row counted.  LDS instructions of one wave
// take effect in issue order.  (Finding the peers by a ballot per digit bit took 48 vector
// instructions a row: the scatters of 193M view pairs and 40 sun maps 3.8 ms, now 3.0.)
// 16-bit keys carry their rank in the upper half (a wave has at most 1024 items).
template <typename KT, int ITEMS>
__device__ __forceinline__ void rank_rows(uint32_t (&key)[ITEMS], uint32_t (&rank)[ITEMS],
                                          uint4 *wtab, int64_t wbase, int64_t hi, uint32_t base, int shift)
{
    static_assert(ITEMS * kWave <= 65536);
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t bit = 1ull << lane;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const bool valid = wbase + it * kWave + lane < hi;
        uint4 *const e = wtab + key_digit<KT>((KT)key[it], base, shift);
        if (valid) atomicOr(reinterpret_cast<unsigned long long *>(e), bit);
        __builtin_amdgcn_wave_barrier();
        const uint4 x = *e;
        const uint64_t m = ((uint64_t)x.y << 32) | x.x;
        const uint32_t before = __popcll(m & (bit - 1));
        if (valid && before == 0) *e = make_uint4(0, 0, x.z + (uint32_t)__popcll(m), 0);
        __builtin_amdgcn_wave_barrier();
        if (sizeof(KT) == 2) key[it] |= (x.z + before) << 16;
        else rank[it] = x.z + before;
    }
    // the digits are taken from the keys again, not kept
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) asm("" : "+v"(key[it]));
}

template <typename KT>
__device__ __forceinline__ uint32_t rank_of(uint32_t key, uint32_t rank)
{
    return sizeof(KT) == 2 ? key >> 16 : rank;
}

// With `ranges` (the last pass), every block also reports, per key, the first and last
// output position of its run: ranges[2k] = min over blocks, ranges[2k + 1] = max + 1.
// A block holds its items in LDS sorted by the whole key (stable on the top digit of
// items that the lower passes left sorted), so equal keys are adjacent there.
template <typename KT>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const KT *kin, const uint32_t *vin, KT *kout, uint32_t *vout,
    const uint32_t *offs, const SegDesc *segs, int nseg, const unsigned long long *n_dev,
    int64_t cap, int64_t n_host, int shift, uint32_t *ranges, int64_t nkeys,
    uint32_t *rank_out)
{
    constexpr bool kLocal = sizeof(KT) == 2;
    __shared__ uint32_t wcnt[kSortWaves][256];
    __shared__ uint32_t dbase[256];          // block-local start of each digit's run
    __shared__ uint32_t gshift[256];         // global start minus local start, per digit
    __shared__ uint32_t lds_w[kSortWaves];
    __shared__ KT skey[kSortTile];
    // per wave and digit, the row's lanes and the count before it (ranking); later the values
    __shared__ uint4 tab[kSortWaves * 256];
    uint32_t *const sval = reinterpret_cast<uint32_t *>(tab);
    static_assert(sizeof(tab) >= sizeof(uint32_t) * kSortTile);
    const BlockRange br = block_range(segs, nseg, n_dev, cap, n_host, sort_block(blockIdx.x, gridDim.x));
    if (!br.live) return;   // uniform over the block
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int64_t wbase = br.lo + (int64_t)w * (kSortItems * kWave);
    uint4 *const wtab = tab + w * 256;
    for (int i = lane; i < 256; i += kWave) wtab[i] = make_uint4(0, 0, 0, 0);
    uint32_t key[kSortItems], val[kSortItems], rank[kSortItems];
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const int64_t i = wbase + it * kWave + lane;
        const bool valid = i < br.hi;
        key[it] = valid ? (uint32_t)kin[i] : 0u;
        val[it] = valid ? vin[i] : 0u;
    }
    rank_rows<KT, kSortItems>(key, rank, wtab, wbase, br.hi, br.base, shift);
    for (int i = lane; i < 256; i += kWave) wcnt[w][i] = wtab[i].z;
    __syncthreads();
    {
        // per digit: prefix over the waves, then an exclusive scan over the digits gives
        // each digit's run inside the block; the run goes to offs[digit, block] globally
        const int d = threadIdx.x;
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < kSortWaves; ++k) {
            const uint32_t c = wcnt[k][d];
            wcnt[k][d] = run;
            run += c;
        }
        uint32_t tot;
        const uint32_t excl = block_exclusive_scan(run, lds_w, &tot);
        dbase[d] = excl;
        gshift[d] = offs[br.hidx0 + (int64_t)d * br.hstride] - excl;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
        const int64_t i = wbase + it * kWave + lane;
        if (i < br.hi) {
            const uint32_t d = key_digit<KT>((KT)key[it], br.base, shift);
            const uint32_t lp = dbase[d] + wcnt[w][d] + rank_of<KT>(key[it], rank[it]);
            if (lp < (uint32_t)kSortTile) {   // always true when the counts agree
                skey[lp] = (KT)key[it];
                sval[lp] = val[it];
            }
        }
    }
    __syncthreads();
    // digit runs are contiguous in LDS and in the output: consecutive threads write
    // consecutive addresses within a run
    const int nloc = (int)(br.hi - br.lo);
    const int64_t n_out = segs ? (int64_t)segs[nseg].end : live_count(n_dev, cap, n_host);
    for (int i = threadIdx.x; i < nloc; i += kSortThreads) {
        const KT k = skey[i];
        const uint32_t pos = gshift[key_digit<KT>(k, br.base, shift)] + (uint32_t)i;
        if (pos < n_out) {   // always true when histogram and scatter agree
            if (kout) kout[pos] = k;
            vout[pos] = sval[i];
            if (rank_out && sval[i] < (uint32_t)n_out) rank_out[sval[i]] = pos;
            // the tile a key names: local keys sit on the segment's base
            const int64_t gk = kLocal ? (int64_t)br.base + (int64_t)k : (int64_t)k;
            if (ranges && gk < nkeys) {
                if (i == 0 || skey[i - 1] != k) atomicMin(&ranges[2 * gk], pos);
                if (i == nloc - 1 || skey[i + 1] != k) atomicMax(&ranges[2 * gk + 1], pos + 1);
            }
        }
    }
}

__global__ void k_ranges_finish(uint32_t *ranges, int64_t nkeys)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nkeys) return;
    uint2 r = reinterpret_cast<uint2 *>(ranges)[k];
    if (r.x == 0xFFFFFFFFu) reinterpret_cast<uint2 *>(ranges)[k] = make_uint2(0u, 0u);
}

hipError_t finish_ranges(uint32_t *ranges, int64_t nkeys, hipStream_t st)
{
    if (nkeys <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ranges_finish, dim3((unsigned)((nkeys + 255) / 256)), dim3(256), 0, st, ranges,
                       nkeys);
    return hipGetLastError();
}

// ------------------------------------------------------------ sorts of few blocks
// With few blocks the sort's time is its launches: five per pass above (histogram, three of
// the scan, scatter).  Here a pass is two.  Digit counts are rows of 256 per block,
// [block][digit]; a scatter block sums the rows of its segment itself (all of them for the
// digit totals, those before it for its own offsets).  Block b of segment v has row start_v /
// TILE + v + (b's place in the segment): rows of different segments are disjoint, and no
// segment table is needed.  Reading all rows grows with the square of the blocks: up to 128
// blocks of 1024 items, then up to 256 of 2048 and 4096 (1M items), beyond which the scans
// above are as fast.  (Counting the next pass's digits while scattering saves the histogram launch, but
// keys that share a digit then meet on one address: 80 us for a pass of 190,000 pairs.)
// Depth order of 20,000 surfels: 21 launches, 104 us -> 8 launches, 44 us (fewer still by
// k_depth_merge); of 1M: 145 -> 125 us.
constexpr int kSmallRows4 = 128, kSmallRows = 256;

SmallSort plan_small_sort(int64_t cap, int32_t nseg, int bits)
{
    const int passes = bits <= 8 ? 1 : (bits + 7) / 8;
    const int64_t extra = nseg > 0 ? nseg + 1 : 1;
    for (int items : {4, 8, 16}) {
        const int64_t rows = cap / (items * kSortThreads) + extra;
        if (rows <= (items == 4 ? kSmallRows4 : kSmallRows)) return SmallSort{items, rows, passes};
    }
    return SmallSort{0, 0, passes};
}

// Depth keys and their first digits' counts
template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_depth_keys_hist(const float *__restrict__ mean,
                                                                  int64_t n, float bz,
                                                                  uint32_t *__restrict__ keys,
                                                                  uint32_t *__restrict__ hist)
{
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * (ITEMS * kSortThreads) + threadIdx.x;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = lo + it * kSortThreads;
        if (i < n) {
            const uint32_t k = depth_key(bz, mean[3 * i + 2]);
            keys[i] = k;
            atomicAdd(&h[k & 255u], 1u);
        }
    }
    __syncthreads();
    hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

// Segments of the tile sort (offs == NULL: one segment of all items)
struct SmallSegs {
    const uint32_t *offs;
    int64_t stride;
    int32_t nseg;
    const ViewDesc *views;
};

// Block b's segment and its items [i0, i1) (none: i0 >= i1)
struct SmallBlock {
    int64_t start, end, row0, i0, i1;
    uint32_t base;
};

template <int TILE>
__device__ __forceinline__ SmallBlock small_block(const SmallSegs &sg, int64_t n, int64_t b)
{
    SmallBlock s{0, n, 0, 0, 0, 0};
    if (sg.offs) {
        int lo = 0, hi = sg.nseg - 1;                 // last segment whose first row is <= b
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (min((int64_t)sg.offs[mid * sg.stride], n) / TILE + mid <= b) lo = mid; else hi = mid - 1;
        }
        s.start = min((int64_t)sg.offs[lo * sg.stride], n);
        s.end = min((int64_t)sg.offs[(lo + 1) * sg.stride], n);
        s.row0 = s.start / TILE + lo;
        s.base = (uint32_t)sg.views[lo].tile_off;
    }
    s.i0 = s.start + (b - s.row0) * TILE;
    s.i1 = b < s.row0 ? s.i0 : min(s.end, s.i0 + TILE);
    return s;
}

template <typename KT, int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_small_hist(const KT *__restrict__ keys, SmallSegs sg,
                                                             const unsigned long long *__restrict__ n_dev,
                                                             int64_t cap, int64_t n_host, int shift,
                                                             uint32_t *__restrict__ hist)
{
    __shared__ uint32_t h[256];
    const SmallBlock s = small_block<ITEMS * kSortThreads>(sg, live_count(n_dev, cap, n_host), blockIdx.x);
    if (s.i0 >= s.i1) return;                         // uniform over the block; its row is not read
    uint32_t key[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = s.i0 + it * kSortThreads + threadIdx.x;
        key[it] = i < s.i1 ? (uint32_t)keys[i] : 0u;
    }
    h[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (s.i0 + it * kSortThreads + threadIdx.x < s.i1)
            atomicAdd(&h[key_digit<KT>((KT)key[it], s.base, shift)], 1u);
    __syncthreads();
    hist[(int64_t)blockIdx.x * 256 + threadIdx.x] = h[threadIdx.x];
}

template <typename KT, int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_small_scatter(
    const KT *__restrict__ kin, const uint32_t *__restrict__ vin, KT *__restrict__ kout,
    uint32_t *__restrict__ vout, const uint32_t *__restrict__ hist, int64_t rows, SmallSegs sg, const unsigned long long *__restrict__ n_dev, int64_t cap,
    int64_t n_host, int shift, uint32_t *__restrict__ ranges, int64_t nkeys,
    uint32_t *__restrict__ rank_out)
{
    constexpr int TILE = ITEMS * kSortThreads;
    constexpr bool kLocal = sizeof(KT) == 2;
    __shared__ uint32_t wcnt[kSortWaves][256];
    __shared__ uint4 csum[2][kSortWaves][kWave];      // column sums per wave: all rows, rows before
    __shared__ uint32_t dbase[256], gshift[256];
    __shared__ uint32_t lds_w[kSortWaves];
    // the waves' ranking tables (see rank_rows); later the values and keys in digit order
    constexpr int kTab = kSortWaves * 256, kOut = (int)(sizeof(KT) + 4) * TILE / 16;
    __shared__ uint4 tab[kTab > kOut ? kTab : kOut];
    uint32_t *const sval = reinterpret_cast<uint32_t *>(tab);
    KT *const skey = reinterpret_cast<KT *>(sval + TILE);
    const int64_t n = live_count(n_dev, cap, n_host);
    const SmallBlock sb = small_block<TILE>(sg, n, blockIdx.x);
    const int64_t start = sb.start, end = sb.end, row0 = sb.row0, i0 = sb.i0, i1 = sb.i1;
    const int64_t mine = blockIdx.x - row0;
    const uint32_t base = sb.base;
    if (i0 >= i1) return;                             // uniform over the block
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int64_t wbase = i0 + (int64_t)w * (ITEMS * kWave);
    uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = wbase + it * kWave + lane;
        const bool valid = i < i1;
        key[it] = valid ? (uint32_t)kin[i] : 0u;
        val[it] = valid ? (vin ? vin[i] : (uint32_t)i) : 0u;
    }
    uint4 *const wtab = tab + w * 256;
    for (int i = lane; i < 256; i += kWave) wtab[i] = make_uint4(0, 0, 0, 0);
    // column sums of the segment's rows, four digits per lane and a quarter of the rows per wave
    const int64_t nrows = min((end - start + TILE - 1) / TILE, rows - row0);
    uint4 all = make_uint4(0, 0, 0, 0), bef = make_uint4(0, 0, 0, 0);
    const uint4 *hrow = reinterpret_cast<const uint4 *>(hist + row0 * 256) + lane;
#pragma unroll 8
    for (int64_t r = w; r < nrows; r += kSortWaves) {
        const uint4 x = hrow[r * 64];
        all.x += x.x; all.y += x.y; all.z += x.z; all.w += x.w;
        if (r < mine) { bef.x += x.x; bef.y += x.y; bef.z += x.z; bef.w += x.w; }
    }
    csum[0][w][lane] = all;
    csum[1][w][lane] = bef;
    __syncthreads();
    rank_rows<KT, ITEMS>(key, rank, wtab, wbase, i1, base, shift);
    for (int i = lane; i < 256; i += kWave) wcnt[w][i] = wtab[i].z;
    __syncthreads();
    {
        const int d = threadIdx.x;
        const uint32_t *c0 = reinterpret_cast<const uint32_t *>(csum[0]), *c1 = reinterpret_cast<const uint32_t *>(csum[1]);
        uint32_t total = 0, before = 0, run = 0;
#pragma unroll
        for (int k = 0; k < kSortWaves; ++k) {
            total += c0[k * 256 + d];
            before += c1[k * 256 + d];
            const uint32_t c = wcnt[k][d];
            wcnt[k][d] = run;
            run += c;
        }
        uint32_t tot;
        const uint32_t below = block_exclusive_scan(total, lds_w, &tot);
        const uint32_t excl = block_exclusive_scan(run, lds_w, &tot);
        dbase[d] = excl;
        gshift[d] = (uint32_t)start + below + before - excl;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t i = wbase + it * kWave + lane;
        if (i < i1) {
            const uint32_t d = key_digit<KT>((KT)key[it], base, shift);
            const uint32_t lp = dbase[d] + wcnt[w][d] + rank_of<KT>(key[it], rank[it]);
            if (lp < (uint32_t)TILE) {                // always true when the counts agree
                skey[lp] = (KT)key[it];
                sval[lp] = val[it];
            }
        }
    }
    __syncthreads();
    const int nloc = (int)(i1 - i0);
    for (int i = threadIdx.x; i < nloc; i += kSortThreads) {
        const KT k = skey[i];
        const int64_t pos = (int64_t)gshift[key_digit<KT>(k, base, shift)] + i;
        // within the segment whenever counts and items agree
        const uint32_t p32 = (uint32_t)pos;
        if (p32 < start || p32 >= end) continue;
        const uint32_t v = sval[i];
        if (kout) kout[p32] = k;
        vout[p32] = v;
        if (rank_out && v < (uint32_t)n) rank_out[v] = p32;
        const int64_t gk = kLocal ? (int64_t)base + (int64_t)k : (int64_t)k;
        if (ranges && gk < nkeys) {
            if (i == 0 || skey[i - 1] != k) atomicMin(&ranges[2 * gk], p32);
            if (i == nloc - 1 || skey[i + 1] != k) atomicMax(&ranges[2 * gk + 1], p32 + 1);
        }
    }
}

template <typename KT>
static void small_passes(const SmallSort &plan, KT *ka, uint32_t *va, KT *kb, uint32_t *vb, bool index_vals,
                         bool have_hist, int64_t cap, const unsigned long long *n_dev, int64_t n_host,
                         uint32_t *hist, const SmallSegs &sg, uint32_t *ranges, int64_t nkeys,
                         uint32_t *rank_out, bool *result_in_b, hipStream_t st)
{
    *result_in_b = false;
    for (int p = 0; p < plan.passes; ++p) {
        const bool last = p == plan.passes - 1;
        const int shift = 8 * p;
        const uint32_t *vin = p == 0 && index_vals ? nullptr : va;
        KT *ko = last ? nullptr : kb;      // nothing reads the sorted keys
        const dim3 grid((unsigned)plan.rows), blk(kSortThreads);
        auto pass = [&](auto hist_kernel, auto scatter_kernel) {
            if (p > 0 || !have_hist)
                hipLaunchKernelGGL(hist_kernel, grid, blk, 0, st, ka, sg, n_dev, cap, n_host, shift, hist);
            hipLaunchKernelGGL(scatter_kernel, grid, blk, 0, st, ka, vin, ko, vb, hist, plan.rows, sg,
                               n_dev, cap, n_host, shift, last ? ranges : nullptr, nkeys,
                               last ? rank_out : nullptr);
        };
        if (plan.items == 4) pass(k_small_hist<KT, 4>, k_small_scatter<KT, 4>);
        else if (plan.items == 8) pass(k_small_hist<KT, 8>, k_small_scatter<KT, 8>);
        else pass(k_small_hist<KT, 16>, k_small_scatter<KT, 16>);
        std::swap(ka, kb);
        std::swap(va, vb);
        *result_in_b = !*result_in_b;
    }
}

template <typename KT>
hipError_t small_sort_tiles(const SmallSort &plan, KT *keys_a, uint32_t *vals_a, KT *keys_b,
                            uint32_t *vals_b, int64_t cap, const unsigned long long *n_dev, int bits,
                            uint32_t *hist, bool *result_in_b, hipStream_t st, const SortSegments &seg)
{
    const SmallSegs sg{seg.offs, seg.stride, seg.nseg, seg.views};
    small_passes<KT>(plan, keys_a, vals_a, keys_b, vals_b, false, false, cap, n_dev, 0, hist, sg,
                     seg.nkeys > 0 ? seg.ranges : nullptr, seg.nkeys, nullptr, result_in_b, st);
    return hipGetLastError();
}

template hipError_t small_sort_tiles<uint32_t>(const SmallSort &, uint32_t *, uint32_t *, uint32_t *, uint32_t *,
                                               int64_t, const unsigned long long *, int, uint32_t *, bool *,
                                               hipStream_t, const SortSegments &);
template hipError_t small_sort_tiles<uint16_t>(const SmallSort &, uint16_t *, uint32_t *, uint16_t *, uint32_t *,
                                               int64_t, const unsigned long long *, int, uint32_t *, bool *,
                                               hipStream_t, const SortSegments &);

// Depth order of few surfels in two launches: chunks of 1024 sorted in LDS, then every item
// finds its place by binary search in all chunks, whose keys fit one CU's LDS.  Stable: equal
// keys of earlier chunks come first.  20,000 surfels: 8 launches of eight-bit passes and 41 us
// -> 2 launches and 26 us.  The line at kMergeMax is what a CU's LDS holds beside nothing else
// (a second block of 128 KB does not fit); the searches also grow with n^2 / 1024.
constexpr int kChunkItems = 4, kChunk = kChunkItems * kSortThreads;
constexpr int kMergeThreads = 256, kMergeMax = 32768;

__global__ __launch_bounds__(kSortThreads) void k_depth_chunks(const float *__restrict__ mean, int64_t n,
                                                               float bz, uint32_t *__restrict__ keys,
                                                               uint32_t *__restrict__ vals)
{
    __shared__ uint4 tab[kSortWaves * 256];
    __shared__ uint32_t wcnt[kSortWaves][256];
    __shared__ uint32_t dbase[256];
    __shared__ uint32_t lds_w[kSortWaves];
    __shared__ uint32_t skey[kChunk];
    __shared__ uint16_t sidx[kChunk];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int64_t i0 = (int64_t)blockIdx.x * kChunk;
    const int cnt = (int)min((int64_t)kChunk, n - i0);
    const int at = w * (kChunkItems * kWave) + lane;
    uint4 *const wtab = tab + w * 256;
    uint32_t key[kChunkItems], idx[kChunkItems], rank[kChunkItems];
#pragma unroll
    for (int it = 0; it < kChunkItems; ++it) {
        const int i = at + it * kWave;
        key[it] = i < cnt ? depth_key(bz, mean[3 * (i0 + i) + 2]) : 0u;
        idx[it] = (uint32_t)i;
    }
    for (int shift = 0; shift < 32; shift += 8) {
        for (int i = lane; i < 256; i += kWave) wtab[i] = make_uint4(0, 0, 0, 0);
        rank_rows<uint32_t, kChunkItems>(key, rank, wtab, (int64_t)w * (kChunkItems * kWave), cnt, 0, shift);
        for (int i = lane; i < 256; i += kWave) wcnt[w][i] = wtab[i].z;
        __syncthreads();
        {
            const int d = threadIdx.x;
            uint32_t run = 0;
#pragma unroll
            for (int k = 0; k < kSortWaves; ++k) {
                const uint32_t c = wcnt[k][d];
                wcnt[k][d] = run;
                run += c;
            }
            uint32_t tot;
            dbase[d] = block_exclusive_scan(run, lds_w, &tot);
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kChunkItems; ++it) {
            const uint32_t d = key_digit<uint32_t>(key[it], 0, shift);
            const uint32_t lp = dbase[d] + wcnt[w][d] + rank[it];
            if (at + it * kWave < cnt && lp < (uint32_t)kChunk) {
                skey[lp] = key[it];
                sidx[lp] = (uint16_t)idx[it];
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kChunkItems; ++it) {
            const int i = at + it * kWave;
            if (i < cnt) {
                key[it] = skey[i];
                idx[it] = sidx[i];
            }
        }
    }
#pragma unroll
    for (int it = 0; it < kChunkItems; ++it) {
        const int i = at + it * kWave;
        if (i < cnt) {
            keys[i0 + i] = key[it];
            vals[i0 + i] = (uint32_t)i0 + idx[it];
        }
    }
}

// Keys of a sorted chunk of m (at most kChunk) that come before k.
template <bool EQUAL>
__device__ __forceinline__ uint32_t keys_before(const uint32_t *chunk, uint32_t m, uint32_t k)
{
    uint32_t pos = 0;
#pragma unroll
    for (uint32_t s = kChunk; s > 0; s >>= 1) {
        const uint32_t x = chunk[min(pos + s, m) - 1];
        const bool before = EQUAL ? x <= k : x < k;
        pos += pos + s <= m && before ? s : 0u;
    }
    return pos;
}

__global__ __launch_bounds__(kMergeThreads) void k_depth_merge(const uint32_t *__restrict__ keys,
                                                               const uint32_t *__restrict__ vals, int n,
                                                               uint32_t *__restrict__ order,
                                                               uint32_t *__restrict__ rank)
{
    __shared__ __align__(16) uint32_t all[kMergeMax];
    const int n4 = n / 4;
#pragma unroll 8
    for (int i = threadIdx.x; i < n4; i += kMergeThreads)
        reinterpret_cast<uint4 *>(all)[i] = reinterpret_cast<const uint4 *>(keys)[i];
    if (threadIdx.x < n - 4 * n4) all[4 * n4 + threadIdx.x] = keys[4 * n4 + threadIdx.x];
    __syncthreads();
    const int i = blockIdx.x * kMergeThreads + threadIdx.x;
    if (i >= n) return;
    static_assert(kChunk % kMergeThreads == 0);       // a block's items lie in one chunk
    const int c = (int)(blockIdx.x * kMergeThreads) / kChunk, chunks = (n + kChunk - 1) / kChunk;
    const uint32_t k = all[i];
    uint32_t pos = (uint32_t)(i - c * kChunk);
#pragma unroll 4
    for (int q = 0; q < c; ++q) pos += keys_before<true>(all + q * kChunk, kChunk, k);
#pragma unroll 4
    for (int q = c + 1; q < chunks; ++q)
        pos += keys_before<false>(all + q * kChunk, (uint32_t)min(kChunk, n - q * kChunk), k);
    const uint32_t v = vals[i];
    if (pos < (uint32_t)n && v < (uint32_t)n) {       // always
        order[pos] = v;
        if (rank) rank[v] = pos;
    }
}

__global__ void k_depth_keys(const float *__restrict__ mean, int64_t n, float bz,
                             uint32_t *__restrict__ keys, uint32_t *__restrict__ vals)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[i] = depth_key(bz, mean[3 * i + 2]);
    vals[i] = (uint32_t)i;
}

hipError_t depth_sort(const float *mean, int64_t n, float bz, uint32_t *keys_a, uint32_t *vals_a,
                      uint32_t *keys_b, uint32_t *vals_b, void *temp, uint32_t *rank,
                      bool *result_in_b, hipStream_t st)
{
    *result_in_b = false;
    if (n <= 0) return hipSuccess;
    if (n <= kMergeMax) {
        hipLaunchKernelGGL(k_depth_chunks, dim3((unsigned)((n + kChunk - 1) / kChunk)), dim3(kSortThreads), 0,
                           st, mean, n, bz, keys_b, vals_b);
        hipLaunchKernelGGL(k_depth_merge, dim3((unsigned)((n + kMergeThreads - 1) / kMergeThreads)),
                           dim3(kMergeThreads), 0, st, keys_b, vals_b, (int)n, vals_a, rank);
        return hipGetLastError();
    }
    const SmallSort plan = plan_small_sort(n, 0, 32);
    if (plan.rows == 0) {
        hipLaunchKernelGGL(k_depth_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, mean, n, bz,
                           keys_a, vals_a);
        return radix_sort_pairs(keys_a, vals_a, keys_b, vals_b, n, nullptr, n, 32, temp, result_in_b, st,
                                nullptr, rank);
    }
    uint32_t *hist = reinterpret_cast<uint32_t *>(temp);
    const dim3 grid((unsigned)plan.rows), blk(kSortThreads);
    if (plan.items == 4)
        hipLaunchKernelGGL(k_depth_keys_hist<4>, grid, blk, 0, st, mean, n, bz, keys_a, hist);
    else if (plan.items == 8)
        hipLaunchKernelGGL(k_depth_keys_hist<8>, grid, blk, 0, st, mean, n, bz, keys_a, hist);
    else
        hipLaunchKernelGGL(k_depth_keys_hist<16>, grid, blk, 0, st, mean, n, bz, keys_a, hist);
    small_passes<uint32_t>(plan, keys_a, vals_a, keys_b, vals_b, true, true, n, nullptr, n, hist,
                           SmallSegs{nullptr, 0, 0, nullptr}, nullptr, 0, rank, result_in_b, st);
    return hipGetLastError();
}

static int64_t sort_blocks(int64_t items) { return (items + kSortTile - 1) / kSortTile; }

size_t radix_temp_bytes(int64_t max_items, int32_t max_segs)
{
    const size_t small = (size_t)kSmallRows * 256 * sizeof(uint32_t);
    const int64_t nb = sort_blocks(max_items > 0 ? max_items : 1) + max_segs;
    const int64_t hist = 256 * nb;
    const int64_t parts = (hist + kSortTile - 1) / kSortTile + 1;
    return std::max(small, (size_t)(hist + parts) * sizeof(uint32_t) + 256 +
                               (size_t)(max_segs + 1) * sizeof(SegDesc) + 256);
}

template <typename KT>
hipError_t radix_sort_pairs(KT *keys_a, uint32_t *vals_a, KT *keys_b,
                            uint32_t *vals_b, int64_t cap, const unsigned long long *n_dev,
                            int64_t n_host, int bits, void *temp, bool *result_in_b,
                            hipStream_t st, const SortSegments *seg, uint32_t *rank_out)
{
    *result_in_b = false;
    const int64_t items = n_dev ? cap : n_host;
    const int32_t nseg = seg ? seg->nseg : 0;
    const int64_t nb = sort_blocks(items) + nseg;
    if (sort_blocks(items) == 0) return hipSuccess;
    uint32_t *hist = reinterpret_cast<uint32_t *>(temp);
    const int64_t hlen = 256 * nb;
    const int64_t nparts = (hlen + kSortTile - 1) / kSortTile;
    uint32_t *parts = hist + hlen;
    SegDesc *segs = nullptr;
    if (seg) {
        const size_t off = ((size_t)(hlen + nparts + 1) * sizeof(uint32_t) + 255) & ~size_t(255);
        segs = reinterpret_cast<SegDesc *>(static_cast<char *>(temp) + off);
        hipLaunchKernelGGL(k_seg_table, dim3(1), dim3(kSegThreads), 0, st, seg->offs, seg->stride,
                           nseg, seg->views, n_dev, cap, segs);
    }
    uint32_t *ranges = seg && seg->nkeys > 0 ? seg->ranges : nullptr;
    const int passes = bits <= 8 ? 1 : (bits + 7) / 8;   // one pass at least: ranges come from it
    KT *ki = keys_a, *ko = keys_b;
    uint32_t *vi = vals_a, *vo = vals_b;
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * p;
        hipLaunchKernelGGL(k_radix_hist<KT>, dim3((unsigned)nb), dim3(kSortThreads), 0, st, ki, segs,
                           nseg, n_dev, cap, n_host, shift, hist);
        hipLaunchKernelGGL(k_hist_scan_reduce, dim3((unsigned)nparts), dim3(kSortThreads), 0,
                           st, hist, hlen, parts);
        hipLaunchKernelGGL(k_hist_scan_partials, dim3(1), dim3(kScanPartialsThreads), 0, st, parts,
                           nparts);
        hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nparts), dim3(kSortThreads), 0, st,
                           hist, hlen, parts, hist);
        // the keys of the last pass are not read again once the ranges are out
        const bool last = p == passes - 1;
        hipLaunchKernelGGL(k_radix_scatter<KT>, dim3((unsigned)nb), dim3(kSortThreads), 0, st, ki,
                           vi, last && ranges ? nullptr : ko, vo, hist, segs, nseg, n_dev, cap,
                           n_host, shift, last ? ranges : nullptr, seg ? seg->nkeys : 0,
                           last ? rank_out : nullptr);
        std::swap(ki, ko);
        std::swap(vi, vo);
        *result_in_b = !*result_in_b;
    }
    return hipGetLastError();
}

template hipError_t radix_sort_pairs<uint32_t>(uint32_t *, uint32_t *, uint32_t *, uint32_t *, int64_t,
                                               const unsigned long long *, int64_t, int, void *, bool *,
                                               hipStream_t, const SortSegments *, uint32_t *);
template hipError_t radix_sort_pairs<uint16_t>(uint16_t *, uint32_t *, uint16_t *, uint32_t *, int64_t,
                                               const unsigned long long *, int64_t, int, void *, bool *,
                                               hipStream_t, const SortSegments *, uint32_t *);

}  // namespace ss
