// Geometry-aware initialisation of the surfels on a DSM (SatSplat, arXiv 2606.28581, Sec.
// 3.4): each DSM cell gets an area weight a = |dx x dy| from its finite differences,
// surfel centres are drawn with probability proportional to a, and each surfel's frame is
// built by Gram-Schmidt against the local surface normal.
//
// DSM: node heights z[j][i] at (x0 + i g, y0 + j g); cell (j, i) spans nodes j..j+1,
// i..i+1, its tangents are (g, 0, dzx) and (0, g, dzy) with dzx, dzy the means of its two
// edge differences, a = g sqrt(dzx^2 + dzy^2 + g^2), normal (-dzx, -dzy, g) / sqrt(...).
// The weights are integers (65536 per flat cell: floor(65536 a / g^2 + 1/2)) and their
// prefix sums are uint64, so every sampling decision is exact; the geometry is FP64 from
// the FP32 heights.  Sample k draws Philox4x32-10 (Salmon et al., SC 2011; key = seed,
// counters (k, 0, 0, 0) and (k, 1, 0, 0)): the first two words pick the cell, the next
// two the position inside it (bilinear height), three more a random vector that
// Gram-Schmidt turns into t_u (t_v = n x t_u).  Scales are the surface-area spacing
// sqrt(area / N); opacity and albedo are given constants.
#include "ss_internal.h"
#include <algorithm>

namespace ss {

constexpr int kInitThreads = 256;
constexpr int kScanPer = 8;                                  // cells per thread in the scan
constexpr int kScanBlock = kInitThreads * kScanPer;          // cells per scan block
constexpr int kGroup = 32;                                   // cells per prefix entry: one line of weights
constexpr int kGroups = kScanBlock / kGroup;
constexpr double kWeightOne = 65536.0;

struct Philox4 {
    uint32_t v[4];
};

__device__ __forceinline__ Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1)
{
    constexpr uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
        const uint32_t hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
        const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += W0; k1 += W1;
    }
    return Philox4{{c0, c1, c2, c3}};
}

struct CellSlopes {
    double dzx, dzy, s;   // s = sqrt(dzx^2 + dzy^2 + g^2)
};

__device__ __forceinline__ CellSlopes cell_slopes(const float *__restrict__ z, int nx, int cj, int ci,
                                                  double g)
{
    const double z00 = z[(size_t)cj * nx + ci], z10 = z[(size_t)cj * nx + ci + 1];
    const double z01 = z[(size_t)(cj + 1) * nx + ci], z11 = z[(size_t)(cj + 1) * nx + ci + 1];
    CellSlopes c;
    c.dzx = 0.5 * ((z10 - z00) + (z11 - z01));
    c.dzy = 0.5 * ((z01 - z00) + (z11 - z10));
    c.s = sqrt(c.dzx * c.dzx + c.dzy * c.dzy + g * g);
    return c;
}

// The distribution is kept on three levels, so that a sample's search touches few lines far
// from it: the cells' weights, per group of kGroup cells the weight before it inside its
// block of kScanBlock cells, and per block the weight of the blocks before it.
//
// Weights, group prefixes and the block's total.  A thread evaluates every 256th cell of the
// block (coalesced heights), the scan takes 8 consecutive ones from LDS.  Cells past the
// last one weigh nothing.  Bound by the FP64 arithmetic per cell; one pass over z instead of
// a weight pass, two scan passes and a per-cell prefix of 8 bytes (16M cells: 212 us in four
// launches -> 60 us in two).
__global__ __launch_bounds__(kInitThreads) void k_dsm_weights(int nx, int ny, const float *__restrict__ z,
                                                              double g, uint32_t *__restrict__ w,
                                                              uint32_t *__restrict__ groups,
                                                              unsigned long long *__restrict__ totals)
{
    __shared__ uint32_t sw[kScanBlock];
    __shared__ unsigned long long wsum[kInitThreads / 64];
    const int64_t ncx = nx - 1, nc = ncx * (ny - 1);
    const int64_t c0 = (int64_t)blockIdx.x * kScanBlock;
    const uint32_t row0 = (uint32_t)(c0 / ncx), col0 = (uint32_t)(c0 % ncx);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        const uint32_t off = k * kInitThreads + threadIdx.x;
        uint32_t wt = 0;
        if (c0 + off < nc) {
            const uint32_t x = col0 + off, dr = x / (uint32_t)ncx;
            const CellSlopes s = cell_slopes(z, nx, (int)(row0 + dr), (int)(x - dr * (uint32_t)ncx), g);
            const double area = g * s.s;
            wt = (uint32_t)floor(area / (g * g) * kWeightOne + 0.5);
        }
        sw[off] = wt;
        w[c0 + off] = wt;      // w is padded to whole blocks
    }
    __syncthreads();
    unsigned long long sum = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) sum += sw[threadIdx.x * kScanPer + k];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long inc = sum;
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    unsigned long long before = inc - sum;
    for (int k = 0; k < wave; ++k) before += wsum[k];
    constexpr int kPer = kGroup / kScanPer;               // threads per group
    if (threadIdx.x % kPer == 0) groups[(int64_t)blockIdx.x * kGroups + threadIdx.x / kPer] = (uint32_t)before;
    if (threadIdx.x == kInitThreads - 1) totals[blockIdx.x] = before + sum;
}

// Exclusive scan of the block totals in place by one block; totals[nblocks] gets the sum.
constexpr int kOffThreads = 1024, kOffPer = 4;

__global__ __launch_bounds__(kOffThreads) void k_scan_offsets(unsigned long long *__restrict__ totals,
                                                              int64_t nblocks)
{
    __shared__ unsigned long long wsum[kOffThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long carry = 0;
    for (int64_t b0 = 0; b0 < nblocks; b0 += kOffThreads * kOffPer) {
        const int64_t i = b0 + (int64_t)threadIdx.x * kOffPer;
        unsigned long long v[kOffPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kOffPer; ++k) {
            v[k] = i + k < nblocks ? totals[i + k] : 0ull;
            sum += v[k];
        }
        unsigned long long inc = sum;
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned long long y = __shfl_up(inc, d, 64);
            if (lane >= d) inc += y;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        unsigned long long run = carry + inc - sum;
        for (int k = 0; k < kOffThreads / 64; ++k) {
            if (k < wave) run += wsum[k];
            carry += wsum[k];
        }
#pragma unroll
        for (int k = 0; k < kOffPer; ++k) {
            if (i + k < nblocks) totals[i + k] = run;
            run += v[k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) totals[nblocks] = carry;
}

// Index of the last of n ascending values that is <= t (the first one is)
template <typename T, typename I>
__device__ __forceinline__ I last_not_above(const T *__restrict__ v, I n, T t)
{
    I lo = 0, hi = n - 1;
    while (lo < hi) {
        const I mid = (lo + hi + 1) >> 1;
        if (v[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// r % d for any r and d >= 2^16, with 1 / d rounded to double: the quotient is below 2^48,
// so its estimate is off by at most one.
__device__ __forceinline__ unsigned long long mod_by(unsigned long long r, unsigned long long d, double inv)
{
    unsigned long long m = r - (unsigned long long)((double)r * inv) * d;
    if ((long long)m < 0) m += d;
    return m >= d ? m - d : m;
}

// One sample per thread and turn; blocks are persistent and hold (up to kTop of) the block
// offsets in LDS.  A binary search per sample over a per-cell prefix walks 24 levels of a
// 128 MB array; every level is a load whose 64 lanes hit 64 lines, at one line per clock and
// CU.  The search here runs in LDS down to a block of 2048 cells, then over 256 bytes of
// group prefixes and one line of weights.  What is left is one line of weights and two of
// heights per sample, 2.3 GB with the outputs at about the rate of a device copy (5M samples
// of 16M cells: 970 -> 406 us; with the block search in memory 538, groups of 16 cells with
// 8-byte prefixes 508).
constexpr int kTop = 8192, kSampleThreads = 1024;

__global__ __launch_bounds__(kSampleThreads) void k_dsm_sample(
    int nx, int ny, const float *__restrict__ z, double x0, double y0, double g,
    const uint32_t *__restrict__ w, const uint32_t *__restrict__ groups,
    const unsigned long long *__restrict__ offsets, int64_t nblocks, int64_t nc, int64_t n,
    uint32_t key0, uint32_t key1,
    float opacity, float albedo, float *__restrict__ mean, float *__restrict__ tu,
    float *__restrict__ tv, float *__restrict__ scale, float *__restrict__ opac,
    float *__restrict__ alb, int64_t *__restrict__ cell_out)
{
    __shared__ unsigned long long top[kTop];
    const int64_t step = (nblocks + kTop - 1) / kTop;       // blocks per entry
    const int ntop = (int)((nblocks + step - 1) / step);
    for (int i = threadIdx.x; i < ntop; i += kSampleThreads) top[i] = offsets[i * step];
    __syncthreads();
    const unsigned long long total = offsets[nblocks];
    const double inv_total = 1.0 / (double)total;
    const float sp = (float)sqrt((double)total * g * g / kWeightOne / (double)n);
    const int64_t ncx = nx - 1;
    for (int64_t k = (int64_t)blockIdx.x * kSampleThreads + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * kSampleThreads) {
        const Philox4 a = philox4x32_10((uint32_t)k, 0u, 0u, 0u, key0, key1);
        const Philox4 b = philox4x32_10((uint32_t)k, 1u, 0u, 0u, key0, key1);
        const unsigned long long r64 = ((unsigned long long)a.v[1] << 32) | a.v[0];
        const unsigned long long t = total >= 65536ull ? mod_by(r64, total, inv_total) : r64 % total;
        // first cell whose cumulative weight exceeds t: the last block and group that start at or
        // below t hold it, and in the group every cell whose running sum stays at or below t
        // comes before it
        const int entry = last_not_above((const unsigned long long *)top, ntop, t);
        int64_t b0 = entry * step;
        if (step > 1) b0 += last_not_above(offsets + b0, min(step, nblocks - b0), t);
        unsigned long long rem = t - offsets[b0];
        int64_t q = b0 * kGroups;
        if (offsets[b0 + 1] - offsets[b0] <= 0xFFFFFFFFull) {
            q += last_not_above(groups + q, kGroups, (uint32_t)rem);
            rem -= groups[q];
        } else {
            // slopes steep enough that a block's weight leaves 32 bits: cell by cell
            for (int e = 0; e < kScanBlock - kGroup; e += kGroup, ++q) {
                unsigned long long sum = 0;
                for (int k2 = 0; k2 < kGroup; ++k2) sum += w[q * kGroup + k2];
                if (sum > rem) break;
                rem -= sum;
            }
        }
        const uint4 *wq = reinterpret_cast<const uint4 *>(w + q * kGroup);
        uint4 x[kGroup / 4];
#pragma unroll
        for (int e = 0; e < kGroup / 4; ++e) x[e] = wq[e];
        unsigned long long run = 0;
        int before = 0;
#pragma unroll
        for (int e = 0; e < kGroup / 4; ++e) {
            run += x[e].x; before += run <= rem;
            run += x[e].y; before += run <= rem;
            run += x[e].z; before += run <= rem;
            run += x[e].w; before += run <= rem;
        }
        const int64_t lo = min(q * kGroup + before, nc - 1);
        const int cj = (int)(lo / ncx), ci = (int)(lo - cj * ncx);
        const double fx = (double)a.v[2] / 4294967296.0, fy = (double)a.v[3] / 4294967296.0;
        const double z00 = z[(size_t)cj * nx + ci], z10 = z[(size_t)cj * nx + ci + 1];
        const double z01 = z[(size_t)(cj + 1) * nx + ci], z11 = z[(size_t)(cj + 1) * nx + ci + 1];
        const double zz = (z00 * (1.0 - fx) + z10 * fx) * (1.0 - fy) + (z01 * (1.0 - fx) + z11 * fx) * fy;
        mean[3 * k] = (float)(x0 + ((double)ci + fx) * g);
        mean[3 * k + 1] = (float)(y0 + ((double)cj + fy) * g);
        mean[3 * k + 2] = (float)zz;
        const CellSlopes s = cell_slopes(z, nx, cj, ci, g);
        const double is = 1.0 / s.s;
        const double nn[3] = {-s.dzx * is, -s.dzy * is, g * is};
        double r[3] = {(double)b.v[0] / 2147483648.0 - 1.0, (double)b.v[1] / 2147483648.0 - 1.0,
                       (double)b.v[2] / 2147483648.0 - 1.0};
        double rn = r[0] * nn[0] + r[1] * nn[1] + r[2] * nn[2];
        double u[3] = {r[0] - rn * nn[0], r[1] - rn * nn[1], r[2] - rn * nn[2]};
        double ul = sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
        if (ul < 1e-6) {   // the random vector lies along the normal: use the x axis
            u[0] = 1.0 - nn[0] * nn[0];
            u[1] = -nn[1] * nn[0];
            u[2] = -nn[2] * nn[0];
            ul = sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
        }
        const double iul = 1.0 / ul;
        for (int c = 0; c < 3; ++c) u[c] *= iul;
        const double v[3] = {nn[1] * u[2] - nn[2] * u[1], nn[2] * u[0] - nn[0] * u[2], nn[0] * u[1] - nn[1] * u[0]};
        for (int c = 0; c < 3; ++c) {
            tu[3 * k + c] = (float)u[c];
            tv[3 * k + c] = (float)v[c];
            alb[3 * k + c] = albedo;
        }
        scale[2 * k] = sp;
        scale[2 * k + 1] = sp;
        opac[k] = opacity;
        if (cell_out) cell_out[k] = lo;
    }
}

static inline int64_t dsm_cells(int nx, int ny) { return (int64_t)(nx - 1) * (ny - 1); }
static inline int64_t scan_blocks(int64_t nc) { return (nc + kScanBlock - 1) / kScanBlock; }

// Workspace: weights (padded to whole blocks), group prefixes, block offsets and their sum
struct DsmLayout {
    size_t groups, offsets, total;
};

static DsmLayout dsm_layout(int nx, int ny)
{
    const size_t nb = (size_t)scan_blocks(dsm_cells(nx, ny));
    auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
    DsmLayout L;
    L.groups = al(nb * kScanBlock * 4);
    L.offsets = L.groups + al(nb * kGroups * 4);
    L.total = L.offsets + al((nb + 1) * 8);
    return L;
}

size_t dsm_init_workspace_bytes(int nx, int ny) { return dsm_layout(nx, ny).total; }

hipError_t launch_dsm_init(int nx, int ny, const float *z, double x0, double y0, double g, int64_t n,
                           uint64_t seed, float opacity, float albedo, void *ws, float *mean,
                           float *tu, float *tv, float *scale, float *opac, float *alb,
                           int64_t *cell, hipStream_t st)
{
    const int64_t nc = dsm_cells(nx, ny), nb = scan_blocks(nc);
    const DsmLayout L = dsm_layout(nx, ny);
    char *p = static_cast<char *>(ws);
    uint32_t *w = reinterpret_cast<uint32_t *>(p);
    uint32_t *groups = reinterpret_cast<uint32_t *>(p + L.groups);
    unsigned long long *offsets = reinterpret_cast<unsigned long long *>(p + L.offsets);
    hipLaunchKernelGGL(k_dsm_weights, dim3((unsigned)nb), dim3(kInitThreads), 0, st, nx, ny, z, g, w,
                       groups, offsets);
    hipLaunchKernelGGL(k_scan_offsets, dim3(1), dim3(kOffThreads), 0, st, offsets, nb);
    // two blocks per CU fill its wave slots and share its LDS
    const int64_t sample_blocks = std::min<int64_t>((n + kSampleThreads - 1) / kSampleThreads, 512);
    if (n > 0)
        hipLaunchKernelGGL(k_dsm_sample, dim3((unsigned)sample_blocks), dim3(kSampleThreads), 0, st, nx, ny, z, x0, y0, g, w, groups, offsets, nb, nc, n,
                           (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32), opacity, albedo, mean,
                           tu, tv, scale, opac, alb, cell);
    return hipGetLastError();
}

}  // namespace ss
