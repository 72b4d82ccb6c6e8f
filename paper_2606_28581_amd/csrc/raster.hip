// Affine-camera 2D Gaussian surfel rasterizer for gfx950 (SatSplat, arXiv 2606.28581,
// Sec. 3.2-3.3): projection, binning, forward compositing, backward adjoint.
//
// Work is organised in depth-rank space: after the global centre-depth sort the
// surfel parameters are gathered once into rank order, so projection, the pair-count
// scan and the (view, rank) records are contiguous, and tile lists hold ranks.
#include "ss_internal.h"
#include <algorithm>
#include <cmath>

namespace ss {

constexpr float kNegHalfLog2e = -0.72134752044448170f;   // -0.5 * log2(e)
constexpr int kParamFloats = 16;                          // gathered surfel: 4 x float4

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ int find_view(const ViewDesc *views, int nv, int tile)
{
    int lo = 0, hi = nv - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (views[mid].tile_off <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------- into rank order
// sorted[rank[i]] = (p, t_u, t_v, s_u, s_v, o, albedo, 0) of surfel i, 16 floats.  Reading by
// rank order would fetch a line from each of six arrays per surfel for 60 bytes; here the
// arrays are read in order, a block's rows are put together in LDS and each leaves as one
// 64-byte piece (1M surfels: 116 -> 36 us, 2M: 245 -> 73 us).
constexpr int kPermBlock = 256;
constexpr int kPermRow = kParamFloats + 1;            // padded LDS row

template <int C>
__device__ __forceinline__ void rows_in(const float *__restrict__ src, int64_t i0, int cnt, int col,
                                        float *rows)
{
    for (int e = threadIdx.x; e < cnt * C; e += kPermBlock) rows[(e / C) * kPermRow + col + e % C] = src[i0 * C + e];
}

template <int C>
__device__ __forceinline__ void rows_out(const float *rows, int64_t i0, int cnt, int col,
                                         float *__restrict__ dst)
{
    for (int e = threadIdx.x; e < cnt * C; e += kPermBlock) dst[i0 * C + e] = rows[(e / C) * kPermRow + col + e % C];
}

__global__ __launch_bounds__(kPermBlock) void k_gather_params(const uint32_t *__restrict__ rank, SurfelPtrs s,
                                                              float4 *__restrict__ out)
{
    __shared__ float rows[kPermBlock * kPermRow];
    const int64_t i0 = (int64_t)blockIdx.x * kPermBlock;
    const int cnt = (int)min((int64_t)kPermBlock, s.n - i0);
    rows_in<3>(s.mean, i0, cnt, 0, rows);
    rows_in<3>(s.t_u, i0, cnt, 3, rows);
    rows_in<3>(s.t_v, i0, cnt, 6, rows);
    rows_in<2>(s.scale, i0, cnt, 9, rows);
    rows_in<1>(s.opacity, i0, cnt, 11, rows);
    rows_in<3>(s.albedo, i0, cnt, 12, rows);
    __syncthreads();
    for (int e = threadIdx.x; e < cnt * 4; e += kPermBlock) {
        const uint32_t r = rank[i0 + (e >> 2)];
        const float *p = rows + (e >> 2) * kPermRow + 4 * (e & 3);
        const float4 x = make_float4(p[0], p[1], p[2], (e & 3) == 3 ? 0.f : p[3]);
        if (r < s.n) out[4 * (int64_t)r + (e & 3)] = x;   // always: ranks are a permutation
    }
}

hipError_t launch_gather_params(const uint32_t *rank, const SurfelPtrs &s, float *out,
                                hipStream_t st)
{
    if (s.n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_params, dim3((unsigned)((s.n + kPermBlock - 1) / kPermBlock)),
                       dim3(kPermBlock), 0, st, rank, s, reinterpret_cast<float4 *>(out));
    return hipGetLastError();
}

// Affine projection of one surfel's tangent frame (Sec. 3.2, Eqs. affine2dgs_uv2screen,
// affine2dgs_Qq): M = [s_u t_u, s_v t_v], T = B M, Q = T^-1 (zero when T is degenerate),
// and the sign that orients the normal m = t_u x t_v against the viewing direction
// d = B_x x B_y taken looking down (d_z < 0).  FP64; the projection and its backward both
// call it, so the backward sees the very Q and sign the forward used.
struct SurfelAffine {
    double M[3][2], T[2][2], Q[2][2], m[3];
    double nsign;
    bool deg;
};

__device__ __forceinline__ SurfelAffine surfel_affine(const double (&B)[2][3], const double (&tu)[3],
                                                      const double (&tv)[3], double su, double sv,
                                                      double det_rel_eps)
{
    SurfelAffine a;
    for (int i = 0; i < 3; ++i) { a.M[i][0] = su * tu[i]; a.M[i][1] = sv * tv[i]; }
    for (int row = 0; row < 2; ++row)
        for (int q = 0; q < 2; ++q) {
            double acc = 0.0;
            for (int i = 0; i < 3; ++i) acc += B[row][i] * a.M[i][q];
            a.T[row][q] = acc;
        }
    const double(&T)[2][2] = a.T;
    const double det = T[0][0] * T[1][1] - T[0][1] * T[1][0];
    const double fro2 = T[0][0] * T[0][0] + T[0][1] * T[0][1] + T[1][0] * T[1][0] + T[1][1] * T[1][1];
    a.deg = !(fabs(det) > det_rel_eps * fro2);
    a.Q[0][0] = a.Q[0][1] = a.Q[1][0] = a.Q[1][1] = 0.0;
    if (!a.deg) {
        a.Q[0][0] = T[1][1] / det; a.Q[0][1] = -T[0][1] / det;
        a.Q[1][0] = -T[1][0] / det; a.Q[1][1] = T[0][0] / det;
    }
    a.m[0] = tu[1] * tv[2] - tu[2] * tv[1];
    a.m[1] = tu[2] * tv[0] - tu[0] * tv[2];
    a.m[2] = tu[0] * tv[1] - tu[1] * tv[0];
    double dvec[3] = {B[0][1] * B[1][2] - B[0][2] * B[1][1], B[0][2] * B[1][0] - B[0][0] * B[1][2],
                      B[0][0] * B[1][1] - B[0][1] * B[1][0]};
    if (dvec[2] > 0) { dvec[0] = -dvec[0]; dvec[1] = -dvec[1]; dvec[2] = -dvec[2]; }
    const double nd = a.m[0] * dvec[0] + a.m[1] * dvec[1] + a.m[2] * dvec[2];
    a.nsign = nd > 0 ? -1.0 : 1.0;
    return a;
}

// ------------------------------------------------------------------- projection
// One thread per rank r and VPT views.  Geometry in FP64 (the binning contract: tile
// ranges must be bit-identical to an FP64 reference), records rounded to FP32.
//   T = B'_xy [s_u t_u, s_v t_v]   c = B'_xy p + b'_xy   Q = T^-1   (Eq. affine2dgs_Qq)
//   degenerate iff |det T| <= eps |T|_F^2 ("Degenerate Solutions")
//   support: alpha >= alpha_min needs rho <= 2 ln(o / alpha_min); the uv-ellipse
//   {T w : |w|^2 <= rho_max} has x half-extent r |T row 0|, the low-pass disk radius
//   sigma r; pixel i is in the box iff i + 0.5 lies within the half-extent of c.
// Bound by its writes (128 + 8 bytes per view record, 64 + 8 per sun record) once the FP64
// work that all views of a surfel share - the logarithm of r, the normal's root and division,
// products of the frame - is done for four of them at a time: 2M surfels x (40 views + 40
// suns) 3.88 -> 3.39 ms (4.9 TB/s), x (8 + 8) of 500k 220 -> 177 us, 20 suns of 1M 465 -> 405 us.
// Eight views at a time: 3.49 ms and 181 us.  View records at their 96 bytes instead of 128-byte
// slots: 2.85 ms, which the raster kernels' gathers, then over two lines, give back.
template <int VPT>
__global__ __launch_bounds__(256) void k_project(
    const float4 *__restrict__ sp, int64_t n, int32_t nv,
    const ViewDesc *__restrict__ views, const float *__restrict__ Fxy,
    const float *__restrict__ dF, const SunCam *__restrict__ sun,
    const float *__restrict__ vis_rank, float bz, int ts, RasterConsts rc,
    float4 *__restrict__ rec, short4 *__restrict__ tiles, uint32_t *__restrict__ counts,
    uint32_t *__restrict__ sums, const uint32_t *__restrict__ tmask, uint2 *__restrict__ ranges,
    int64_t nranges)
{
    // empty ranges for the tile sort
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nranges;
         i += (int64_t)gridDim.x * blockDim.x)
        ranges[i] = make_uint2(0xFFFFFFFFu, 0u);
    // The block's 256 records are staged in LDS and written back as one contiguous run per view.
    // Blocks run view-innermost (block = rank block x groups of VPT views + group), in
    // xcd_tile's chunked order, so the views of one rank block share the surfel parameters in
    // one L2.
    __shared__ float4 srec[256 * kRecVec4];
    __shared__ unsigned long long wsum[kRankBlock / 64];
    const int64_t L = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int groups = (nv + VPT - 1) / VPT;
    const int64_t rb = L / groups, r0 = rb * blockDim.x;
    const int v0 = (int)(L - rb * groups) * VPT;
    const bool valid = r0 + threadIdx.x < n;
    const int64_t r = valid ? r0 + threadIdx.x : n - 1;   // lanes past the end repeat the last
    const float4 pa = sp[4 * r], pb = sp[4 * r + 1], pc = sp[4 * r + 2], pd = sp[4 * r + 3];
    const double p[3] = {pa.x, pa.y, pa.z};
    const double tu[3] = {pa.w, pb.x, pb.y};
    const double tv[3] = {pb.z, pb.w, pc.x};
    const double su = pc.y, sv = pc.z, o = pc.w;
    // the same for every view: the support radius and the normal up to its sign
    const double rr = o >= rc.alpha_min_d ? sqrt(2.0 * log(o / rc.alpha_min_d)) : 0.0;
    float nrm[3];
    {
        const double m[3] = {tu[1] * tv[2] - tu[2] * tv[1], tu[2] * tv[0] - tu[0] * tv[2],
                             tu[0] * tv[1] - tu[1] * tv[0]};
        const double s = 1.0 / sqrt(m[0] * m[0] + m[1] * m[1] + m[2] * m[2]);
        for (int k = 0; k < 3; ++k) nrm[k] = (float)(s * m[k]);
    }
#pragma unroll 1
    for (int v = v0; v < min(v0 + VPT, nv); ++v) {
        if (VPT > 1 && v > v0) __syncthreads();           // the last view's records are out
        const ViewDesc vd = views[v];
        double B[2][3], b[2];
        if (sun) {
            for (int q = 0; q < 3; ++q) { B[0][q] = sun[v].B[q]; B[1][q] = sun[v].B[3 + q]; }
            b[0] = sun[v].b[0]; b[1] = sun[v].b[1];
        } else {
            for (int row = 0; row < 2; ++row) {
                for (int q = 0; q < 3; ++q)
                    B[row][q] = (double)Fxy[8 * v + 4 * row + q] +
                                (dF ? (double)dF[8 * v + 4 * row + q] : 0.0);
                b[row] = (double)Fxy[8 * v + 4 * row + 3] + (dF ? (double)dF[8 * v + 4 * row + 3] : 0.0);
            }
        }
        const SurfelAffine sa = surfel_affine(B, tu, tv, su, sv, rc.det_rel_eps_d);
        const double(&M)[3][2] = sa.M;
        const double(&T)[2][2] = sa.T;
        const double(&Q)[2][2] = sa.Q;
        const bool deg = sa.deg;
        const double nsign = sa.nsign;
        double c[2];
        for (int row = 0; row < 2; ++row) {
            double acc = b[row];
            for (int i = 0; i < 3; ++i) acc += B[row][i] * p[i];
            c[row] = acc;
        }
        const bool filt = (rc.lowpass_mode == 0) || deg;
        // support box -> pixel and tile ranges
        int ilo = 0, ihi = -1, jlo = 0, jhi = -1;
        if (o >= rc.alpha_min_d) {
            double hx = 0.0, hy = 0.0;
            if (!deg) {
                hx = rr * sqrt(T[0][0] * T[0][0] + T[0][1] * T[0][1]);
                hy = rr * sqrt(T[1][0] * T[1][0] + T[1][1] * T[1][1]);
            }
            if (filt) {
                const double f = rc.sigma_d * rr;
                if (f > hx) hx = f;
                if (f > hy) hy = f;
            }
            double xl = ceil(c[0] - hx - 0.5), xh = floor(c[0] + hx - 0.5);
            double yl = ceil(c[1] - hy - 0.5), yh = floor(c[1] + hy - 0.5);
            if (isfinite(xl) && isfinite(xh) && isfinite(yl) && isfinite(yh)) {
                if (xl < 0) xl = 0;
                if (yl < 0) yl = 0;
                if (xh > vd.W - 1) xh = vd.W - 1;
                if (yh > vd.H - 1) yh = vd.H - 1;
                if (xl <= xh && yl <= yh) {
                    ilo = (int)xl; ihi = (int)xh; jlo = (int)yl; jhi = (int)yh;
                }
            }
        }
        const int64_t slot = (int64_t)v * n + r;
        short4 tl;
        uint32_t cnt = 0;
        if (ilo <= ihi) {
            tl.x = (short)(ilo / ts); tl.y = (short)(ihi / ts);
            tl.z = (short)(jlo / ts); tl.w = (short)(jhi / ts);
            if (tmask) {
                for (int ty = tl.z; ty <= tl.w; ++ty)
                    for (int tx = tl.x; tx <= tl.y; ++tx)
                        cnt += tmask[vd.tile_off + ty * vd.tiles_x + tx] != 0u;
            } else {
                cnt = (uint32_t)(tl.y - tl.x + 1) * (uint32_t)(tl.w - tl.z + 1);
            }
        } else {
            tl.x = 0; tl.y = -1; tl.z = 0; tl.w = -1;
        }
        if (valid) {
            tiles[slot] = tl;
            if (tmask) counts[slot] = cnt;
        } else {
            cnt = 0;
        }
        // the block's pair count, clamped
        {
            unsigned long long x = cnt;
            for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
            if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = x;
        }
        // record
        const float chx = (float)c[0], chy = (float)c[1];
        const uint32_t boxx = ((uint32_t)(uint16_t)ilo) | ((uint32_t)(uint16_t)ihi << 16);
        const uint32_t boxy = ((uint32_t)(uint16_t)jlo) | ((uint32_t)(uint16_t)jhi << 16);
        const float inf = __builtin_inff();
        float4 *R = srec + kRecVec4 * threadIdx.x;
        R[0] = make_float4(__uint_as_float(boxx), __uint_as_float(boxy), chx, chy);
        R[1] = make_float4((float)(c[0] - (double)chx), (float)(c[1] - (double)chy),
                           deg ? inf : 0.f, filt ? 0.f : inf);
        R[2] = make_float4((float)Q[0][0], (float)Q[0][1], (float)Q[1][0], (float)Q[1][1]);
        R[3] = make_float4((float)o, (float)((double)bz - p[2]), (float)M[2][0], (float)M[2][1]);
        const float vv = vis_rank ? vis_rank[r * nv + v] : 1.f;
        R[4] = make_float4(pd.x, pd.y, pd.z, vv);
        const float sg = (float)nsign;                    // +-1: the products are exact
        R[5] = make_float4(sg * nrm[0], sg * nrm[1], sg * nrm[2], sg);
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long x = wsum[0] + wsum[1] + wsum[2] + wsum[3];
            sums[(int64_t)v * rank_blocks(n) + rb] = (uint32_t)min(x, 0xFFFFFFFFull);
        }
        const int64_t nrec = min((int64_t)blockDim.x, n - r0);
        // whole slots, so every written line is written in full
        if (sun) {
            float4 *dst = rec + ((size_t)v * (size_t)n + (size_t)r0) * kSunRecStride4;
            for (int i = threadIdx.x; i < nrec * kSunRecStride4; i += blockDim.x)
                dst[i] = srec[(i >> 2) * kRecVec4 + (i & 3)];
        } else {
            float4 *dst = rec + ((size_t)v * (size_t)n + (size_t)r0) * kRecStride4;
            for (int i = threadIdx.x; i < nrec * kRecStride4; i += blockDim.x) {
                const int k = i & 7;
                dst[i] = k < kRecVec4 ? srec[(i >> 3) * kRecVec4 + k] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    }
}

hipError_t launch_project(const float *sorted, int64_t n, int32_t nv, const ViewDesc *views,
                          const float *Fxy, const float *dF, const SunCam *sun,
                          const float *vis_rank, float bz, int ts, const RasterConsts &rc,
                          float *rec, short4 *tiles, uint32_t *counts, uint32_t *sums,
                          const uint32_t *tmask, uint32_t *ranges, int64_t nranges, hipStream_t st)
{
    if (n <= 0)      // nothing to project: empty tiles only
        return ranges ? fill_u32(ranges, 0u, 2 * nranges, st) : hipSuccess;
    const int64_t blocks = rank_blocks(n) * nv;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
#define SS_PROJECT(VPT_, BLOCKS_)                                                                      \
    hipLaunchKernelGGL((k_project<VPT_>), dim3((unsigned)(BLOCKS_)), dim3(kRankBlock), 0, st,          \
                       reinterpret_cast<const float4 *>(sorted), n, nv, views, Fxy, dF, sun, vis_rank, \
                       bz, ts, rc, reinterpret_cast<float4 *>(rec), tiles, counts, sums, tmask,        \
                       reinterpret_cast<uint2 *>(ranges), ranges ? nranges : 0)
    // four views a block once that still leaves 8 blocks for every CU
    const int64_t grouped = rank_blocks(n) * ((nv + 3) / 4);
    if (nv >= 4 && grouped >= 2048) SS_PROJECT(4, grouped);
    else SS_PROJECT(1, blocks);
#undef SS_PROJECT
    return hipGetLastError();
}

// Visibility arrives per view in surfel order; the projection reads it per rank.  The
// depth order is one permutation for all views, so one pass over surfels k (coalesced
// reads of every view's vis[v][k]) writes the nv values of surfel k contiguously at its
// rank: out[rank(k) * nv + v].
// A block transposes a chunk of surfels through LDS (rows padded to nv + 1 floats):
// reads run along k per view, writes along v per surfel (one contiguous run each).
__global__ __launch_bounds__(256) void k_vis_to_rank(const float *__restrict__ vis, int64_t n,
                                                     int32_t nv, int chunk,
                                                     const uint32_t *__restrict__ rank,
                                                     float *__restrict__ out)
{
    extern __shared__ float sv[];
    const int64_t k0 = (int64_t)blockIdx.x * chunk;
    const int cnt = (int)min((int64_t)chunk, n - k0);
    const int row = nv + 1;
    for (int i = threadIdx.x; i < cnt * nv; i += blockDim.x) {
        const int v = i / cnt, kk = i - v * cnt;
        sv[kk * row + v] = vis[(int64_t)v * n + k0 + kk];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < cnt * nv; i += blockDim.x) {
        const int kk = i / nv, v = i - kk * nv;
        const uint32_t r = min(rank[k0 + kk], (uint32_t)(n - 1));
        out[(int64_t)r * nv + v] = sv[kk * row + v];
    }
}

hipError_t launch_vis_to_rank(const float *vis, int64_t n, int32_t nv, const uint32_t *rank, float *out,
                              hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (nv <= 0) return hipSuccess;
    // chunk x (nv + 1) floats of LDS, at most 64 KB
    const int chunk = (int)std::max<int64_t>(1, std::min<int64_t>(64, 16384 / (nv + 1)));
    const size_t lds = (size_t)chunk * (nv + 1) * sizeof(float);
    hipLaunchKernelGGL(k_vis_to_rank, dim3((unsigned)((n + chunk - 1) / chunk)), dim3(256), lds, st,
                       vis, n, nv, chunk, rank, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------------ emit
// One thread per kEmitRanks consecutive ranks of a view: one (tile id, rank) pair per overlapped
// tile.  A block's ranks own one contiguous run of the output, which starts at the scanned
// pair sum of its first kRankBlock; inside it the threads' places come from a scan of their
// counts here (the tile rectangles give them, or `counts` where a tile mask cut them).  Runs of up to kEmitStage pairs are
// assembled in LDS and written out coalesced, longer ones go straight to memory.  Pairs
// beyond the bound capacity are dropped (the scan already raised the overflow flag).
// Bound by the latency of a block's few steps: two ranks a thread halve the blocks (2M surfels
// x (40 views + 40 sun maps) 1.28 -> 0.84 ms, 1M x 20 sun maps 195 -> 166 us); four make the
// large sizes 0.76 ms and 157 us, but leave one view of 1M too few blocks (30 -> 42 us).
constexpr int kEmitThreads = kRankBlock, kEmitRanks = 2;
constexpr int kEmitStage = 2048;

template <typename KT>
__global__ __launch_bounds__(kEmitThreads) void k_emit(
    int64_t n, const ViewDesc *__restrict__ views, const short4 *__restrict__ tiles,
    const uint32_t *__restrict__ counts, const uint32_t *__restrict__ base, uint64_t cap,
    KT *__restrict__ keys, uint32_t *__restrict__ vals, const uint32_t *__restrict__ tmask)
{
    constexpr bool kLocal = sizeof(KT) == 2;   // tile id within the view, else global
    __shared__ KT sk[kEmitStage];
    __shared__ uint32_t sv[kEmitStage];
    __shared__ uint32_t lds_w[kEmitThreads / 64];
    const int v = blockIdx.y;
    const int64_t r0 = ((int64_t)blockIdx.x * kEmitThreads + threadIdx.x) * kEmitRanks;
    const uint64_t b_lo = base[(int64_t)v * rank_blocks(n) + kEmitRanks * (int64_t)blockIdx.x];
    const ViewDesc vd = views[v];
    short4 ts[kEmitRanks];
    uint32_t cnt = 0;
#pragma unroll
    for (int k = 0; k < kEmitRanks; ++k) {
        ts[k] = r0 + k < n ? tiles[(int64_t)v * n + r0 + k] : make_short4(0, -1, 0, -1);
        if (counts) cnt += r0 + k < n ? counts[(int64_t)v * n + r0 + k] : 0u;
        else cnt += (uint32_t)(ts[k].y - ts[k].x + 1) * (uint32_t)(ts[k].w - ts[k].z + 1);
    }
    uint32_t total;
    const uint32_t before = block_exclusive_scan(cnt, lds_w, &total);
    const bool staged = total <= (uint32_t)kEmitStage;   // uniform over the block
    uint64_t l = before;
#pragma unroll
    for (int k = 0; k < kEmitRanks; ++k) {
        const short4 t = ts[k];
        const uint32_t r = (uint32_t)(r0 + k);
        for (int ty = t.z; ty <= t.w; ++ty)
            for (int tx = t.x; tx <= t.y; ++tx) {
                const uint32_t lkey = (uint32_t)(ty * vd.tiles_x + tx);
                const uint32_t gkey = (uint32_t)vd.tile_off + lkey;
                if (tmask && tmask[gkey] == 0u) continue;
                const KT key = (KT)(kLocal ? lkey : gkey);
                if (!staged) {
                    if (b_lo + l < cap) {
                        keys[b_lo + l] = key;
                        vals[b_lo + l] = r;
                    }
                } else if (l < (uint64_t)kEmitStage) {
                    sk[l] = key;
                    sv[l] = r;
                }
                ++l;
            }
    }
    if (!staged) return;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < total; i += kEmitThreads) {
        if (b_lo + i < cap) {
            keys[b_lo + i] = sk[i];
            vals[b_lo + i] = sv[i];
        }
    }
}

hipError_t launch_emit(int64_t n, int32_t nv, const ViewDesc *views, const short4 *tiles,
                       const uint32_t *counts, const uint32_t *base, uint64_t cap, void *keys,
                       bool keys16, uint32_t *vals, const uint32_t *tmask, hipStream_t st)
{
    if (n <= 0 || cap == 0) return hipSuccess;
    const dim3 grid((unsigned)((rank_blocks(n) + kEmitRanks - 1) / kEmitRanks), (unsigned)nv);
    const uint32_t *cn = tmask ? counts : nullptr;
    if (keys16)
        hipLaunchKernelGGL(k_emit<uint16_t>, grid, dim3(kEmitThreads), 0, st, n, views, tiles, cn, base,
                           cap, static_cast<uint16_t *>(keys), vals, tmask);
    else
        hipLaunchKernelGGL(k_emit<uint32_t>, grid, dim3(kEmitThreads), 0, st, n, views, tiles, cn, base,
                           cap, static_cast<uint32_t *>(keys), vals, tmask);
    return hipGetLastError();
}

// ------------------------------------------------------------ tile dispatch order
// Block b of a raster launch runs on XCD b % 8 as that XCD's (b / 8)-th block.  XCD x
// owns the blocks b = 8 i + x, i < n_x, and xcd_tile<CHUNKED>(b) names the tile each one
// rasterizes; the order below keeps that tile set per XCD and renumbers i so that the
// heavy tiles (list length >= 2 x mean) come first.  Three passes over (x, block of
// kOrdBlock consecutive i): count heavy tiles, scan the counts per XCD, write.
constexpr int kOrdBlock = 1024;

int tile_order_blocks(int32_t ntiles)
{
    const int per_xcd = (ntiles + 7) / 8;
    return (per_xcd + kOrdBlock - 1) / kOrdBlock;
}

template <bool CHUNKED>
__device__ __forceinline__ bool heavy_tile(const uint32_t *ranges, int32_t ntiles,
                                           unsigned long long total, int x, int i, int &tile)
{
    const int b = 8 * i + x;
    if (b >= ntiles) { tile = -1; return false; }
    tile = xcd_tile<CHUNKED>(b, ntiles);
    const uint2 r = tile_range(ranges, tile);
    const uint64_t len = r.y - r.x;
    // len >= 2 total / ntiles without division
    return len * (uint64_t)ntiles >= 2ull * total && len > 0;
}

template <bool CHUNKED>
__global__ __launch_bounds__(kOrdBlock) void k_order_count(const uint32_t *__restrict__ ranges,
                                                           int32_t ntiles,
                                                           const unsigned long long *__restrict__ total,
                                                           uint32_t *__restrict__ parts)
{
    __shared__ uint32_t wsum[kOrdBlock / 64];
    const int x = blockIdx.y, i = blockIdx.x * kOrdBlock + threadIdx.x;
    int tile;
    const bool h = heavy_tile<CHUNKED>(ranges, ntiles, *total, x, i, tile);
    const uint64_t bal = __ballot(h);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = (uint32_t)__popcll(bal);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t s = 0;
        for (int w = 0; w < kOrdBlock / 64; ++w) s += wsum[w];
        parts[x * gridDim.x + blockIdx.x] = s;
    }
}

// One block per XCD: exclusive scan of its block counts in place; parts[8 nblk + x] gets
// the XCD's heavy total.
__global__ __launch_bounds__(256) void k_order_scan(uint32_t *__restrict__ parts, int nblk)
{
    __shared__ uint32_t carry;
    __shared__ uint32_t wsum[4];
    const int x = blockIdx.x;
    uint32_t *p = parts + (size_t)x * nblk;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nblk; base += 256) {
        const int k = base + threadIdx.x;
        const uint32_t v = k < nblk ? p[k] : 0u;
        // inclusive scan within the wave, then across the 4 waves
        uint32_t inc = v;
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t t = __shfl_up(inc, d, 64);
            if (lane >= d) inc += t;
        }
        if (lane == 63) wsum[w] = inc;
        __syncthreads();
        uint32_t before = carry;
        for (int q = 0; q < w; ++q) before += wsum[q];
        if (k < nblk) p[k] = before + inc - v;
        __syncthreads();
        if (threadIdx.x == 255) carry = before + inc;
        __syncthreads();
    }
    if (threadIdx.x == 0) parts[(size_t)8 * nblk + x] = carry;
}

template <bool CHUNKED>
__global__ __launch_bounds__(kOrdBlock) void k_order_write(const uint32_t *__restrict__ ranges,
                                                           int32_t ntiles,
                                                           const unsigned long long *__restrict__ total,
                                                           const uint32_t *__restrict__ parts,
                                                           uint32_t *__restrict__ order)
{
    __shared__ uint32_t wsum[kOrdBlock / 64];
    const int x = blockIdx.y, i = blockIdx.x * kOrdBlock + threadIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int tile;
    const bool h = heavy_tile<CHUNKED>(ranges, ntiles, *total, x, i, tile);
    const uint64_t bal = __ballot(h);
    if (lane == 0) wsum[w] = (uint32_t)__popcll(bal);
    __syncthreads();
    uint32_t before = parts[x * gridDim.x + blockIdx.x];
    for (int q = 0; q < w; ++q) before += wsum[q];
    before += (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));   // heavy tiles before i
    if (tile < 0) return;
    const uint32_t heavy_total = parts[(size_t)8 * gridDim.x + x];
    const uint32_t ni = h ? before : heavy_total + ((uint32_t)i - before);
    order[8 * (size_t)ni + x] = (uint32_t)tile;
}

hipError_t launch_tile_order(const uint32_t *ranges, int32_t ntiles,
                             const unsigned long long *total_pairs, bool chunked,
                             uint32_t *order, uint32_t *parts, hipStream_t st)
{
    if (ntiles <= 0) return hipSuccess;
    const int nblk = tile_order_blocks(ntiles);
    const dim3 grid((unsigned)nblk, 8);
    if (chunked)
        hipLaunchKernelGGL(k_order_count<true>, grid, dim3(kOrdBlock), 0, st, ranges, ntiles, total_pairs, parts);
    else
        hipLaunchKernelGGL(k_order_count<false>, grid, dim3(kOrdBlock), 0, st, ranges, ntiles, total_pairs, parts);
    hipLaunchKernelGGL(k_order_scan, dim3(8), dim3(256), 0, st, parts, nblk);
    if (chunked)
        hipLaunchKernelGGL(k_order_write<true>, grid, dim3(kOrdBlock), 0, st, ranges, ntiles, total_pairs,
                           parts, order);
    else
        hipLaunchKernelGGL(k_order_write<false>, grid, dim3(kOrdBlock), 0, st, ranges, ntiles, total_pairs,
                           parts, order);
    return hipGetLastError();
}

// ------------------------------------------------------------ per-pair evaluation
// The same FP32 sequence runs in the forward and the backward so both take the same
// discrete decisions (skip, stop, branch).
struct PairEval {
    float dx, dy, u0, u1, G, oG, alpha;
    bool ub;
};

__device__ __forceinline__ PairEval eval_pair(const float4 r0, const float4 r1, const float4 r2,
                                              const float4 r3, float fx, float fy,
                                              const RasterConsts rc)
{
    PairEval e;
    e.dx = __fsub_rn(__fsub_rn(fx, r0.z), r1.x);
    e.dy = __fsub_rn(__fsub_rn(fy, r0.w), r1.y);
    e.u0 = __fmaf_rn(r2.y, e.dy, __fmul_rn(r2.x, e.dx));
    e.u1 = __fmaf_rn(r2.w, e.dy, __fmul_rn(r2.z, e.dx));
    const float ru = __fmaf_rn(e.u0, e.u0, __fmaf_rn(e.u1, e.u1, r1.z));
    const float rf = __fmaf_rn(__fmaf_rn(e.dx, e.dx, __fmul_rn(e.dy, e.dy)), rc.inv_s2, r1.w);
    e.ub = ru <= rf;
    const float rho = e.ub ? ru : rf;
    e.G = ex2(__fmul_rn(rho, kNegHalfLog2e));
    e.oG = __fmul_rn(r3.x, e.G);
    // min(alpha_max, oG) for oG >= 0, in one median-of-three instruction
    e.alpha = __builtin_amdgcn_fmed3f(e.oG, 0.f, rc.alpha_max);
    return e;
}

// ------------------------------------------------------------- per-pixel coverage
// chunk_mask: lane t holds record c0 + t of a chunk of up to 64 (valid = t < count);
// returns, for the calling lane's pixel (wx0 + lane % 8, wy0 + lane / 8), the 64-bit
// mask of chunk records whose pixel box contains that pixel.  A box is separable into a
// column range and a row range, so 8 ballots over column bits and 8 over row bits give
// the whole 64 x 64 coverage matrix; lane p keeps column mask p % 8 AND row mask p / 8.
// Outside the box alpha < alpha_min holds exactly (the box bounds both rho branches at
// the alpha_min level), so skipping those pairs changes no result.
__device__ __forceinline__ uint64_t chunk_mask(float box_x, float box_y, bool valid, int wx0, int wy0,
                                               int lane)
{
    uint32_t colbits = 0, rowbits = 0;
    if (valid) {
        const uint32_t x = __float_as_uint(box_x), y = __float_as_uint(box_y);
        const int clo = max((int)(int16_t)(x & 0xFFFFu) - wx0, 0);
        const int chi = min((int)(int16_t)(x >> 16) - wx0, 7);
        const int rlo = max((int)(int16_t)(y & 0xFFFFu) - wy0, 0);
        const int rhi = min((int)(int16_t)(y >> 16) - wy0, 7);
        if (clo <= chi) colbits = (0xFFu >> (7 - chi)) & (0xFFu << clo);
        if (rlo <= rhi) rowbits = (0xFFu >> (7 - rhi)) & (0xFFu << rlo);
    }
    const int lc = lane & 7, lr = lane >> 3;
    uint64_t cm = 0, rm = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const uint64_t bc = __ballot((colbits >> c) & 1u);
        const uint64_t br = __ballot((rowbits >> c) & 1u);
        cm = lc == c ? bc : cm;
        rm = lr == c ? br : rm;
    }
    return cm & rm;
}

// ---------------------------------------------------------------- raster forward
// A pixel's running sums.
struct PixelSums {
    float Tr = 1.f, aD = 0.f, a0 = 0.f, a1 = 0.f, a2 = 0.f, aV = 0.f, n0 = 0.f, n1 = 0.f, n2 = 0.f;
    // distortion: accumulated value, reference depth, shifted first and second moments
    float dacc = 0.f, zref = 0.f, M1 = 0.f, M2 = 0.f;
    bool has_ref = false, done;
    int ncontrib = 0, neval = 0;
};

// A record in LDS, as structure of arrays: centre (high and low part), Q, (o, z0, k) as one
// float4 each, and for views albedo with visibility, and the normal.  The record's two branch
// biases are folded in: a record without an ellipse has Q = NaN, so that its low-pass branch
// is taken by comparison, and without the low-pass filter (FILT false) every other one takes
// the ellipse.  48 bytes for a depth-only pair and 76 for a view's instead of 56 and 84: the
// reads of 64 lanes, each at its own record, are what the walk waits for besides VALU issue
// (40 views of 2M surfels: 8.19 -> 7.85 ms, their sun maps 4.46 -> 4.35 ms).
constexpr int kFwdSlots = 64;

template <bool DEPTH_ONLY, bool FILT>
__device__ __forceinline__ void stage_record(float4 *lds, int slot, float4 r0, float4 r1, float4 r2,
                                             float4 r3, float4 r4, float4 r5)
{
    bool ell = !(r1.z > 0.f);
    // Q beyond FP32: Q delta is infinite or, at the centre, NaN, and with no low-pass branch to
    // take instead the pair has no weight at any pixel.  Staged without an ellipse and with no
    // opacity its depth stays finite as well.
    if (!FILT && !(isfinite(r2.x) && isfinite(r2.y) && isfinite(r2.z) && isfinite(r2.w))) {
        ell = false;
        r3.x = 0.f;
    }
    const float none = __uint_as_float(0x7FC00000u);
    lds[slot] = make_float4(r0.z, r0.w, r1.x, r1.y);
    lds[kFwdSlots + slot] = ell ? r2 : make_float4(none, none, none, none);
    lds[2 * kFwdSlots + slot] = r3;
    if (!DEPTH_ONLY) { lds[3 * kFwdSlots + slot] = r4; lds[4 * kFwdSlots + slot] = r5; }
}

// eval_pair's arithmetic on a staged record.
template <bool FILT>
__device__ __forceinline__ PairEval eval_staged(const float4 c, const float4 q, float o, bool ell, float fx,
                                                float fy, const RasterConsts &rc)
{
    PairEval e;
    e.dx = __fsub_rn(__fsub_rn(fx, c.x), c.z);
    e.dy = __fsub_rn(__fsub_rn(fy, c.y), c.w);
    e.u0 = __fmaf_rn(q.y, e.dy, __fmul_rn(q.x, e.dx));
    e.u1 = __fmaf_rn(q.w, e.dy, __fmul_rn(q.z, e.dx));
    const float ru = __fmaf_rn(e.u0, e.u0, __fmul_rn(e.u1, e.u1));
    const float rf = __fmul_rn(__fmaf_rn(e.dx, e.dx, __fmul_rn(e.dy, e.dy)), rc.inv_s2);
    e.ub = FILT ? ell && ru <= rf : ell;
    e.G = ex2(__fmul_rn(e.ub ? ru : rf, kNegHalfLog2e));
    e.oG = __fmul_rn(o, e.G);
    e.alpha = __builtin_amdgcn_fmed3f(e.oG, 0.f, rc.alpha_max);
    return e;
}

// Composites the staged records of mask m (bit j: slot j) onto this lane's pixel, front to
// back, until its transmittance would drop below T_min.  Returns the composited ones
// (counted in ncontrib instead when CM is false).
template <bool DEPTH_ONLY, bool HAS_VIS, bool DIST, bool FILT>
__device__ __forceinline__ unsigned long long composite(const float4 *lds, uint64_t m, float fx,
                                                        float fy, const RasterConsts &rc, float ds,
                                                        PixelSums &p)
{
    constexpr int BS = kFwdSlots;
    constexpr bool CM = !DEPTH_ONLY;
    unsigned long long cmc = 0ull;
    while (m != 0) {
        const int jc = (int)__builtin_ctzll(m);
        m &= m - 1;
        const float4 c = lds[jc], q = lds[BS + jc], r3 = lds[2 * BS + jc];
        ++p.neval;
        const PairEval e = eval_staged<FILT>(c, q, r3.x, FILT || q.x == q.x, fx, fy, rc);
        // branch-free: a skipped pair accumulates with weight 0 (w * x + a == a
        // exactly for the finite record fields), so no exec-mask juggling per pair
        const bool hit = e.alpha >= rc.alpha_min;
        const float Tn = __fmul_rn(p.Tr, __fsub_rn(1.f, e.alpha));
        const bool stop = hit && Tn < rc.T_min;
        const bool take = hit && !stop;
        const float w = take ? __fmul_rn(e.alpha, p.Tr) : 0.f;
        const float z = e.ub ? __fmaf_rn(-r3.z, e.u0, __fmaf_rn(-r3.w, e.u1, r3.y)) : r3.y;
        p.aD = __fmaf_rn(w, z, p.aD);
        if (!DEPTH_ONLY) {
            const float4 r4 = lds[3 * BS + jc], r5 = lds[4 * BS + jc];
            p.a0 = __fmaf_rn(w, r4.x, p.a0);
            p.a1 = __fmaf_rn(w, r4.y, p.a1);
            p.a2 = __fmaf_rn(w, r4.z, p.a2);
            if (HAS_VIS) p.aV = __fmaf_rn(w, r4.w, p.aV);
            p.n0 = __fmaf_rn(w, r5.x, p.n0);
            p.n1 = __fmaf_rn(w, r5.y, p.n1);
            p.n2 = __fmaf_rn(w, r5.z, p.n2);
        }
        if (DIST) {
            // sum_{j<i} w_j (m_i - m_j)^2 = m'(m' (1 - T) - 2 M1) + M2 with m' the
            // depth relative to the first contributor
            p.zref = (take && !p.has_ref) ? z : p.zref;
            p.has_ref = p.has_ref || take;
            const float mp = (z - p.zref) * ds;
            p.dacc = fmaf(w, fmaf(mp, fmaf(mp, 1.f - p.Tr, -2.f * p.M1), p.M2), p.dacc);
            p.M1 = fmaf(w, mp, p.M1);
            p.M2 = fmaf(w * mp, mp, p.M2);
        }
        if (CM) cmc |= take ? 1ull << jc : 0ull;
        p.Tr = take ? Tn : p.Tr;
        if (!CM) p.ncontrib += take ? 1 : 0;   // else it follows from cmc once per chunk
        p.done = p.done || stop;
        m = stop ? 0ull : m;
    }
    return cmc;
}

// LDS written by other lanes of the wave is read after this, and the other way round.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wave per 8x8 pixel block of a tile (SHARE: four of them a block).  Records are staged in LDS, up to 64 at a time;
// each lane builds the mask of those that cover its pixel and composites them front to
// back until its transmittance would drop below T_min; a wave whose 64 pixels all stopped
// is done.
// 8x8 tiles stage their list as it is, in batches of rc.batch, the next batch prefetched
// into registers.  The blocks of a larger tile share its list but each is covered by a part
// of it (about a third at 16x16), so a block first tests the records' boxes, 64 positions at a
// time, and stages the ones that meet it densely: the walk takes the longest pixel of every
// staged batch, and that is shorter for 64 records at once than for three times 20.  16x16
// tiles against one block of four waves that shared the staged list: 20 sun maps of 1M
// surfels 2175 -> 1578 us, three ~530^2 views of 150k surfels 141 -> 129 us.
// SHARE: the blocks of a tile drift apart, and each then reads the tile's boxes from beyond L2 on its
// own (5M surfels in 1024^2 maps: 67 GB a launch against the 18 of a shared read).  Four waves
// of one block, for 16x16 pixels, read a quarter of the boxes each, test them for all four, and
// meet at a barrier every 256 records: slower while lists are short, for a block then holds its
// place until its longest wave ends, faster where they are long (9.9 -> 8.0 ms there).
// The loop over a lane's own mask diverges on purpose: a uniform loop (idle lanes on a zeroed
// slot, work counters in scalar registers) issues 8 % fewer VALU instructions and runs 3-8 %
// longer, since idle lanes then read LDS too.
template <int TS, bool DEPTH_ONLY, bool HAS_VIS, bool DIST, bool FILT, bool SHARE>
__global__ __launch_bounds__(SHARE ? 256 : 64) void k_raster_fwd(
    int32_t nv, const ViewDesc *__restrict__ views, int32_t ntiles, const uint32_t *__restrict__ ranges,
    const uint32_t *__restrict__ lists, const float4 *__restrict__ rec, int64_t n,
    RasterConsts rc, const float *__restrict__ colC, const float *__restrict__ colc,
    const float *__restrict__ amb, const SunCam *__restrict__ sun, float *__restrict__ image,
    float *__restrict__ Aout, float *__restrict__ Vout, float *__restrict__ Dout,
    float *__restrict__ Nout, float *__restrict__ Tout, int32_t *__restrict__ lastout,
    unsigned long long *__restrict__ stats, unsigned long long *__restrict__ cmask,
    DistArgs da)
{
    constexpr int WPR = TS / 8, SUB = WPR * WPR, NT = TS * TS;
    constexpr bool DENSE = TS > 8;
    // view passes record, per pixel and 64-position word of the tile list, which records it
    // composited (the backward walks only those)
    constexpr bool CM = !DEPTH_ONLY;
    constexpr int RS = DEPTH_ONLY ? kSunRecStride4 : kRecStride4;   // record slot
    constexpr int NW = SHARE ? 4 : 1, REG = SUB / NW;           // waves a block, blocks a tile
    constexpr int SLOTS = kFwdSlots * (DEPTH_ONLY ? 3 : 5);
    __shared__ float4 lds_all[NW * SLOTS];
    const int wv = SHARE ? (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    float4 *const lds = lds_all + wv * SLOTS;
    // blocks go round-robin to the 8 XCDs: the blocks of a tile stay on the tile's XCD
    const int b = (int)blockIdx.x;
    const int vb = REG == 1 ? b : 8 * (b / (8 * REG)) + b % 8;
    const int reg = REG == 1 ? 0 : (b / 8) % REG;
    const int sub = SHARE ? (2 * (reg >> 1) + (wv >> 1)) * WPR + 2 * (reg & 1) + (wv & 1) : reg;
    if (vb >= ntiles) return;
    // sun maps are equal in size and even in work: one contiguous run of tiles per XCD
    const int tile = rc.torder ? (int)rc.torder[vb] : xcd_tile<!DEPTH_ONLY>(vb, ntiles);
    const int v = find_view(views, nv, tile);
    const ViewDesc vd = views[v];
    const int lt = tile - vd.tile_off;
    const int tx = lt % vd.tiles_x, ty = lt / vd.tiles_x;
    const int lane = SHARE ? threadIdx.x & 63 : threadIdx.x;
    const int wx0 = tx * TS + (sub % WPR) * 8, wy0 = ty * TS + (sub / WPR) * 8;
    const int px = wx0 + (lane & 7), py = wy0 + (lane >> 3);
    const bool inside = px < vd.W && py < vd.H;
    const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
    const uint2 range = tile_range(ranges, tile);
    const uint32_t start = range.x, end = range.y;
    const float4 *recv = rec + (size_t)v * (size_t)n * RS;
    PixelSums p;
    p.done = !inside;
    int lastpos = 0;
    float4 q0, q1, q2, q3, q4, q5;               // records on their way to LDS
    const size_t wbase = (size_t)(start >> 6) + (size_t)tile;   // tiles' word ranges are disjoint
    unsigned long long *const word_at = CM && cmask ? cmask + wbase * NT + sub * 64 + lane : nullptr;
    unsigned long long wacc = 0ull;
    if constexpr (!DENSE) {
        int wcur = -1;
        const int B = min(rc.batch, 64);
        uint32_t nidx = 0;                        // list entries of the batch after the prefetched one
#define SS_FETCH_FWD(IDX)                                                              \
    {                                                                                  \
        const float4 *src_ = recv + (size_t)min((IDX), (uint32_t)(n - 1)) * RS;       \
        q0 = src_[0]; q1 = src_[1]; q2 = src_[2]; q3 = src_[3];                        \
        if (!DEPTH_ONLY) { q4 = src_[4]; q5 = src_[5]; }                               \
    }
        if (start < end && lane < (int)min((uint32_t)B, end - start)) SS_FETCH_FWD(lists[start + lane]);
        if (start + B < end && lane < (int)min((uint32_t)B, end - start - B)) nidx = lists[start + B + lane];
        for (uint32_t b0 = start; b0 < end; b0 += B) {
            const int nb = (int)min((uint32_t)B, end - b0);
            __syncthreads();
            if (lane < nb) stage_record<DEPTH_ONLY, FILT>(lds, lane, q0, q1, q2, q3, q4, q5);
            const float box_x = q0.x, box_y = q0.y;
            __syncthreads();
            const uint32_t b1 = b0 + B, b2 = b1 + B;
            if (b1 < end && lane < (int)min((uint32_t)B, end - b1)) SS_FETCH_FWD(nidx);
            if (b2 < end && lane < (int)min((uint32_t)B, end - b2)) nidx = lists[b2 + lane];
            if (__ballot(!p.done) == 0) break;
            uint64_t m = chunk_mask(box_x, box_y, lane < nb, wx0, wy0, lane);
            if (p.done) m = 0;
            const unsigned long long cmc = composite<DEPTH_ONLY, HAS_VIS, DIST, FILT>(lds, m, fx, fy, rc, da.ds, p);
            const int P0 = (int)(b0 - start);
            if (CM && cmc != 0ull) {
                lastpos = P0 + 64 - (int)__builtin_clzll(cmc);
                p.ncontrib += (int)__popcll(cmc);
            }
            if (CM && cmask) {
                // positions [P0, P0 + nb) fall in word P0 / 64 and, when the batch depth does
                // not divide 64, also in the next word
                const int w = P0 >> 6, sh = P0 & 63;
                if (w != wcur) {
                    if (wcur >= 0) word_at[(size_t)wcur * NT] = wacc;
                    wacc = 0ull;
                    wcur = w;
                }
                wacc |= cmc << sh;
                if (sh + nb > 64) {
                    word_at[(size_t)wcur * NT] = wacc;
                    wacc = cmc >> (64 - sh);
                    wcur = w + 1;
                }
            }
        }
        if (CM && cmask && wcur >= 0) word_at[(size_t)wcur * NT] = wacc;
    } else {
        // staged positions of up to 64 consecutive words of the list, one mask each
        __shared__ unsigned long long segs_all[CM ? NW * 64 : 1];
        __shared__ float2 boxes_all[NW * 64];
        unsigned long long *const segs = segs_all + (CM ? wv * 64 : 0);
        float2 *const boxes = boxes_all + wv * 64;
        // SHARE: four words of the list at a time, one read by each wave: their entries, which
        // records meet which wave's block, which waves are done; two buffers, one barrier
        __shared__ uint32_t entries[2][NW * 64];
        __shared__ unsigned long long meet[2][NW][4];
        __shared__ int over[2][4];
        const int nw = (int)((end - start + 63) >> 6);
        const int rx0 = wx0 - 8 * (wv & 1), ry0 = wy0 - 8 * (wv >> 1);   // the waves' 16x16 pixels
        auto entry = [&](int w) {                 // the lane's list entry in word w (0 past the end)
            const uint32_t k = start + 64u * (uint32_t)w + (uint32_t)lane;
            return k < end ? lists[k] : 0u;
        };
        auto slot = [&](uint32_t idx) { return recv + (size_t)min(idx, (uint32_t)(n - 1)) * RS; };
        // heads of the wave's next word, list entries of the one after it
        uint32_t idx_h = wv < nw ? entry(wv) : 0u, idx_n = wv + NW < nw ? entry(wv + NW) : 0u;
        float4 head = make_float4(0.f, 0.f, 0.f, 0.f);
        auto head_of = [&](uint32_t idx) {
            if constexpr (SHARE) {
                const float2 b = *reinterpret_cast<const float2 *>(slot(idx));
                return make_float4(b.x, b.y, 0.f, 0.f);
            } else
                return slot(idx)[0];
        };
        if (wv < nw) head = head_of(idx_h);
        // Every wave of the block calls this for words NW * g .. NW * g + NW - 1, g = 0, 1, ..., also
        // when its own pixels have stopped, until the list ends or all waves say that they have.
        [[maybe_unused]] auto group = [&](int g, bool stopped) {
            const int bf = g & 1, w = NW * g + wv;
            const int x = __float_as_int(head.x), y = __float_as_int(head.y);
            const int x0 = (x << 16) >> 16, x1 = x >> 16, y0 = (y << 16) >> 16, y1 = y >> 16;
            const bool in = w < nw && start + 64u * (uint32_t)w + (uint32_t)lane < end;
            const bool cl = in && x0 <= rx0 + 7 && x1 >= rx0, cr = in && x0 <= rx0 + 15 && x1 >= rx0 + 8;
            const bool rl = y0 <= ry0 + 7 && y1 >= ry0, rr = y0 <= ry0 + 15 && y1 >= ry0 + 8;
            const uint64_t m0 = __ballot(cl && rl), m1 = __ballot(cr && rl);
            const uint64_t m2 = __ballot(cl && rr), m3 = __ballot(cr && rr);
            entries[bf][wv * 64 + lane] = idx_h;
            if (lane == 0) {
                unsigned long long *const mw = meet[bf][wv];
                mw[0] = m0; mw[1] = m1; mw[2] = m2; mw[3] = m3;
                over[bf][wv] = stopped;
            }
            idx_h = idx_n;
            if (w + NW < nw) head = head_of(idx_h);
            if (w + 2 * NW < nw) idx_n = entry(w + 2 * NW);
            __syncthreads();
            return (over[bf][0] & over[bf][1] & over[bf][2] & over[bf][3]) != 0;
        };
        int wq = -1, staged = 0, nseg = 0, w0 = 0;
        uint64_t U = 0;                           // records of word wq still to stage (uniform)
        for (;;) {
            if (U == 0 && ++wq < nw) {
                if constexpr (SHARE) {
                    if (wq % NW == 0) group(wq / NW, false);
                    const int bf = (wq / NW) & 1;
                    const unsigned long long mm = meet[bf][wq % NW][wv];
                    U = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(mm >> 32)) << 32) |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)mm);
                    if ((U >> lane) & 1ull) {
                        const float4 *src = slot(entries[bf][(wq % NW) * 64 + lane]);
                        q0 = src[0]; q1 = src[1]; q2 = src[2]; q3 = src[3];
                        if (!DEPTH_ONLY) { q4 = src[4]; q5 = src[5]; }
                    }
                } else {
                    const int x = __float_as_int(head.x), y = __float_as_int(head.y);
                    const bool meets = ((x << 16) >> 16) <= wx0 + 7 && (x >> 16) >= wx0 &&
                                       ((y << 16) >> 16) <= wy0 + 7 && (y >> 16) >= wy0 &&
                                       start + 64u * (uint32_t)wq + (uint32_t)lane < end;
                    U = __ballot(meets);
                    if (meets) {
                        const float4 *src = slot(idx_h);
                        q0 = head; q1 = src[1]; q2 = src[2]; q3 = src[3];
                        if (!DEPTH_ONLY) { q4 = src[4]; q5 = src[5]; }
                    }
                    idx_h = idx_n;
                    if (wq + 1 < nw) head = head_of(idx_h);
                    if (wq + 2 < nw) idx_n = entry(wq + 2);
                }
                if (U == 0) {
                    if (!CM) continue;
                    if (lane == 0) segs[nseg] = 0ull;
                    if (++nseg < 64) continue;
                }
            }
            if (U != 0) {
                const int k = staged + __popcll(U & ((1ull << lane) - 1ull));
                const bool sel = ((U >> lane) & 1ull) && k < 64;
                const uint64_t take = __ballot(sel);
                U &= ~take;
                if (sel) {
                    stage_record<DEPTH_ONLY, FILT>(lds, k, q0, q1, q2, q3, q4, q5);
                    boxes[k] = make_float2(q0.x, q0.y);
                }
                staged += (int)__popcll(take);
                if (CM) {
                    if (lane == 0) segs[nseg] = take;
                    ++nseg;
                }
                if (staged < 64 && (!CM || nseg < 64)) continue;
            }
            wave_sync();
            unsigned long long cmc = 0ull;
            if (staged > 0) {
                const float2 box = boxes[lane < staged ? lane : 0];
                uint64_t m = chunk_mask(box.x, box.y, lane < staged, wx0, wy0, lane);
                if (p.done) m = 0;
                cmc = composite<DEPTH_ONLY, HAS_VIS, DIST, FILT>(lds, m, fx, fy, rc, da.ds, p);
            }
            const bool all_done = __ballot(!p.done) == 0;
            if (CM) {
                // slots back to the positions that they came from, word by word
                p.ncontrib += (int)__popcll(cmc);
                int s = 0;
                for (int k = 0; k < nseg; ++k) {
                    const unsigned long long sg = segs[k];
                    uint64_t mask = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(sg >> 32)) << 32) |
                                    (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)sg);
                    while (mask != 0) {
                        const int j = (int)__builtin_ctzll(mask);
                        mask &= mask - 1;
                        wacc |= ((cmc >> s) & 1ull) << j;
                        ++s;
                    }
                    if (k < nseg - 1 || U == 0 || all_done) {
                        if (wacc != 0ull) lastpos = 64 * (w0 + k) + 64 - (int)__builtin_clzll(wacc);
                        if (cmask) word_at[(size_t)(w0 + k) * NT] = wacc;
                        wacc = 0ull;
                    }
                }
                w0 += U != 0 ? nseg - 1 : nseg;   // a word cut short goes on in the next batch
                nseg = 0;
            }
            wave_sync();
            staged = 0;
            if (wq >= nw || all_done) break;
        }
        if constexpr (SHARE)
            for (int g = wq / NW + 1; NW * g < nw; ++g)
                if (group(g, true)) break;
    }
#undef SS_FETCH_FWD
    {
        // work counters: one 64-bit atomic per wave and counter, into the tile's slot
        unsigned long long c = (unsigned long long)p.ncontrib, e = (unsigned long long)p.neval;
        for (int d = 32; d > 0; d >>= 1) {
            c += __shfl_xor(c, d, 64);
            e += __shfl_xor(e, d, 64);
        }
        if (lane == 0) {
            unsigned long long *slot = stats + (size_t)(tile % kStatSlots) * kStatStride;
            atomicAdd(slot, c);
            atomicAdd(slot + 1, e);
        }
    }
    if (!inside) return;
    const int64_t P = (int64_t)vd.W * vd.H;
    const int64_t local = (int64_t)py * vd.W + px;
    const int64_t g = vd.pix_off + local;
    if (DEPTH_ONLY) {
        Dout[g] = (float)((double)p.aD + (double)p.Tr * sun[v].zfar);
        return;
    }
    float C[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1}, cb[3] = {0, 0, 0}, La[3] = {0, 0, 0};
    if (colC) for (int k = 0; k < 9; ++k) C[k] = colC[9 * v + k];
    if (colc) for (int k = 0; k < 3; ++k) cb[k] = colc[3 * v + k];
    if (amb) for (int k = 0; k < 3; ++k) La[k] = amb[3 * v + k];
    const float Vp = HAS_VIS ? p.aV : 1.f;
    const float A[3] = {p.a0, p.a1, p.a2};
    const int64_t b3 = 3 * vd.pix_off + local;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float ca = C[3 * ch] * A[0] + C[3 * ch + 1] * A[1] + C[3 * ch + 2] * A[2] + cb[ch];
        image[b3 + ch * P] = ca * (Vp + (1.f - Vp) * La[ch]);
        Aout[b3 + ch * P] = A[ch];
    }
    Nout[b3] = p.n0; Nout[b3 + P] = p.n1; Nout[b3 + 2 * P] = p.n2;
    Vout[g] = Vp;
    Dout[g] = p.aD;
    Tout[g] = p.Tr;
    lastout[g] = lastpos;
    if (DIST) {
        da.dist[g] = p.dacc;
        da.aux[g] = p.zref;
        da.aux[da.P + g] = p.M1;
        da.aux[2 * da.P + g] = p.M2;
    }
}

// 8x8 blocks of a tile, and the grid of a kernel that runs one wave for each of them.
constexpr int ts_sub(int ts) { return (ts / 8) * (ts / 8); }
static int64_t raster_blocks(int sub, int32_t ntiles)
{
    return sub == 1 ? ntiles : ((int64_t)ntiles + 7) / 8 * 8 * sub;
}

// Depth-only maps of larger tiles with at least this many surfels per tile take the blocks whose
// waves read the list together (SHARE).  Whole passes of 20 sun maps, one wave a block -> shared,
// by surfels per tile, in us:
//   512^2 maps, 16x16 tiles   293: 1083 -> 1202   488: 1600 -> 1738   684: 2253 -> 2255
//                             879: 2923 -> 2765  1172: 3927 -> 3614
//   512^2 maps, 32x32 tiles   234:  480 ->  532  1172: 1355 -> 1304  4688: 7527 -> 4141
//   1024^2 maps, 32x32 tiles  293: 1637 -> 1840   977: 4140 -> 3893
// The kernel alone at 1024^2 and 16x16: 244: 1580 -> 2012 us, 1221: 9.9 -> 8.0 ms.
constexpr int64_t kShareSurfels = 768;

template <int TS, bool DO, bool HV>
static void launch_fwd_t(int32_t ntiles, hipStream_t st, int32_t nv,
                         const ViewDesc *views, const uint32_t *ranges, const uint32_t *lists,
                         const float *rec, int64_t n, const RasterConsts &rc,
                         const float *colC, const float *colc, const float *amb,
                         const SunCam *sun, float *image, float *A, float *V, float *D,
                         float *N, float *T, int32_t *last, unsigned long long *stats,
                         unsigned long long *cmask, const DistArgs *dist)
{
    const DistArgs da = dist ? *dist : DistArgs{0.f, nullptr, nullptr, nullptr, 0};
    const bool share = DO && TS > 8 && n * nv >= kShareSurfels * ntiles;
    const dim3 grid((unsigned)raster_blocks(ts_sub(TS) / (share ? 4 : 1), ntiles)), block(share ? 256 : 64);
#define SS_FWD_LAUNCH(DIST_, FILT_, SHARE_)                                                            \
    hipLaunchKernelGGL((k_raster_fwd<TS, DO, HV, DIST_, FILT_, SHARE_>), grid, block, 0, st, nv, views, \
                       ntiles, ranges, lists, reinterpret_cast<const float4 *>(rec), n, rc, colC, colc, \
                       amb, sun, image, A, V, D, N, T, last, stats, cmask, da)
    if (share) {
        if (rc.lowpass_mode == 0) SS_FWD_LAUNCH(false, true, (DO && TS > 8));
        else SS_FWD_LAUNCH(false, false, (DO && TS > 8));
    } else if (!DO && dist) {
        if (rc.lowpass_mode == 0) SS_FWD_LAUNCH(!DO, true, false);
        else SS_FWD_LAUNCH(!DO, false, false);
    } else {
        if (rc.lowpass_mode == 0) SS_FWD_LAUNCH(false, true, false);
        else SS_FWD_LAUNCH(false, false, false);
    }
#undef SS_FWD_LAUNCH
}

size_t cmask_words(int64_t pair_cap, int32_t tiles, int ts)
{
    return ((size_t)(pair_cap > 0 ? pair_cap : 0) / 64 + (size_t)(tiles > 0 ? tiles : 0) + 1) * ts * ts;
}

hipError_t launch_raster_fwd(int ts, bool depth_only, bool has_vis, int32_t total_tiles,
                             int32_t nv, const ViewDesc *views, const uint32_t *ranges,
                             const uint32_t *lists, const float *rec, int64_t n,
                             const RasterConsts &rc, const float *colC, const float *colc,
                             const float *amb, const SunCam *sun, float *image, float *A,
                             float *V, float *D, float *N, float *T, int32_t *last,
                             unsigned long long *stats, unsigned long long *cmask, hipStream_t st,
                             const DistArgs *dist)
{
    if (total_tiles <= 0) return hipSuccess;
#define SS_FWD(TS_)                                                                              \
    if (ts == TS_) {                                                                             \
        if (depth_only)                                                                          \
            launch_fwd_t<TS_, true, false>(total_tiles, st, nv, views, ranges, lists, rec, n, rc,   \
                                           colC, colc, amb, sun, image, A, V, D, N, T, last, stats, cmask, dist);\
        else if (has_vis)                                                                        \
            launch_fwd_t<TS_, false, true>(total_tiles, st, nv, views, ranges, lists, rec, n, rc,   \
                                           colC, colc, amb, sun, image, A, V, D, N, T, last, stats, cmask, dist);\
        else                                                                                     \
            launch_fwd_t<TS_, false, false>(total_tiles, st, nv, views, ranges, lists, rec, n, rc,  \
                                            colC, colc, amb, sun, image, A, V, D, N, T, last, stats, cmask, dist);\
    }
    SS_FWD(8) else SS_FWD(16) else SS_FWD(32) else return hipErrorInvalidValue;
#undef SS_FWD
    return hipGetLastError();
}

// ------------------------------------------------------- wave transpose reduction
// 16 per-lane values -> lane l holds the wave sum of value (l >> 2) & 15 (lanes with
// l % 4 == 0 then hold all 16 sums).  Each level halves the vector a lane carries: the
// two cross-row levels use gfx950's lane swaps (permlane32 / permlane16: one VALU op
// exchanges half of two registers between the partner rows, then one add), the two
// in-row levels use DPP row mirrors, the last two are full DPP quad sums.  No LDS.
template <int CTRL>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_amdgcn_update_dpp(0.f, v, CTRL, 0xF, 0xF, true);
}

__device__ __forceinline__ void swap_rows32(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

__device__ __forceinline__ void swap_rows16(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

__device__ __forceinline__ float wave_transpose_reduce16(float (&x)[16], int lane)
{
    float y8[8], y4[4], y2[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) {           // lanes 0-31 keep value k, 32-63 value k + 8
        float a = x[k], b = x[k + 8];
        swap_rows32(a, b);
        y8[k] = a + b;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {           // even rows keep k, odd rows k + 4
        float a = y8[k], b = y8[k + 4];
        swap_rows16(a, b);
        y4[k] = a + b;
    }
    const bool b3 = lane & 8, b2 = lane & 4;
#pragma unroll
    for (int k = 0; k < 2; ++k) {           // row mirror: partner 15 - i differs in bit 3
        const float keep = b3 ? y4[k + 2] : y4[k];
        const float send = b3 ? y4[k] : y4[k + 2];
        y2[k] = keep + dpp<0x140>(send);
    }
    // half-row mirror: partner 7 - i differs in bit 2
    float y = (b2 ? y2[1] : y2[0]) + dpp<0x141>(b2 ? y2[0] : y2[1]);
    y += dpp<0x4E>(y);                      // quad_perm [2,3,0,1]
    y += dpp<0xB1>(y);                      // quad_perm [1,0,3,2]
    return y;
}

// Within one 16-lane row: 16 per-lane values -> lane i holds the row sum of value i.
// Four levels, each pairing lanes that differ in one index bit (row mirror: bit 3,
// half-row mirror: bit 2, quad permutes: bits 1 and 0); every level keeps the half of
// the vector selected by that bit and adds the partner's copy of it.  The two halves of
// the first two levels are whole 4-lane DPP banks (bank b = lanes 4b..4b+3 of a row), so
// each kept value is one DPP add per half written under a bank mask; the compiler does
// not see into the asm, so each block waits out the VALU-write -> DPP-read hazard itself.
__device__ __forceinline__ float row_transpose_reduce16(const float (&x)[16], int lane)
{
    const bool b1 = lane & 2, b0 = lane & 1;
    float y8[8], y4[4], y2[2];
    // lanes 0-7 (banks 0, 1) keep values 0-7, lanes 8-15 (banks 2, 3) values 8-15; y8[k]
    // starts as x[k + 8] and is overwritten in place (an instruction reads its sources
    // before it writes)
#pragma unroll
    for (int k = 0; k < 8; ++k) y8[k] = x[k + 8];
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %0, %8, %8 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %1, %1 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %9, %9 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %2, %2 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %10, %10 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %3, %3, %3 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %11, %11 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %4, %4, %4 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %4, %12, %12 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %5, %5, %5 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %5, %13, %13 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %6, %6, %6 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %6, %14, %14 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %7, %7, %7 row_mirror row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %7, %15, %15 row_mirror row_mask:0xf bank_mask:0x3\n\t"
        : "+v"(y8[0]), "+v"(y8[1]), "+v"(y8[2]), "+v"(y8[3]), "+v"(y8[4]), "+v"(y8[5]),
          "+v"(y8[6]), "+v"(y8[7])
        : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]));
    // lanes with bit 2 clear (banks 0, 2) keep values 0-3, the others 4-7
#pragma unroll
    for (int k = 0; k < 4; ++k) y4[k] = y8[k + 4];
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %0, %4, %4 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %1, %5, %5 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %2, %6, %6 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "v_add_f32_dpp %3, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
        "v_add_f32_dpp %3, %7, %7 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        "s_nop 1"
        : "+v"(y4[0]), "+v"(y4[1]), "+v"(y4[2]), "+v"(y4[3])
        : "v"(y8[0]), "v"(y8[1]), "v"(y8[2]), "v"(y8[3]));
#pragma unroll
    for (int k = 0; k < 2; ++k)
        y2[k] = (b1 ? y4[k + 2] : y4[k]) + dpp<0x4E>(b1 ? y4[k] : y4[k + 2]);
    return (b0 ? y2[1] : y2[0]) + dpp<0xB1>(b0 ? y2[0] : y2[1]);
}

template <int CTRL>
__device__ __forceinline__ int dpp_i(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}

// OR of a 64-bit mask over the 16 lanes of a row (same four partner patterns).
__device__ __forceinline__ uint64_t row_or64(uint64_t v)
{
    int lo = (int)(uint32_t)v, hi = (int)(uint32_t)(v >> 32);
    lo |= dpp_i<0x140>(lo); hi |= dpp_i<0x140>(hi);
    lo |= dpp_i<0x141>(lo); hi |= dpp_i<0x141>(hi);
    lo |= dpp_i<0x4E>(lo); hi |= dpp_i<0x4E>(hi);
    lo |= dpp_i<0xB1>(lo); hi |= dpp_i<0xB1>(hi);
    return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

// Maximum over the 16 lanes of a row (same four partner patterns).
__device__ __forceinline__ int row_max(int v)
{
    v = max(v, dpp_i<0x140>(v));
    v = max(v, dpp_i<0x141>(v));
    v = max(v, dpp_i<0x4E>(v));
    v = max(v, dpp_i<0xB1>(v));
    return v;
}

// Per-pixel adjoints of Eq. image_formation: the upstream colour gradient through the
// colour transform and shading gives the gradients of the composited albedo (gA), of
// the composited visibility (gV), and the pixel's 15 per-view colour-parameter terms
// (cg[0..8] = dC, cg[9..11] = dc, cg[12..14] = dL_a, cg[15] = 0).
struct PixelAdjoint {
    float gA0, gA1, gA2, gV, gD, gN0, gN1, gN2, Tr;
    int last;
};

// Distortion state of a pixel in the backward: upstream gradient, reference depth, total
// weight 1 - T_final, shifted moments sum w m', sum w m'^2 over all its contributors.
struct DistPixel {
    float gDist, zref, At, M1, M2;
};

template <bool HAS_VIS>
__device__ __forceinline__ PixelAdjoint pixel_adjoint(
    bool inside, int v, int64_t g, int64_t b3, int64_t P, const float *__restrict__ colC,
    const float *__restrict__ colc, const float *__restrict__ amb, const float *__restrict__ Ain,
    const float *__restrict__ Vin, const float *__restrict__ Tin,
    const int32_t *__restrict__ lastin, const float *__restrict__ dI,
    const float *__restrict__ dD, const float *__restrict__ dN, float (&cg)[16])
{
    PixelAdjoint a{0, 0, 0, 0, 0, 0, 0, 0, 1.f, 0};
#pragma unroll
    for (int k = 0; k < 16; ++k) cg[k] = 0.f;
    if (!inside) return a;
    float C[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1}, cb[3] = {0, 0, 0}, La[3] = {0, 0, 0};
    if (colC) for (int k = 0; k < 9; ++k) C[k] = colC[9 * v + k];
    if (colc) for (int k = 0; k < 3; ++k) cb[k] = colc[3 * v + k];
    if (amb) for (int k = 0; k < 3; ++k) La[k] = amb[3 * v + k];
    const float A[3] = {Ain[b3], Ain[b3 + P], Ain[b3 + 2 * P]};
    const float Vp = HAS_VIS ? Vin[g] : 1.f;
    float gI[3] = {0, 0, 0};
    if (dI) { gI[0] = dI[b3]; gI[1] = dI[b3 + P]; gI[2] = dI[b3 + 2 * P]; }
    float gs[3];
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const float ca = C[3 * ch] * A[0] + C[3 * ch + 1] * A[1] + C[3 * ch + 2] * A[2] + cb[ch];
        const float shade = HAS_VIS ? Vp + (1.f - Vp) * La[ch] : 1.f;
        gs[ch] = gI[ch] * shade;
        if (HAS_VIS) {
            a.gV += gI[ch] * ca * (1.f - La[ch]);
            cg[12 + ch] = gI[ch] * ca * (1.f - Vp);
        }
        cg[9 + ch] = gs[ch];
#pragma unroll
        for (int q = 0; q < 3; ++q) cg[3 * ch + q] = gs[ch] * A[q];
    }
    a.gA0 = C[0] * gs[0] + C[3] * gs[1] + C[6] * gs[2];
    a.gA1 = C[1] * gs[0] + C[4] * gs[1] + C[7] * gs[2];
    a.gA2 = C[2] * gs[0] + C[5] * gs[1] + C[8] * gs[2];
    if (dD) a.gD = dD[g];
    if (dN) { a.gN0 = dN[b3]; a.gN1 = dN[b3 + P]; a.gN2 = dN[b3 + 2 * P]; }
    a.Tr = Tin[g];
    a.last = lastin[g];
    return a;
}

__device__ __forceinline__ DistPixel pixel_distortion_state(bool inside, int64_t g, float Tr,
                                                            const DistArgs &da)
{
    DistPixel d{0, 0, 0, 0, 0};
    if (!inside) return d;
    d.gDist = da.d_dist ? da.d_dist[g] : 0.f;
    d.zref = da.aux[g];
    d.M1 = da.aux[da.P + g];
    d.M2 = da.aux[2 * da.P + g];
    d.At = 1.f - Tr;
    return d;
}

// Per-pair terms of the walk: 1 / (1 - alpha), the pair's depth z (the centre depth on
// the low-pass branch), g . f (the upstream gradient dotted with the pair's composited
// features, plus the distortion's d dist / d w term) and the depth gradient per unit
// weight; u zeroed on the low-pass branch.
struct PairTerms {
    float rom, z, gf, gDe, u0, u1;
};

template <bool DIST>
__device__ __forceinline__ PairTerms pair_terms(const PairEval &e, float4 r3, float4 r4, float4 r5,
                                                const PixelAdjoint &pa, const DistPixel &dp,
                                                bool has_vis, float ds)
{
    PairTerms t;
    t.rom = __builtin_amdgcn_rcpf(1.f - e.alpha);
    t.u0 = e.ub ? e.u0 : 0.f;
    t.u1 = e.ub ? e.u1 : 0.f;
    t.z = __fmaf_rn(-r3.z, t.u0, __fmaf_rn(-r3.w, t.u1, r3.y));
    float gf = fmaf(pa.gA0, r4.x, fmaf(pa.gA1, r4.y, fmaf(pa.gA2, r4.z, fmaf(pa.gD, t.z,
               fmaf(pa.gN0, r5.x, fmaf(pa.gN1, r5.y, pa.gN2 * r5.z))))));
    if (has_vis) gf = fmaf(pa.gV, r4.w, gf);
    float gDe = pa.gD;
    if (DIST) {
        // d dist / d w_k = sum_j w_j (m'_k - m'_j)^2, d dist / d m_k = 2 w_k sum_j w_j (m'_k - m'_j)
        const float mp = (t.z - dp.zref) * ds;
        gf = fmaf(dp.gDist, fmaf(mp, fmaf(mp, dp.At, -2.f * dp.M1), dp.M2), gf);
        gDe = fmaf(2.f * dp.gDist * ds, fmaf(mp, dp.At, -dp.M1), pa.gD);
    }
    t.gf = gf;
    t.gDe = gDe;
    return t;
}

// The 16 record-gradient values of one pair from its weight w, dL/dalpha and dL/dz.
// The pair's branch enters once, through u (zero on the low-pass branch): the k, Q and
// u-centre terms vanish by multiplication, and the low-pass term of the centre gradient
// is zeroed on the u branch.  With rho2 = -oG dal (unclamped),
//   dL/dc = -(Q^T dL/du + delta rho2 / sigma^2 [low-pass branch]).
__device__ __forceinline__ void pair_record_grads(const PairEval &e, float w, float dal, float dz,
                                                  float u0, float u1, float4 r2, float4 r3,
                                                  const PixelAdjoint &pa, float inv_s2,
                                                  float alpha_max, float (&gr)[16])
{
    const float dzu = e.ub ? dz : 0.f;
    gr[G_AR] = w * pa.gA0; gr[G_AG] = w * pa.gA1; gr[G_AB] = w * pa.gA2;
    gr[G_NX] = w * pa.gN0; gr[G_NY] = w * pa.gN1; gr[G_NZ] = w * pa.gN2;
    gr[G_Z0] = dz;
    const float gd = e.oG < alpha_max ? dal : 0.f;       // zero where alpha is clamped
    gr[G_O] = e.G * gd;
    const float rho2 = -(e.oG * gd);
    const float du0 = fmaf(u0, rho2, -r3.z * dzu);
    const float du1 = fmaf(u1, rho2, -r3.w * dzu);
    gr[G_KU] = -u0 * dz;
    gr[G_KV] = -u1 * dz;
    gr[G_Q00] = du0 * e.dx;
    gr[G_Q01] = du0 * e.dy;
    gr[G_Q10] = du1 * e.dx;
    gr[G_Q11] = du1 * e.dy;
    const float nfd = e.ub ? 0.f : -(inv_s2 * rho2);
    gr[G_CX] = fmaf(-r2.x, du0, fmaf(-r2.z, du1, e.dx * nfd));
    gr[G_CY] = fmaf(-r2.y, du0, fmaf(-r2.w, du1, e.dy * nfd));
}

// Gradients of one (record, pixel) pair in the sequential back-to-front walk.  Updates
// the pixel's transmittance Tr and suffix gS when the pair contributes, returns the 16
// record gradient values in gr (zero when it does not).
template <bool DIST>
__device__ __forceinline__ void pair_gradients(const PairEval &e, bool contrib, float4 r2,
                                               float4 r3, float4 r4, float4 r5,
                                               const PixelAdjoint &pa, const DistPixel &dp,
                                               bool has_vis, float inv_s2, float alpha_max,
                                               float ds, float &Tr, float &gS, float (&gr)[16])
{
    const PairTerms t = pair_terms<DIST>(e, r3, r4, r5, pa, dp, has_vis, ds);
    const float Tb = Tr * t.rom;
    const float w = contrib ? e.alpha * Tb : 0.f;
    const float dal = contrib ? fmaf(Tb, t.gf, -gS * t.rom) : 0.f;
    gS = fmaf(w, t.gf, gS);
    Tr = contrib ? Tb : Tr;
    pair_record_grads(e, w, dal, w * t.gDe, t.u0, t.u1, r2, r3, pa, inv_s2, alpha_max, gr);
}

// --------------------------------------------------------------- raster backward
// Back to front over each pixel's contributors [0, last): transmittance before a
// surfel is recovered as T_i = T_{i+1} / (1 - alpha_i) from T_final, the suffix
// g . sum_{j>i} w_j f_j is accumulated on the way, and per pair
//   dL/dalpha_i = T_i (g . f_i) - (g . S_i) / (1 - alpha_i)           (Eq. rasterization)
// then through alpha = min(alpha_max, o G), G = exp(-rho/2), rho = |Q delta|^2 or
// |delta|^2 / sigma^2, delta = x - c, z = z0 - k . u.  Each 16-lane row of a wave owns a
// 4x4 quadrant of the wave's 8x8 pixels and walks, back to front, the staged records
// whose box meets the quadrant (4 ballots per chunk of 64).  A lane takes part in a pair
// only where the forward composited it - the forward's box and FP32 alpha tests and the
// pixel's `last` - so the walk revisits exactly the forward's pairs.  (Only on a workspace
// without room for the forward's contributor masks at the plan's tile size: one bound with
// less than the full size, or at another tile size; with them the kernel below runs.)
// The 16 record-gradient values are reduced within the row and added with one atomic per
// lane, so one instruction carries the sums of up to four records.
// The colour adjoint of Eq. image_formation runs first per pixel; its 15 per-view
// sums are reduced per tile into colour_partials.
template <int TS, bool HAS_VIS, bool DIST>
__global__ __launch_bounds__(TS *TS) __attribute__((amdgpu_waves_per_eu(TS == 8 ? 5 : 4))) void k_raster_bwd(
    int32_t nv, const ViewDesc *__restrict__ views, const uint32_t *__restrict__ ranges,
    const uint32_t *__restrict__ lists, const float4 *__restrict__ rec, int64_t n,
    RasterConsts rc, const float *__restrict__ colC, const float *__restrict__ colc,
    const float *__restrict__ amb, const float *__restrict__ Ain,
    const float *__restrict__ Vin, const float *__restrict__ Tin,
    const int32_t *__restrict__ lastin, const float *__restrict__ dI,
    const float *__restrict__ dD, const float *__restrict__ dN, float *__restrict__ recgrad,
    float *__restrict__ colour_partials, DistArgs da)
{
    constexpr int NT = TS * TS;
    constexpr int NW = NT / 64;
    // LDS: the staged batch (at offset 0, so a record's address is one multiply), its
    // ranks, the waves' colour sums, the tile's largest `last`
    extern __shared__ float4 lds[];
    uint32_t *lds_idx = reinterpret_cast<uint32_t *>(lds + min(rc.batch, NT) * kRecVec4);
    float(*red)[16] = reinterpret_cast<float(*)[16]>(lds_idx + min(rc.batch, NT));
    int &max_last = *reinterpret_cast<int *>(red + NW);
    const int tile = rc.torder ? (int)rc.torder[blockIdx.x] : xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int v = find_view(views, nv, tile);
    const ViewDesc vd = views[v];
    const int lt = tile - vd.tile_off;
    const int tx = lt % vd.tiles_x, ty = lt / vd.tiles_x;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    constexpr int WPR = TS / 8;
    const int wx0 = tx * TS + (wave % WPR) * 8, wy0 = ty * TS + (wave / WPR) * 8;
    // 16-lane row `quad` owns the 4x4 quadrant (quad & 1, quad >> 1) of the wave's block
    const int quad = lane >> 4;
    const int px = wx0 + 4 * (quad & 1) + (lane & 3), py = wy0 + 4 * (quad >> 1) + ((lane >> 2) & 3);
    const bool inside = px < vd.W && py < vd.H;
    const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
    const int64_t P = (int64_t)vd.W * vd.H;
    const int64_t local = (int64_t)py * vd.W + px;
    const int64_t g = vd.pix_off + local;
    const int64_t b3 = 3 * vd.pix_off + local;
    if (tid == 0) max_last = 0;

    // colour adjoint (Eq. image_formation)
    float cg[16];
    const PixelAdjoint pa = pixel_adjoint<HAS_VIS>(inside, v, g, b3, P, colC, colc, amb, Ain, Vin,
                                                   Tin, lastin, dI, dD, dN, cg);
    const DistPixel dp = DIST ? pixel_distortion_state(inside, g, pa.Tr, da) : DistPixel{0, 0, 0, 0, 0};
    float Tr = pa.Tr;
    const int mylast = pa.last;
    {
        const float s = wave_transpose_reduce16(cg, lane);
        if ((lane & 3) == 0) red[wave][lane >> 2] = s;
    }
    __syncthreads();
    if (tid < 16) {
        float s = 0.f;
        for (int w = 0; w < NW; ++w) s += red[w][tid];
        colour_partials[(int64_t)tile * 16 + tid] = s;
    }
    if (mylast > 0) atomicMax(&max_last, mylast);
    __syncthreads();

    const uint2 range = tile_range(ranges, tile);
    const uint32_t start = range.x;
    const int tile_len = (int)(range.y - start);
    const float4 *recv = rec + (size_t)v * (size_t)n * kRecStride4;
    float *gv = recgrad + (size_t)v * (size_t)n * kGradFloats;
    float gS = 0.f;
    const int batch = min(rc.batch, NT);
    const float inv_s2 = rc.two_inv_s2 * 0.5f;
    const int blk_last = min(max_last, tile_len);   // a stale `last` cannot read past the list
    // the row walks records up to the largest `last` among its 16 pixels
    const int row_last = row_max(mylast);
    // one record per thread; the batch before the current one (back to front) is
    // fetched into registers while the current one is processed
    float4 q0, q1, q2, q3, q4, q5;
    uint32_t qidx = 0;
#define SS_FETCH_BWD(BB, CNT)                                                          \
    if (tid < (CNT)) {                                                                 \
        qidx = min(lists[start + (BB) + tid], (uint32_t)(n - 1));                      \
        const float4 *src_ = recv + (size_t)qidx * kRecStride4;                           \
        q0 = src_[0]; q1 = src_[1]; q2 = src_[2]; q3 = src_[3]; q4 = src_[4]; q5 = src_[5]; \
    }
    // batches [k * batch, (k + 1) * batch) of the list, back to front; the first one is cut at
    // the tile's largest `last`
    const int nbat = (blk_last + batch - 1) / batch;
    if (nbat > 0) {
        const int bb0 = (nbat - 1) * batch;
        SS_FETCH_BWD(bb0, blk_last - bb0);
    }
    for (int kb = nbat - 1; kb >= 0; --kb) {
        const int bb = kb * batch;
        const int nb = min(bb + batch, blk_last) - bb;
        __syncthreads();
        if (tid < nb) {
            float4 *dst = lds + tid * kRecVec4;
            dst[0] = q0; dst[1] = q1; dst[2] = q2; dst[3] = q3; dst[4] = q4; dst[5] = q5;
            lds_idx[tid] = qidx;
        }
        __syncthreads();
        if (kb > 0) SS_FETCH_BWD(bb - batch, batch);
        for (int c0 = ((nb - 1) >> 6) << 6; c0 >= 0; c0 -= 64) {
            const int cnt = min(64, nb - c0);
            uint64_t m = 0;
            // lane t tests chunk record c0 + t against the wave's four 4x4 quadrants
            uint32_t qbits = 0;
            if (lane < cnt) {
                const float4 h = lds[(c0 + lane) * kRecVec4];
                const uint32_t x = __float_as_uint(h.x), y = __float_as_uint(h.y);
                const int xlo = (int)(int16_t)(x & 0xFFFFu), xhi = (int)(int16_t)(x >> 16);
                const int ylo = (int)(int16_t)(y & 0xFFFFu), yhi = (int)(int16_t)(y >> 16);
                const bool c0h = xlo <= wx0 + 3 && xhi >= wx0, c1h = xlo <= wx0 + 7 && xhi >= wx0 + 4;
                const bool r0h = ylo <= wy0 + 3 && yhi >= wy0, r1h = ylo <= wy0 + 7 && yhi >= wy0 + 4;
                qbits = (uint32_t)(c0h && r0h) | ((uint32_t)(c1h && r0h) << 1) |
                        ((uint32_t)(c0h && r1h) << 2) | ((uint32_t)(c1h && r1h) << 3);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t bq = __ballot((qbits >> q) & 1u);
                m = quad == q ? bq : m;
            }
            const int lim = row_last - (bb + c0);        // chunk records j < lim can contribute
            m &= lim >= 64 ? ~0ull : (lim <= 0 ? 0ull : ((1ull << lim) - 1ull));
            // row-uniform walk, highest position first
            if (__ballot(m != 0) != 0) do {
                const bool act = m != 0;
                const int jl = act ? 63 - (int)__builtin_clzll(m) : 0;
                const int j = c0 + jl;
                if (act) m &= ~(1ull << jl);
                const float4 *R = lds + __mul24(j, kRecVec4);   // j < 256: 24-bit multiply
                const float4 r0 = R[0], r1 = R[1], r2 = R[2], r3 = R[3], r4 = R[4], r5 = R[5];
                // branch-free: every lane evaluates the row's record; lanes that do not
                // contribute (outside [0, last) or alpha < alpha_min) get zero gradients
                // and leave T and the suffix unchanged
                const PairEval e = eval_pair(r0, r1, r2, r3, fx, fy, rc);
                // the forward's own decision for this pair: the same FP32 alpha test inside
                // the pixel's FP64 box (the forward never evaluates a pair outside it)
                const uint32_t bx = __float_as_uint(r0.x), by = __float_as_uint(r0.y);
                const int xlo = (int)(int16_t)(bx & 0xFFFFu), xhi = (int)(int16_t)(bx >> 16);
                const int ylo = (int)(int16_t)(by & 0xFFFFu), yhi = (int)(int16_t)(by >> 16);
                const bool contrib = act && bb + j < mylast && px >= xlo && px <= xhi && py >= ylo &&
                                     py <= yhi && e.alpha >= rc.alpha_min;
                // a step where no lane of the wave contributes changes nothing (a branch
                // around the rest, and the loop test at the bottom, keep a single back edge:
                // no register copies per step)
                const uint64_t cb = __ballot(contrib);
                if (cb != 0) {
                    float gr[16];
                    pair_gradients<DIST>(e, contrib, r2, r3, r4, r5, pa, dp, HAS_VIS, inv_s2,
                                         rc.alpha_max, da.ds, Tr, gS, gr);
                    const float sum = row_transpose_reduce16(gr, lane);
                    // lane i of a row holds value i of its record's 16-lane sum
                    if (((cb >> (quad * 16)) & 0xFFFFull) != 0)
                        atomicAdd(gv + (size_t)lds_idx[j] * kGradFloats + (lane & 15), sum);
                }
            } while (__ballot(m != 0) != 0);
        }
    }
#undef SS_FETCH_BWD
}

// ------------------------------------- raster backward from contributor masks
// One wave per 8x8 pixel block, record-parallel rows.  The forward's contributor masks say
// which records of the tile list each pixel composited.  The block's four 4x4 quadrants are
// walked one after another, and all four 16-lane rows of the wave work on the *same*
// quadrant: lane i of every row holds pixel i of the quadrant, and each step takes the next
// four records of the quadrant's walk (the union of its 16 pixels' masks, back to front), one
// per row.  The pixel recursion of Eq. rasterization runs across the rows: with
// rom = 1 / (1 - alpha) for a contributing pair (1 otherwise) and x = w (g . f), row r needs T
// before its record = T_cur * prod_{k <= r} rom_k and the suffix g . S = gS_cur +
// sum_{k < r} x_k; both are scans over the four rows, done lane-wise with two lane swaps each
// (rows 0<->1, 2<->3, then 0,1<->2,3), which also give the totals that advance T_cur and
// gS_cur.  Per-pixel state (the adjoint inputs, T, the suffix, the distortion totals) lives in
// LDS between quadrants.
// Only records of the block's union are read.  An 8x8 tile's list is nearly all union, so its
// 64-position words are staged as they are, a word ahead.  The four (sixteen) blocks of a
// larger tile share a list of which each composites a part (a third of it at 16x16 on the
// 0.5 m/px views), so there the records are staged densely, up to 64 from several words: the
// last step of a quadrant's walk is rarely part-filled.
// Bound by VALU issue (140 instructions a step; the pipes are 92 % busy).  One 2048^2 view of
// 1M surfels 495 -> 471 us, 40 views of 2M 18.6 -> 17.8 ms with 80-byte records in LDS (20
// blocks of 8 KB fit a CU) and without the registers that held the next word's records (5 waves
// per SIMD instead of 4).  With the distortion's state in LDS only 16 blocks fit, and with 16x16
// tiles there are few blocks, so those keep the records ahead: 8 training views of 500k surfels
// 1300 -> 1200 us, three ~530^2 views of 150k surfels at 16x16 234 us (273 us without;
// 430 us for the box-test walk above).
// A step of 16 records x 4 pixels, its scans along the lanes of a row and its sum over pixels
// on the FP32 matrix cores, issues a quarter fewer VALU instructions but waits on LDS and the
// matrix pipe at 4 waves per SIMD: 28.3 ms and 749 us.
constexpr int kPstBase = 10, kPstDist = 5;

__device__ __forceinline__ float swap16_lo_hi(float v, float &hi)
{
    // rows [v0, v1, v2, v3] -> lo = [v0, v0, v2, v2], hi = [v1, v1, v3, v3]
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    hi = __uint_as_float(r[1]);
    return __uint_as_float(r[0]);
}

__device__ __forceinline__ float swap32_lo_hi(float v, float &hi)
{
    // rows [v0, v1, v2, v3] -> lo = [v0, v1, v0, v1], hi = [v2, v3, v2, v3]
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    hi = __uint_as_float(r[1]);
    return __uint_as_float(r[0]);
}

// Inclusive product over rows 0..r (per lane position), and the product of all four.
__device__ __forceinline__ float rows_prefix_mul(float f, bool odd, bool upper, float &total)
{
    float b;
    const float a = swap16_lo_hi(f, b);
    const float pair = a * b;                       // f0 f1 in rows 0, 1; f2 f3 in rows 2, 3
    const float p1 = odd ? pair : a;
    float d;
    const float c = swap32_lo_hi(pair, d);          // c = f0 f1, d = f2 f3 in every row
    total = c * d;
    return upper ? p1 * c : p1;
}

// Inclusive sum over rows 0..r, and the sum of all four.
__device__ __forceinline__ float rows_prefix_add(float x, bool odd, bool upper, float &total)
{
    float b;
    const float a = swap16_lo_hi(x, b);
    const float pair = a + b;
    const float p1 = odd ? pair : a;
    float d;
    const float c = swap32_lo_hi(pair, d);
    total = c + d;
    return upper ? p1 + c : p1;
}

// A staged record: centre, Q, (o, z0, k) with o negative where the record has no ellipse,
// albedo with visibility, normal with the record's rank.
constexpr int kBwdVec4 = 5;
// Launches of up to this many 8x8 blocks give every quadrant a wave of its own (SPLIT): a chip
// holds 4096-5120 of these waves, so fewer blocks leave it to its longest ones.  With larger tiles
// the four waves each stage the whole block's records.  Backward stage of one view, one wave a
// block -> four, in us (in brackets with the distortion, whose four-wave form costs 5-12 % more):
//    8x8:  1024 blocks 113 ->  45 (119 ->  47)    8100: 168 -> 124 (169 -> 133)
//         15,625: 243 -> 214 (247 -> 235)       19,044: 268 -> 260 (268 -> 287)
//   16x16: 1024 blocks 132 ->  67 (133 ->  68)    8128: 194 -> 166 (184 -> 178)
//         10,816: 220 -> 215 (223 -> 233)       13,024: 226 -> 234 (224 -> 255)
//   32x32: 1024 blocks 135 ->  71 (140 ->  73)    4096: 165 -> 151 (170 -> 162)
//           6400: 167 -> 162 (171 -> 179)         8576: 197 -> 204 (200 -> 222)
constexpr int64_t bwd_split(int ts) { return ts == 8 ? 16384 : 8192; }

template <int TS, bool HAS_VIS, bool DIST, bool FILT, bool SPLIT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(DIST || TS > 8 ? 4 : 5))) void k_raster_bwd_rp(
    int32_t nv, const ViewDesc *__restrict__ views, int32_t ntiles, const uint32_t *__restrict__ ranges,
    const uint32_t *__restrict__ lists, const float4 *__restrict__ rec, int64_t n,
    RasterConsts rc, const float *__restrict__ colC, const float *__restrict__ colc,
    const float *__restrict__ amb, const float *__restrict__ Ain,
    const float *__restrict__ Vin, const float *__restrict__ Tin,
    const int32_t *__restrict__ lastin, const float *__restrict__ dI,
    const float *__restrict__ dD, const float *__restrict__ dN, float *__restrict__ recgrad,
    float *__restrict__ colour_partials, const unsigned long long *__restrict__ cmask,
    DistArgs da)
{
    constexpr int WPR = TS / 8, SUB = WPR * WPR, NT = TS * TS;
    constexpr bool DENSE = TS > 8, AHEAD = DIST || DENSE;
    constexpr int kPst = kPstBase + (DIST ? kPstDist : 0);
    // staged records (a record's address is one multiply), per-pixel state [field][pixel], the
    // quadrant's walk list, the block's largest `last`
    __shared__ float4 lds[64 * kBwdVec4];
    __shared__ float pst[kPst * 64];
    __shared__ uint32_t qlist[68];
    __shared__ int max_last;
    // blocks go round-robin to the 8 XCDs: the blocks of a tile stay on the tile's XCD
    constexpr int PER = SUB * (SPLIT ? 4 : 1);
    // a split wave stages its quadrant's records; dense batches are made of the whole block's,
    // so that every quadrant is walked in the same steps as by one wave
    constexpr bool MINE = SPLIT && !DENSE;
    const int b = (int)blockIdx.x;
    const int vb = PER == 1 ? b : 8 * (b / (8 * PER)) + b % 8;
    const int part = PER == 1 ? 0 : (b / 8) % PER;
    const int sub = SPLIT ? part >> 2 : part, qsel = SPLIT ? part & 3 : 0;
    if (vb >= ntiles) return;
    const int tile = rc.torder ? (int)rc.torder[vb] : xcd_tile(vb, ntiles);
    const int v = find_view(views, nv, tile);
    const ViewDesc vd = views[v];
    const int lt = tile - vd.tile_off;
    const int tx = lt % vd.tiles_x, ty = lt / vd.tiles_x;
    const int lane = threadIdx.x;
    const int wx0 = tx * TS + (sub % WPR) * 8, wy0 = ty * TS + (sub / WPR) * 8;
    const int row = lane >> 4, li = lane & 15;
    const bool odd = lane & 16, upper = lane & 32;
    // prologue in the owner mapping: lane 16 q + i holds pixel i of quadrant q
    const int opx = wx0 + 4 * (row & 1) + (li & 3), opy = wy0 + 4 * (row >> 1) + (li >> 2);
    const bool inside = opx < vd.W && opy < vd.H;
    const int64_t P = (int64_t)vd.W * vd.H;
    const int64_t local = (int64_t)opy * vd.W + opx;
    const int64_t g = vd.pix_off + local;
    const int64_t b3 = 3 * vd.pix_off + local;
    if (lane == 0) max_last = 0;
    float cg[16];
    {
        const PixelAdjoint pa = pixel_adjoint<HAS_VIS>(inside, v, g, b3, P, colC, colc, amb, Ain, Vin,
                                                       Tin, lastin, dI, dD, dN, cg);
        const float s = wave_transpose_reduce16(cg, lane);
        if ((lane & 3) == 0 && qsel == 0) colour_partials[((int64_t)tile * SUB + sub) * 16 + (lane >> 2)] = s;
        pst[0 * 64 + lane] = pa.gA0; pst[1 * 64 + lane] = pa.gA1; pst[2 * 64 + lane] = pa.gA2;
        pst[3 * 64 + lane] = pa.gV;  pst[4 * 64 + lane] = pa.gD;
        pst[5 * 64 + lane] = pa.gN0; pst[6 * 64 + lane] = pa.gN1; pst[7 * 64 + lane] = pa.gN2;
        pst[8 * 64 + lane] = pa.Tr;  pst[9 * 64 + lane] = 0.f;
        if (DIST) {
            const DistPixel dp = pixel_distortion_state(inside, g, pa.Tr, da);
            pst[10 * 64 + lane] = dp.gDist; pst[11 * 64 + lane] = dp.zref;
            pst[12 * 64 + lane] = dp.At;    pst[13 * 64 + lane] = dp.M1;
            pst[14 * 64 + lane] = dp.M2;
        }
        if (pa.last > 0 && (!MINE || row == qsel)) atomicMax(&max_last, pa.last);
    }
    __syncthreads();
    const uint2 range = tile_range(ranges, tile);
    const uint32_t start = range.x;
    const int blk_last = min(max_last, (int)(range.y - start));   // a stale `last` stays inside the list
    if (blk_last <= 0) return;
    const float4 *recv = rec + (size_t)v * (size_t)n * kRecStride4;
    float *gv = recgrad + (size_t)v * (size_t)n * kGradFloats;
    const float inv_s2 = rc.two_inv_s2 * 0.5f;
    // this lane's pixel's masks: word kb of the list at own_at[kb * NT]
    const unsigned long long *own_at = cmask + ((size_t)(start >> 6) + (size_t)tile) * NT + sub * 64 +
                                       (((opy - wy0) << 3) | (opx - wx0));

    // Walks the staged records, highest slot first; `own` holds the slots that this lane's
    // pixel composited, row q of `un` their union over quadrant q.
    auto walk = [&](const uint64_t own, const uint64_t un) {
        __syncthreads();
#pragma unroll
        for (int qi = 0; qi < (SPLIT ? 1 : 4); ++qi) {
            const int q = SPLIT ? qsel : qi;
            const uint64_t U = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(un >> 32), 16 * q) << 32) |
                               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)un, 16 * q);
            if (U == 0) continue;                     // uniform
            const int nq = __popcll(U);
            // walk list of the quadrant: slot of the k-th set bit from the top
            {
                const bool set = (U >> lane) & 1ull;
                const int k = lane == 63 ? 0 : __popcll(U >> (lane + 1));
                if (set) qlist[k] = (uint32_t)lane;
                // rows past the end of the walk read a staged record too (their weight is zero)
                const uint32_t spare = (uint32_t)__builtin_ctzll(U);
                if (lane >= nq) qlist[lane] = spare;
                if (lane < 4) qlist[64 + lane] = spare;
            }
            const int p = 16 * q + li;               // the quadrant's pixel of this lane
            const float gA0 = pst[0 * 64 + p], gA1 = pst[1 * 64 + p], gA2 = pst[2 * 64 + p];
            const float gV = pst[3 * 64 + p], gD = pst[4 * 64 + p];
            const float gN0 = pst[5 * 64 + p], gN1 = pst[6 * 64 + p], gN2 = pst[7 * 64 + p];
            float Tr = pst[8 * 64 + p], gS = pst[9 * 64 + p];
            DistPixel dp{0, 0, 0, 0, 0};
            if (DIST) {
                dp.gDist = pst[10 * 64 + p]; dp.zref = pst[11 * 64 + p]; dp.At = pst[12 * 64 + p];
                dp.M1 = pst[13 * 64 + p]; dp.M2 = pst[14 * 64 + p];
            }
            const uint64_t ownq =
                ((uint64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(4 * p, (int)(uint32_t)(own >> 32)) << 32) |
                (uint32_t)__builtin_amdgcn_ds_bpermute(4 * p, (int)(uint32_t)own);
            const PixelAdjoint pa{gA0, gA1, gA2, gV, gD, gN0, gN1, gN2, Tr, 0};
            const int qpx = wx0 + 4 * (q & 1) + (li & 3), qpy = wy0 + 4 * (q >> 1) + (li >> 2);
            const float fx = (float)qpx + 0.5f, fy = (float)qpy + 0.5f;
            __syncthreads();                         // the walk list is complete
            // record slots are read one step ahead
            const uint32_t *next = qlist + row;
            int jl_next = (int)*next;
            for (int left = nq; left > 0; left -= 4) {
                const bool act = row < left;
                const int jl = jl_next;
                next += 4;
                jl_next = (int)*next;
                const float4 *R = lds + __mul24(jl, kBwdVec4);
                const float4 c = R[0], r2 = R[1], r3 = R[2], r4 = R[3], r5 = R[4];
                const PairEval e = eval_staged<FILT>(c, r2, fabsf(r3.x), r3.x > 0.f, fx, fy, rc);
                const bool contrib = act && ((ownq >> jl) & 1ull);
                const PairTerms t = pair_terms<DIST>(e, r3, r4, r5, pa, dp, HAS_VIS, da.ds);
                const float f = contrib ? t.rom : 1.f;
                float ptot;
                const float Pinc = rows_prefix_mul(f, odd, upper, ptot);
                const float Tb = Tr * Pinc;          // T before this row's record
                const float w = contrib ? e.alpha * Tb : 0.f;
                const float x = w * t.gf;
                float stot;
                const float Sinc = rows_prefix_add(x, odd, upper, stot);
                const float gSb = gS + (Sinc - x);   // g . S after this row's record
                const float dal = contrib ? fmaf(Tb, t.gf, -gSb * t.rom) : 0.f;
                Tr *= ptot;
                gS += stot;
                float gr[16];
                pair_record_grads(e, w, dal, w * t.gDe, t.u0, t.u1, r2, r3, pa, inv_s2,
                                  rc.alpha_max, gr);
                const float sum = row_transpose_reduce16(gr, lane);
                // every walked record is composited by some pixel of the quadrant
                if (act) atomicAdd(gv + (size_t)__float_as_uint(r5.w) * kGradFloats + li, sum);
            }
            if (row == 0) {
                pst[8 * 64 + p] = Tr;
                pst[9 * 64 + p] = gS;
            }
            __syncthreads();                         // list and state reused by the next quadrant
        }
    };

    // Words of the list, back to front.  Ahead of the word in work (AHEAD): the records of the
    // next, of lanes whose position is in the block's union Un, and masks and list entries of the
    // one after; otherwise the next word's masks and list entries only.
    float2 qc;                                        // record on its way to LDS: centre,
    float3 qb, qn;                                    // its low part and a bias; normal
    float4 q2, q3, q4;
    uint32_t qidx = 0, nidx = 0;
    uint64_t own_n = 0, un_n = 0, Un = 0, own_nn = 0;
    int kb = (blk_last + 63) >> 6;
    auto load_word = [&](int k) {                     // masks and list entries of word k
        const int nb = blk_last - 64 * k;
        own_nn = inside && (!MINE || row == qsel) ? own_at[(size_t)k * NT] : 0ull;
        if (nb < 64) own_nn &= (1ull << nb) - 1ull;
        if (lane < nb) nidx = lists[start + 64 * k + lane];
    };
    auto fetch_word = [&]() {                         // unions and records of the loaded word
        own_n = own_nn;
        un_n = row_or64(own_n);
        Un = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            Un |= ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(un_n >> 32), 16 * q) << 32) |
                  (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)un_n, 16 * q);
        qidx = min(nidx, (uint32_t)(n - 1));
        if ((Un >> lane) & 1ull) {
            const float4 *src = recv + (size_t)qidx * kRecStride4;
            const float *f = reinterpret_cast<const float *>(src);
            qc = *reinterpret_cast<const float2 *>(f + 2);
            qb = *reinterpret_cast<const float3 *>(f + 4);
            q2 = src[2]; q3 = src[3]; q4 = src[4];
            qn = *reinterpret_cast<const float3 *>(f + 20);
        }
    };
    auto stage = [&](int slot) {
        float4 *dst = lds + slot * kBwdVec4;
        dst[0] = make_float4(qc.x, qc.y, qb.x, qb.y);
        dst[1] = q2; dst[3] = q4;
        dst[2] = make_float4(qb.z > 0.f ? -q3.x : q3.x, q3.y, q3.z, q3.w);
        dst[4] = make_float4(qn.x, qn.y, qn.z, __uint_as_float(qidx));
    };
    load_word(kb - 1);
    if (AHEAD) {
        fetch_word();
        if (kb > 1) load_word(kb - 2);
    }
    if constexpr (!DENSE) {
        while (--kb >= 0) {
            if (!AHEAD) {
                fetch_word();
                if (kb > 0) load_word(kb - 1);
            }
            if ((Un >> lane) & 1ull) stage(lane);
            const uint64_t own = own_n, un = un_n;
            if (AHEAD && kb > 0) fetch_word();
            if (AHEAD && kb > 1) load_word(kb - 2);
            walk(own, un);
        }
    } else {
        int staged = 0;                               // slots 63, 62, ... are taken in turn
        uint64_t own_s = 0;
        --kb;
        for (;;) {
            if (kb >= 0) {
                // the last records of the word that still fit
                const int top = lane == 63 ? 0 : __popcll(Un >> (lane + 1));
                const bool sel = ((Un >> lane) & 1ull) && top < 64 - staged;
                uint64_t take = __ballot(sel);
                Un &= ~take;
                if (sel) stage(63 - staged - top);
                while (take != 0) {                   // this pixel's bits to the records' slots
                    const int j = 63 - (int)__builtin_clzll(take);
                    take &= ~(1ull << j);
                    own_s |= ((own_n >> j) & 1ull) << (63 - staged);
                    ++staged;
                }
                if (Un == 0) {
                    if (--kb >= 0) {
                        fetch_word();
                        if (kb > 0) load_word(kb - 1);
                    }
                }
                if (staged < 64 && kb >= 0) continue;
            }
            if (staged > 0) walk(own_s, row_or64(own_s));
            if (kb < 0) break;
            staged = 0;
            own_s = 0;
        }
    }
}

template <int TS, bool HV, bool DIST>
static void launch_bwd_d(size_t lds, hipStream_t st, int32_t ntiles, int32_t nv,
                         const ViewDesc *views, const uint32_t *ranges, const uint32_t *lists,
                         const float *rec, int64_t n, const RasterConsts &rc,
                         const float *colC, const float *colc, const float *amb,
                         const float *A, const float *V, const float *T, const int32_t *last,
                         const float *dI, const float *dD, const float *dN, float *recgrad,
                         float *cp, const unsigned long long *cmask, const DistArgs &da)
{
    if (cmask) {
        const bool split = raster_blocks(ts_sub(TS), ntiles) <= bwd_split(TS);
        const dim3 grid((unsigned)raster_blocks(ts_sub(TS) * (split ? 4 : 1), ntiles));
#define SS_BWD_LAUNCH(FILT_, SPLIT_)                                                                   \
    hipLaunchKernelGGL((k_raster_bwd_rp<TS, HV, DIST, FILT_, SPLIT_>), grid, dim3(64), 0, st, nv, views, \
                       ntiles, ranges, lists, reinterpret_cast<const float4 *>(rec), n, rc, colC,      \
                       colc, amb, A, V, T, last, dI, dD, dN, recgrad, cp, cmask, da)
        if (rc.lowpass_mode == 0) {
            if (split) SS_BWD_LAUNCH(true, true);
            else SS_BWD_LAUNCH(true, false);
        } else {
            if (split) SS_BWD_LAUNCH(false, true);
            else SS_BWD_LAUNCH(false, false);
        }
#undef SS_BWD_LAUNCH
        return;
    }
    hipLaunchKernelGGL((k_raster_bwd<TS, HV, DIST>), dim3((unsigned)ntiles), dim3(TS * TS), lds, st, nv,
                       views, ranges, lists, reinterpret_cast<const float4 *>(rec), n, rc, colC, colc,
                       amb, A, V, T, last, dI, dD, dN, recgrad, cp, da);
}

template <int TS, bool HV>
static void launch_bwd_t(size_t lds, hipStream_t st, int32_t ntiles, int32_t nv,
                         const ViewDesc *views, const uint32_t *ranges, const uint32_t *lists,
                         const float *rec, int64_t n, const RasterConsts &rc,
                         const float *colC, const float *colc, const float *amb,
                         const float *A, const float *V, const float *T, const int32_t *last,
                         const float *dI, const float *dD, const float *dN, float *recgrad,
                         float *cp, const unsigned long long *cmask, const DistArgs *dist)
{
    const DistArgs da = dist ? *dist : DistArgs{0.f, nullptr, nullptr, nullptr, 0};
    if (dist)
        launch_bwd_d<TS, HV, true>(lds, st, ntiles, nv, views, ranges, lists, rec, n, rc, colC, colc,
                                   amb, A, V, T, last, dI, dD, dN, recgrad, cp, cmask, da);
    else
        launch_bwd_d<TS, HV, false>(lds, st, ntiles, nv, views, ranges, lists, rec, n, rc, colC, colc,
                                    amb, A, V, T, last, dI, dD, dN, recgrad, cp, cmask, da);
}

hipError_t launch_raster_bwd(int ts, bool has_vis, int32_t total_tiles, int32_t nv,
                             const ViewDesc *views, const uint32_t *ranges,
                             const uint32_t *lists, const float *rec, int64_t n,
                             const RasterConsts &rc, const float *colC, const float *colc,
                             const float *amb, const float *A, const float *V,
                             const float *T, const int32_t *last, const float *dI,
                             const float *dD, const float *dN, float *recgrad,
                             float *colour_partials, const unsigned long long *cmask,
                             hipStream_t st, const DistArgs *dist)
{
    if (total_tiles <= 0) return hipSuccess;
    const size_t lds = (size_t)min(rc.batch, ts * ts) * (kRecVec4 * sizeof(float4) + sizeof(uint32_t)) +
                       (size_t)(ts * ts / 64) * 16 * sizeof(float) + sizeof(int);
#define SS_BWD(TS_)                                                                          \
    if (ts == TS_) {                                                                         \
        if (has_vis)                                                                         \
            launch_bwd_t<TS_, true>(lds, st, total_tiles, nv, views, ranges, lists, rec, n, rc, \
                                    colC, colc, amb, A, V, T, last, dI, dD, dN, recgrad,     \
                                    colour_partials, cmask, dist);                           \
        else                                                                                 \
            launch_bwd_t<TS_, false>(lds, st, total_tiles, nv, views, ranges, lists, rec, n, rc, \
                                     colC, colc, amb, A, V, T, last, dI, dD, dN, recgrad,    \
                                     colour_partials, cmask, dist);                          \
    }
    SS_BWD(8) else SS_BWD(16) else SS_BWD(32) else return hipErrorInvalidValue;
#undef SS_BWD
    return hipGetLastError();
}

int raster_bwd_sub(int ts, bool masks) { return masks ? ts_sub(ts) : 1; }

// ----------------------------------------------------------- projection backward
// One thread per rank, looping over views: record gradients -> parameter gradients
// (summed over views, written once), and per view the camera-delta gradient dF = [dB | db]
// reduced per block into dF_partials.  The parameter gradients leave as one 64-byte row per
// rank, over the rank's first record gradient, which only this thread reads; k_grads_out
// takes the rows to the caller's arrays in surfel order.  Writing the six arrays from here
// touches a line of each per surfel: 1 view of 1M surfels 110 us, now 40 + 32; 40 views of 2M
// 1440 us, now 1057 + 64.  Up to kPbDirect surfels the arrays sit in L2 and one launch less
// counts for more (20,000 surfels: 10 us against 9 + 5): then this kernel writes them.
//   c = B p + b:        dp += B^T dc,  dB += dc p^T,  db += dc
//   Q = T^-1:           dT = -Q^T dQ Q^T
//   T = B M:            dB += dT M^T,  dM = B^T dT
//   z0 = b_z - p_z,  k = M[2,:]
//   M = [s_u t_u, s_v t_v],  n = nsign m / |m|,  m = t_u x t_v
constexpr int kPbThreads = 256;
constexpr int64_t kPbDirect = 65536;

// The caller's gradient arrays; order: surfel of each rank, or NULL to leave rows
struct GradOut {
    const uint32_t *order;
    float *mean, *tu, *tv, *scale, *opac, *alb;
};

__global__ __launch_bounds__(kPbThreads) void k_project_bwd(
    const float4 *__restrict__ sp, int64_t n, int32_t nv,
    const float *__restrict__ Fxy, const float *__restrict__ dF, double det_rel_eps, float4 *recgrad,
    float *__restrict__ dF_partials, GradOut dst)
{
    __shared__ float red[kPbThreads / 64][16];
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const bool valid = r < n;
    float p[3] = {0, 0, 0}, tu[3] = {0, 0, 0}, tv[3] = {0, 0, 0}, su = 0, sv = 0;
    if (valid) {
        const float4 a = sp[4 * r], b = sp[4 * r + 1], c = sp[4 * r + 2];
        p[0] = a.x; p[1] = a.y; p[2] = a.z;
        tu[0] = a.w; tu[1] = b.x; tu[2] = b.y;
        tv[0] = b.z; tv[1] = b.w; tv[2] = c.x;
        su = c.y; sv = c.z;
    }
    float M[3][2];
    for (int i = 0; i < 3; ++i) { M[i][0] = su * tu[i]; M[i][1] = sv * tv[i]; }
    float m[3] = {tu[1] * tv[2] - tu[2] * tv[1], tu[2] * tv[0] - tu[0] * tv[2],
                  tu[0] * tv[1] - tu[1] * tv[0]};
    const float mn = sqrtf(m[0] * m[0] + m[1] * m[1] + m[2] * m[2]);
    float gp[3] = {0, 0, 0}, gtu[3] = {0, 0, 0}, gtv[3] = {0, 0, 0}, gsu = 0, gsv = 0, go = 0;
    float ga[3] = {0, 0, 0};
    const double pd_tu[3] = {tu[0], tu[1], tu[2]}, pd_tv[3] = {tv[0], tv[1], tv[2]};
    for (int v = 0; v < nv; ++v) {
        float B[2][3];
        double Bd[2][3];
        for (int row = 0; row < 2; ++row)
            for (int q = 0; q < 3; ++q) {
                B[row][q] = Fxy[8 * v + 4 * row + q] + (dF ? dF[8 * v + 4 * row + q] : 0.f);
                Bd[row][q] = (double)Fxy[8 * v + 4 * row + q] +
                             (dF ? (double)dF[8 * v + 4 * row + q] : 0.0);
            }
        float x[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = 0.f;
        if (valid) {
            const size_t slot = (size_t)v * (size_t)n + (size_t)r;
            const float4 g0 = recgrad[4 * slot], g1 = recgrad[4 * slot + 1];
            const float4 g2 = recgrad[4 * slot + 2], g3 = recgrad[4 * slot + 3];
            const float dc[2] = {g0.x, g0.y};
            const float dQ[2][2] = {{g0.z, g0.w}, {g1.x, g1.y}};
            const float dz0 = g1.z, dk0 = g1.w, dk1 = g2.x, dO = g2.y;
            // Q and the normal's sign exactly as the projection stored them in the record
            const SurfelAffine sa = surfel_affine(Bd, pd_tu, pd_tv, (double)su, (double)sv, det_rel_eps);
            const float nsign = (float)sa.nsign;
            const float Q[2][2] = {{(float)sa.Q[0][0], (float)sa.Q[0][1]},
                                   {(float)sa.Q[1][0], (float)sa.Q[1][1]}};
            float t1[2][2], dT[2][2];
            for (int a = 0; a < 2; ++a)
                for (int q = 0; q < 2; ++q) t1[a][q] = Q[0][a] * dQ[0][q] + Q[1][a] * dQ[1][q];
            for (int a = 0; a < 2; ++a)
                for (int q = 0; q < 2; ++q) dT[a][q] = -(t1[a][0] * Q[q][0] + t1[a][1] * Q[q][1]);
            float dM[3][2];
            for (int row = 0; row < 2; ++row) {
                for (int q = 0; q < 3; ++q)
                    x[4 * row + q] = dT[row][0] * M[q][0] + dT[row][1] * M[q][1] + dc[row] * p[q];
                x[4 * row + 3] = dc[row];
            }
            for (int q = 0; q < 3; ++q) {
                dM[q][0] = B[0][q] * dT[0][0] + B[1][q] * dT[1][0];
                dM[q][1] = B[0][q] * dT[0][1] + B[1][q] * dT[1][1];
                gp[q] += B[0][q] * dc[0] + B[1][q] * dc[1];
            }
            gp[2] -= dz0;
            dM[2][0] += dk0;
            dM[2][1] += dk1;
            float dtu[3], dtv[3];
            for (int q = 0; q < 3; ++q) {
                gsu += tu[q] * dM[q][0];
                gsv += tv[q] * dM[q][1];
                dtu[q] = su * dM[q][0];
                dtv[q] = sv * dM[q][1];
            }
            go += dO;
            ga[0] += g2.z; ga[1] += g2.w; ga[2] += g3.x;
            const float dn[3] = {g3.y, g3.z, g3.w};
            const float nn[3] = {nsign * m[0] / mn, nsign * m[1] / mn, nsign * m[2] / mn};
            const float ndn = nn[0] * dn[0] + nn[1] * dn[1] + nn[2] * dn[2];
            float dm[3];
            for (int q = 0; q < 3; ++q) dm[q] = nsign * (dn[q] - nn[q] * ndn) / mn;
            // dt_u += t_v x dm ; dt_v += dm x t_u
            dtu[0] += tv[1] * dm[2] - tv[2] * dm[1];
            dtu[1] += tv[2] * dm[0] - tv[0] * dm[2];
            dtu[2] += tv[0] * dm[1] - tv[1] * dm[0];
            dtv[0] += dm[1] * tu[2] - dm[2] * tu[1];
            dtv[1] += dm[2] * tu[0] - dm[0] * tu[2];
            dtv[2] += dm[0] * tu[1] - dm[1] * tu[0];
            for (int q = 0; q < 3; ++q) { gtu[q] += dtu[q]; gtv[q] += dtv[q]; }
        }
        const float s = wave_transpose_reduce16(x, lane);
        if ((lane & 3) == 0) red[w][lane >> 2] = s;
        __syncthreads();
        if (threadIdx.x < 8) {
            float tot = 0.f;
            for (int k = 0; k < kPbThreads / 64; ++k) tot += red[k][threadIdx.x];
            dF_partials[((int64_t)v * gridDim.x + blockIdx.x) * 8 + threadIdx.x] = tot;
        }
        __syncthreads();
    }
    if (!valid) return;
    if (dst.order) {
        const int64_t i = dst.order[r];
        if (i >= n) return;
        for (int q = 0; q < 3; ++q) {
            dst.mean[3 * i + q] = gp[q];
            dst.tu[3 * i + q] = gtu[q];
            dst.tv[3 * i + q] = gtv[q];
            dst.alb[3 * i + q] = ga[q];
        }
        dst.scale[2 * i] = gsu;
        dst.scale[2 * i + 1] = gsv;
        dst.opac[i] = go;
        return;
    }
    float4 *row = recgrad + 4 * r;
    row[0] = make_float4(gp[0], gp[1], gp[2], gtu[0]);
    row[1] = make_float4(gtu[1], gtu[2], gtv[0], gtv[1]);
    row[2] = make_float4(gtv[2], gsu, gsv, go);
    row[3] = make_float4(ga[0], ga[1], ga[2], 0.f);
}

__global__ __launch_bounds__(kPermBlock) void k_grads_out(
    const uint32_t *__restrict__ rank, int64_t n, const float4 *__restrict__ grads,
    float *__restrict__ d_mean, float *__restrict__ d_tu, float *__restrict__ d_tv,
    float *__restrict__ d_scale, float *__restrict__ d_opac, float *__restrict__ d_alb)
{
    __shared__ float rows[kPermBlock * kPermRow];
    const int64_t i0 = (int64_t)blockIdx.x * kPermBlock;
    const int cnt = (int)min((int64_t)kPermBlock, n - i0);
    for (int e = threadIdx.x; e < cnt * 4; e += kPermBlock) {
        const int64_t r = min((int64_t)rank[i0 + (e >> 2)], n - 1);
        const float4 x = grads[4 * r + (e & 3)];
        float *p = rows + (e >> 2) * kPermRow + 4 * (e & 3);
        p[0] = x.x; p[1] = x.y; p[2] = x.z; p[3] = x.w;
    }
    __syncthreads();
    rows_out<3>(rows, i0, cnt, 0, d_mean);
    rows_out<3>(rows, i0, cnt, 3, d_tu);
    rows_out<3>(rows, i0, cnt, 6, d_tv);
    rows_out<2>(rows, i0, cnt, 9, d_scale);
    rows_out<1>(rows, i0, cnt, 11, d_opac);
    rows_out<3>(rows, i0, cnt, 12, d_alb);
}

int project_bwd_blocks(int64_t n) { return (int)((n + kPbThreads - 1) / kPbThreads); }

hipError_t launch_project_bwd(const float *sorted, int64_t n, const uint32_t *order,
                              const uint32_t *rank, int32_t nv, const float *Fxy, const float *dF, double det_rel_eps,
                              float *recgrad, float *d_mean, float *d_tu, float *d_tv,
                              float *d_scale, float *d_opac, float *d_alb, float *dF_partials,
                              hipStream_t st)
{
    const int nb = project_bwd_blocks(n);
    if (nb == 0) return hipSuccess;
    float4 *rg = reinterpret_cast<float4 *>(recgrad);
    hipLaunchKernelGGL(k_project_bwd, dim3((unsigned)nb), dim3(kPbThreads), 0, st,
                       reinterpret_cast<const float4 *>(sorted), n, nv, Fxy, dF, det_rel_eps, rg,
                       dF_partials,
                       GradOut{n <= kPbDirect ? order : nullptr, d_mean, d_tu, d_tv, d_scale, d_opac, d_alb});
    if (n > kPbDirect)
        hipLaunchKernelGGL(k_grads_out, dim3((unsigned)((n + kPermBlock - 1) / kPermBlock)), dim3(kPermBlock),
                           0, st, rank, n, rg, d_mean, d_tu, d_tv, d_scale, d_opac, d_alb);
    return hipGetLastError();
}

// Per-view sums of the backward's partial rows: `sub` x 16 floats per tile (dC 9, dc 3, dL_a
// 3) and 8 per project_bwd block (dF).  Both are sums of chains with a fixed order (256 chains
// per colour column, chain t over rows t, t + 256, ...; 32 per dF column), so that the colour
// terms and camera deltas of a training run do not depend on how the chains are spread over
// blocks.  Blocks (c, v) with c < chunks carry 256 / chunks colour chains of view v, one
// thread per chain and column with its loads in flight together; with one chunk the block
// also adds the chains up, with more k_view_finish does.  Block (chunks, v) sums the view's
// dF rows.  One block per view, one load at a time, left a single 2048^2 view's 65,536 tile
// rows to one CU (125 us) and took 29 us for the dF rows of 1M surfels; now 16 us for both
// (40 views, 2M surfels: 257 -> 36 us).
constexpr int kVrThreads = 256;
constexpr int kVrChunks = 16;

// Chain sums of view v (acc of thread t: the 16 columns of chain t) -> d_colC, d_colc, d_amb
__device__ __forceinline__ void finish_colour(float (&acc)[16], float (*red)[16], int v,
                                              float *d_colC, float *d_colc, float *d_amb)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const float s = wave_transpose_reduce16(acc, lane);
    if ((lane & 3) == 0) red[w][lane >> 2] = s;
    __syncthreads();
    if (threadIdx.x < 15) {
        const int k = threadIdx.x;
        const float tot = red[0][k] + red[1][k] + red[2][k] + red[3][k];
        if (k < 9) d_colC[9 * v + k] = tot;
        else if (k < 12) d_colc[3 * v + k - 9] = tot;
        else d_amb[3 * v + k - 12] = tot;
    }
}

template <int SUB>
__global__ __launch_bounds__(kVrThreads) void k_view_reduce(
    const float *__restrict__ colour_rows, const ViewDesc *__restrict__ views,
    const float *__restrict__ dF_rows, int nblocks, float *__restrict__ d_colC,
    float *__restrict__ d_colc, float *__restrict__ d_amb, float *__restrict__ d_dF,
    float *__restrict__ parts)
{
    __shared__ float red[kVrThreads / 64][16];
    __shared__ float col[kVrThreads];
    const int v = blockIdx.y, chunks = gridDim.x - 1, c = blockIdx.x, t = threadIdx.x;
    if (c == chunks) {
        const float *p = dF_rows + 8 * (int64_t)v * nblocks + (t & 7);
        float s = 0.f;
#pragma unroll 16
        for (int b = t >> 3; b < nblocks; b += 32) s += p[8 * b];
        col[t] = s;                                        // 32 x 8 chain sums
        __syncthreads();
        if (t < 8) {
            float x = 0.f;
            for (int k = 0; k < 32; ++k) x += col[8 * k + t];
            d_dF[8 * v + t] = x;
        }
        return;
    }
    const int rows = views[v].tiles_x * views[v].tiles_y;
    const float *p = colour_rows + 16 * (int64_t)views[v].tile_off * SUB;
    // a tile's row is the sum of its SUB rows, in order
    auto row = [&](int r, int k) {
        const float *q = p + 16 * (int64_t)r * SUB + k;
        float x = q[0];
#pragma unroll
        for (int w = 1; w < SUB; ++w) x += q[16 * w];
        return x;
    };
    if (chunks == 1) {
        float acc[16];
        for (int k = 0; k < 16; ++k) acc[k] = 0.f;
        for (int r = t; r < rows; r += kVrThreads)
            for (int k = 0; k < 16; ++k) acc[k] += row(r, k);
        finish_colour(acc, red, v, d_colC, d_colc, d_amb);
        return;
    }
    // kVrChunks == 16: thread t carries column t % 16 of chain 16 c + t / 16
    const int chain = 16 * c + (t >> 4);
    float s = 0.f;
#pragma unroll 16 / SUB
    for (int r = chain; r < rows; r += kVrThreads) s += row(r, t & 15);
    parts[((int64_t)v * kVrThreads + chain) * 16 + (t & 15)] = s;
}

__global__ __launch_bounds__(kVrThreads) void k_view_finish(const float *__restrict__ parts,
                                                            float *__restrict__ d_colC,
                                                            float *__restrict__ d_colc,
                                                            float *__restrict__ d_amb)
{
    __shared__ float red[kVrThreads / 64][16];
    const float *p = parts + ((int64_t)blockIdx.x * kVrThreads + threadIdx.x) * 16;
    float acc[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[k] = p[k];
    finish_colour(acc, red, blockIdx.x, d_colC, d_colc, d_amb);
}

size_t view_reduce_parts(int32_t nv) { return (size_t)nv * kVrThreads * 16; }

hipError_t launch_view_reduce(const float *colour_rows, int sub, int64_t max_view_tiles, const float *dF_rows,
                              int nblocks, int32_t nv, const ViewDesc *views, float *d_colC,
                              float *d_colc, float *d_amb, float *d_dF, float *parts, hipStream_t st)
{
    if (nv <= 0) return hipSuccess;
    // up to 8 rows per chain one block per view costs less than a second launch
    const int chunks = max_view_tiles * sub > 8 * kVrThreads ? kVrChunks : 1;
    const dim3 grid((unsigned)chunks + 1, (unsigned)nv);
#define SS_VR(SUB_)                                                                                  \
    hipLaunchKernelGGL((k_view_reduce<SUB_>), grid, dim3(kVrThreads), 0, st, colour_rows, views, dF_rows, \
                       nblocks, d_colC, d_colc, d_amb, d_dF, parts)
    if (sub == 1) SS_VR(1);
    else if (sub == 4) SS_VR(4);
    else if (sub == 16) SS_VR(16);
    else return hipErrorInvalidValue;
#undef SS_VR
    if (chunks > 1)
        hipLaunchKernelGGL(k_view_finish, dim3((unsigned)nv), dim3(kVrThreads), 0, st, parts, d_colC,
                           d_colc, d_amb);
    return hipGetLastError();
}

// Scatter per-(view, rank) rows back to per-(view, surfel) order for debug output.
__global__ void k_unpermute_rows(const uint32_t *__restrict__ order, int64_t n, int32_t nv,
                                 const uint32_t *__restrict__ in, int in_stride,
                                 int row_words, uint32_t *__restrict__ out)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y;
    if (r >= n) return;
    if (order[r] >= n) return;
    const int64_t src = ((int64_t)v * n + r) * in_stride;
    const int64_t dst = ((int64_t)v * n + order[r]) * row_words;
    for (int k = 0; k < row_words; ++k) out[dst + k] = k < in_stride ? in[src + k] : 0u;
}

hipError_t launch_unpermute_rows(const uint32_t *order, int64_t n, int32_t nv,
                                 const uint32_t *in, int in_stride, int row_words,
                                 uint32_t *out, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_unpermute_rows, dim3((unsigned)((n + 255) / 256), (unsigned)nv),
                       dim3(256), 0, st, order, n, nv, in, in_stride, row_words, out);
    return hipGetLastError();
}

// Per-(view, rank) short4 tile ranges -> int32 [view, surfel, 4] in surfel order.
__global__ void k_unpermute_tiles(const uint32_t *__restrict__ order, int64_t n,
                                  const short4 *__restrict__ t, int32_t *__restrict__ out)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int v = blockIdx.y;
    if (r >= n) return;
    if (order[r] >= n) return;
    const short4 s = t[(int64_t)v * n + r];
    int32_t *o = out + 4 * ((int64_t)v * n + order[r]);
    o[0] = s.x; o[1] = s.y; o[2] = s.z; o[3] = s.w;
}

hipError_t launch_unpermute_tiles(const uint32_t *order, int64_t n, int32_t nv, const short4 *t,
                                  int32_t *out, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_unpermute_tiles, dim3((unsigned)((n + 255) / 256), (unsigned)nv),
                       dim3(256), 0, st, order, n, t, out);
    return hipGetLastError();
}

__global__ void k_map_through(const uint32_t *__restrict__ order, int64_t n_order,
                              const unsigned long long *n_dev, int64_t cap,
                              const uint32_t *__restrict__ in, uint32_t *__restrict__ out)
{
    unsigned long long nn = *n_dev;
    const int64_t n = nn < (unsigned long long)cap ? (int64_t)nn : cap;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = order[in[i] < n_order ? in[i] : 0];
}

hipError_t launch_map_through(const uint32_t *order, int64_t n_order,
                              const unsigned long long *n_dev, int64_t cap, const uint32_t *in,
                              uint32_t *out, hipStream_t st)
{
    if (cap <= 0 || n_order <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_map_through, dim3((unsigned)((cap + 255) / 256)), dim3(256), 0, st, order,
                       n_order, n_dev, cap, in, out);
    return hipGetLastError();
}

}  // namespace ss
