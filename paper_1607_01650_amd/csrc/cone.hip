// Cone-beam Joseph projector pair for the 3-D circular scan (the scanner of
// Sec. 3; the fan-beam path is its central plane) on gfx950.
//
// Source s = R (cos t, sin t, 0); flat panel centred at -(D - R)(cos t, sin t,
// 0), bin b of row j at u_b = (b - (B-1)/2) du + offset along (-sin t, cos t,
// 0) and v_j = (j - (J-1)/2) dv along z.  Volume [nz][ny][nx] of cubic voxels,
// projections [V][J][B].  Each ray steps along the in-plane axis it is more
// aligned with; on every plane of that axis its crossing (in-plane coordinate
// and height) is interpolated bilinearly between the four nearest voxel
// centres, and the samples are scaled by the path length per plane.
//
//   k_cone_pad_x, k_cone_pad_y : two zero-padded permuted copies of the
//                volume, [x][z][y] for x-major rays and [y][z][x] for
//                y-major rays, so that a sample's two in-plane taps are
//                adjacent (borders written as zeros by the same kernels: no
//                memset in the path).
//   k_cone_fwd : one thread per ray (64 adjacent bins of one row per
//                wavefront); the ray's constants are formed in FP64 from the
//                view's cos/sin and turned into 32.32 fixed point (in-plane
//                coordinate and height per plane), stepped by integer adds;
//                FP32 bilinear samples summed in FP64.
//   k_cone_pad_z, k_cone_fwd_z : the same with lanes along the rows, on one padded
//                copy [y][x][z]: from 32 rows per chunk, one volume of up to 64
//                slices from 24 (by lines).
//   k_cone_tab, k_cone_scale, k_cone_gather : the transpose in gather form
//                (no atomics, the same result on every run): per-(view, bin)
//                ray constants, projections times each ray's path length,
//                then one thread per voxel column and 4 slices sums over
//                the rays that reach it (see k_cone_gather).
//   k_cone_scale_z, k_cone_gather_z : the same for volumes of 20 slices and
//                more, with lanes along z.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "reduce.h"
#include "volume.h"
#include "xcd.h"

namespace dect {
namespace {

constexpr int kCPad = 2;  // zero lines on each side of the padded copies
constexpr double kTwo32c = 4294967296.0;
constexpr float kTwoM32c = 2.3283064365386963e-10f;

struct ConeDev {
    int nx, ny, nz, V, J, B;
    double voxel, bin, row, off, sod, sdd;
    const double *cs;  // [V][2] cos, sin of the view angle
};

struct ConeRay {
    int64_t a, k, az, kz;  // 32.32 in-plane coordinate and height at plane 0, steps
    float L;               // path length per plane
    int xmaj;
};

__device__ __forceinline__ ConeRay cone_ray(const ConeDev &g, int v, int j, int b)
{
    const double ct = g.cs[2 * v], st = g.cs[2 * v + 1];
    const double u = (b - (g.B - 1) / 2.0) * g.bin + g.off;
    const double w = (j - (g.J - 1) / 2.0) * g.row;
    const double sx = g.sod * ct, sy = g.sod * st;
    const double px = -(g.sdd - g.sod) * ct - u * st, py = -(g.sdd - g.sod) * st + u * ct;
    const double dx = px - sx, dy = py - sy, dz = w;
    const double len = sqrt(dx * dx + dy * dy + dz * dz);
    ConeRay r;
    r.xmaj = fabs(dx) >= fabs(dy);
    double a, k, kz, az;
    if (r.xmaj) {
        k = dy / dx;
        kz = dz / dx;
        const double x0 = (0 - (g.nx - 1) / 2.0) * g.voxel;
        a = (sy + (x0 - sx) * k) / g.voxel + (g.ny - 1) / 2.0;
        az = ((x0 - sx) * kz) / g.voxel + (g.nz - 1) / 2.0;
        r.L = (float)(g.voxel * len / fabs(dx));
    } else {
        k = dx / dy;
        kz = dz / dy;
        const double y0 = (0 - (g.ny - 1) / 2.0) * g.voxel;
        a = (sx + (y0 - sy) * k) / g.voxel + (g.nx - 1) / 2.0;
        az = ((y0 - sy) * kz) / g.voxel + (g.nz - 1) / 2.0;
        r.L = (float)(g.voxel * len / fabs(dy));
    }
    // |a|, |az| stay far below 2^31 for validated geometries (rays outside
    // the volume are clamped to a far coordinate and contribute zero)
    a = fmin(fmax(a, -1.0e6), 1.0e6);
    az = fmin(fmax(az, -1.0e6), 1.0e6);
    r.a = __double2ll_rn(a * kTwo32c);
    r.k = __double2ll_rn(k * kTwo32c);
    r.az = __double2ll_rn(az * kTwo32c);
    r.kz = __double2ll_rn(kz * kTwo32c);
    return r;
}

// vol [nz][ny][nx] -> vx [nx][nz+4][ny+4] and vy [ny][nz+4][nx+4], written
// whole (zero borders included).  NE = 2: the two volumes interleaved
// ([..][2]), so that one load carries a tap of both.
//
// k_cone_pad_x: vx is a transpose (y fastest), staged through a 32 x 32
// LDS tile per (x block, padded-y block, padded slice): read along x, write
// along y.  k_cone_pad_y: vy keeps x fastest, one thread per element.
template <int NE>
__global__ __launch_bounds__(256) void k_cone_pad_x(const float *__restrict__ vol0,
                                                    const float *__restrict__ vol1, int nx, int ny,
                                                    int nz, float *__restrict__ vx)
{
    __shared__ float tile[NE][32][33];
    const int pz = nz + 2 * kCPad, py = ny + 2 * kCPad;
    const int x0 = blockIdx.x * 32, yp0 = blockIdx.y * 32, zp = blockIdx.z;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int z = zp - kCPad;
    const float *vol[2] = {vol0, vol1};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int y = yp0 + ty + 8 * r - kCPad, x = x0 + tx;
        const bool in = x < nx && y >= 0 && y < ny && z >= 0 && z < nz;
#pragma unroll
        for (int e = 0; e < NE; ++e)
            tile[e][ty + 8 * r][tx] = in ? vol[e][((size_t)z * ny + y) * nx + x] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int x = x0 + ty + 8 * r, yp = yp0 + tx;
        if (x < nx && yp < py) {
            const size_t o = ((size_t)x * pz + zp) * py + yp;
#pragma unroll
            for (int e = 0; e < NE; ++e) vx[o * NE + e] = tile[e][tx][ty + 8 * r];
        }
    }
}

template <int NE>
__global__ __launch_bounds__(256) void k_cone_pad_y(const float *__restrict__ vol0,
                                                    const float *__restrict__ vol1, int nx, int ny,
                                                    int nz, float *__restrict__ vy)
{
    const int pz = nz + 2 * kCPad, px = nx + 2 * kCPad;
    const size_t nvy = (size_t)ny * pz * px;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const float *vol[2] = {vol0, vol1};
    if (i < nvy) {  // vy: x fastest
        const int xx = (int)(i % px) - kCPad, zz = (int)(i / px % pz) - kCPad;
        const int y = (int)(i / ((size_t)px * pz));
        const bool in = xx >= 0 && xx < nx && zz >= 0 && zz < nz;
#pragma unroll
        for (int e = 0; e < NE; ++e)
            vy[i * NE + e] = in ? vol[e][((size_t)zz * ny + y) * nx + xx] : 0.f;
    }
}

// four floats at 8-byte alignment: taps h and h + 1 of both volumes
typedef float c4a8 __attribute__((ext_vector_type(4), aligned(8)));
typedef float c2 __attribute__((ext_vector_type(2)));

template <int NE>
__global__ __launch_bounds__(256) void k_cone_fwd(ConeDev g, const float *__restrict__ vx,
                                                  const float *__restrict__ vy,
                                                  float *__restrict__ proj0,
                                                  float *__restrict__ proj1,
                                                  float *__restrict__ lo0,
                                                  float *__restrict__ lo1)
{
    const size_t nray = (size_t)g.V * g.J * g.B;
    const size_t rid = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (rid >= nray) return;
    const int b = (int)(rid % g.B), j = (int)(rid / g.B % g.J), v = (int)(rid / ((size_t)g.B * g.J));
    const ConeRay r = cone_ray(g, v, j, b);
    const int nl = r.xmaj ? g.nx : g.ny, nq = r.xmaj ? g.ny : g.nx;
    const int pq = nq + 2 * kCPad, pz = g.nz + 2 * kCPad;
    const float *base = r.xmaj ? vx : vy;
    int64_t q = r.a, qz = r.az;
    double acc[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) acc[e] = 0.0;
    for (int i0 = 0; i0 < nl; i0 += 4) {
        float s[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) s[e] = 0.f;
        const int i1 = min(nl, i0 + 4);
        for (int i = i0; i < i1; ++i) {
            const int h = min(max((int)(q >> 32), -2), nq);
            const int hz = min(max((int)(qz >> 32), -2), g.nz);
            const float wa = (float)(uint32_t)q * kTwoM32c;
            const float wz = (float)(uint32_t)qz * kTwoM32c;
            const size_t o0 = ((size_t)i * pz + hz + kCPad) * pq + h + kCPad;
            if constexpr (NE == 1) {
                const float *p0 = base + o0;
                const float *p1 = p0 + pq;
                const float lo = fmaf(wa, p0[1] - p0[0], p0[0]);
                const float hi = fmaf(wa, p1[1] - p1[0], p1[0]);
                s[0] += fmaf(wz, hi - lo, lo);
            } else {
                const c4a8 a0 = *(const c4a8 *)(base + 2 * o0);
                const c4a8 a1 = *(const c4a8 *)(base + 2 * (o0 + pq));
                const float lo0 = fmaf(wa, a0.z - a0.x, a0.x), hi0 = fmaf(wa, a1.z - a1.x, a1.x);
                const float lo1 = fmaf(wa, a0.w - a0.y, a0.y), hi1 = fmaf(wa, a1.w - a1.y, a1.y);
                s[0] += fmaf(wz, hi0 - lo0, lo0);
                s[1] += fmaf(wz, hi1 - lo1, lo1);
            }
            q += r.k;
            qz += r.kz;
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[e] += (double)s[e];
    }
    // the FP64 ray sum rounded to FP32; with lo buffers also its rounding
    // error, so that proj + lo carries the sum to about 2^-48
    const double v0 = acc[0] * (double)r.L;
    const float h0 = (float)v0;
    proj0[rid] = h0;
    if (lo0) lo0[rid] = (float)(v0 - (double)h0);
    if constexpr (NE == 2) {
        const double v1 = acc[1] * (double)r.L;
        const float h1 = (float)v1;
        proj1[rid] = h1;
        if (lo1) lo1[rid] = (float)(v1 - (double)h1);
    }
}

// vol [nz][ny][nx] -> vp [ny+4][nx+4][nz+4] (NE = 2: the two volumes
// interleaved), slices adjacent, written whole with its zero borders: the
// layout k_cone_fwd_z reads for both ray classes.  32 x 32 tiles of one image
// line turned through LDS.
template <int NE>
__global__ __launch_bounds__(256) void k_cone_pad_z(const float *__restrict__ vol0,
                                                    const float *__restrict__ vol1, int nx, int ny,
                                                    int nz, float *__restrict__ vp)
{
    __shared__ float tile[NE][32][33];
    const int pz = nz + 2 * kCPad, px = nx + 2 * kCPad;
    const int xp0 = blockIdx.x * 32, zp0 = blockIdx.y * 32, yp = blockIdx.z;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int y = yp - kCPad, x = xp0 + tx - kCPad;
    const float *vol[2] = {vol0, vol1};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int z = zp0 + ty + 8 * r - kCPad;
        const bool in = x >= 0 && x < nx && y >= 0 && y < ny && z >= 0 && z < nz;
#pragma unroll
        for (int e = 0; e < NE; ++e)
            tile[e][ty + 8 * r][tx] = in ? vol[e][((size_t)z * ny + y) * nx + x] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int xp = xp0 + ty + 8 * r, zp = zp0 + tx;
        if (xp < px && zp < pz) {
            const size_t o = (((size_t)yp * px + xp) * pz + zp) * NE;
#pragma unroll
            for (int e = 0; e < NE; ++e) vp[o + e] = tile[e][tx][ty + 8 * r];
        }
    }
}

// proj = A3 vol with lanes along the panel's rows, for panels of enough rows:
// one (view, bin) per wavefront, up to 64 rows (lane = row).  The in-plane
// coordinate is then the wavefront's (scalar arithmetic), the taps of the
// lanes lie along one or two runs of slices of one copy of the volume that
// serves both ray classes, and only the planes on which the ray is inside the
// image are walked.  Same samples, groups and sums as k_cone_fwd: the results
// are equal bit for bit.
//
// LINE, for one volume of up to 64 slices: lane = slice as well.  A wavefront
// loads the two lines that a plane's sample lies between once, 4 bytes per
// lane next to each other, mixes them into one line in LDS (the same in-plane
// interpolation as per row, at slices in place of rows) and each lane then
// reads its two slices there.  Bound by VALU issue, some 16 instructions per
// sample.  (For a pair the VALU binds either way: 1.01 against 1.00 ms at the
// size below.)
//
// Without LINE, bound by the vector memory path: two 8-byte loads per lane and
// sample, which the L1 serves four lanes at a time (18 accesses a load; the
// address and data units are busy 98% of the time), and the L2 misses of the
// volume.  Blocks are dealt in groups of eight views by eight bundles, which
// cross the same part of the volume (4.47 -> 4.34 ms).
//
// 512 x 512 x 64, 360 x 64 x 736, k_cone_fwd / without / with LINE: 8.6 / 4.2 /
// 2.2 ms; a pair on 320 x 289 x 40, 240 x 40 x 460: 1.79 / 1.00 ms.
// Wavefronts per block without LINE: 4, 8 and 16 take 4.19, 4.22 and 4.31 ms
// (with it 8 take 7% longer than 4); two 4-byte loads per row in place of an
// 8-byte one take 6.0 ms.
constexpr int kFZWaves = 4;
constexpr int kFZGroup = 8;
// Rows per chunk from which it is the faster one: it takes the same time for
// any number of rows (512 x 512 x 64 with every ray inside the volume, 360
// views: 5.25 ms, with LINE 2.85), k_cone_fwd 0.13 ms per row there (2.22 ms
// for 16, 3.06 for 24; 256 x 256 x 32, 180 views: 0.54 ms for 32 rows, 0.54
// here, with LINE 0.37).
constexpr int kFZMinRows = 32, kFZMinRowsLine = 24;

template <int NE> struct ZPair;
template <> struct ZPair<1> { typedef float T __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct ZPair<2> { typedef float T __attribute__((ext_vector_type(4), aligned(8))); };

constexpr int kFZSlices = 64;  // slices at most with LINE (one per lane)
constexpr int kFZUnroll = 4;   // planes per FP32 sum, and whose lines are in flight together

template <int NE, bool LINE>
__global__ __launch_bounds__(kFZWaves * 64) void k_cone_fwd_z(ConeDev g,
                                                              const float *__restrict__ vp,
                                                              int rper,
                                                              float *__restrict__ proj0,
                                                              float *__restrict__ proj1,
                                                              float *__restrict__ lo0,
                                                              float *__restrict__ lo1)
{
    typedef typename ZPair<NE>::T P;
    static_assert(NE == 1 || !LINE, "lines of one volume");
    // LINE: a wavefront's image lines, slices -2 .. nz + 1 at entries 0 ..
    __shared__ float line[LINE ? kFZWaves : 1][LINE ? kFZUnroll : 1][LINE ? kFZSlices + 2 * kCPad : 1];
    __shared__ double out[NE][64][kFZWaves + 1];
    const unsigned item = xcd_order(block_linear(), grid_blocks());
    // blocks in groups of kFZGroup views by kFZGroup bundles
    const int nbun = (int)gridDim.x, nv = (int)gridDim.y;
    const int it = (int)(item % (unsigned)(nbun * nv));
    const int v0 = it / (kFZGroup * nbun) * kFZGroup, vn = min(kFZGroup, nv - v0);
    const int r0 = it - v0 * nbun, u0 = r0 / (kFZGroup * vn) * kFZGroup;
    const int un = min(kFZGroup, nbun - u0), rr = r0 - u0 * vn;
    const int bb = (u0 + rr % un) * kFZWaves, v = v0 + rr / un;
    const int j0 = (int)(item / (unsigned)(nbun * nv)) * rper;
    const int nj = min(rper, g.J - j0);
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = bb + wid;
    if (b < g.B) {
        // the in-plane terms are the same for every row
        const ConeRay r = cone_ray(g, v, j0 + min(lane, nj - 1), b);
        auto uniform = [](int64_t x) {
            const unsigned lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)x);
            const unsigned hi = __builtin_amdgcn_readfirstlane((int)(x >> 32));
            return (int64_t)(((uint64_t)hi << 32) | lo);
        };
        const int64_t a = uniform(r.a), k = uniform(r.k);
        const bool xmaj = __builtin_amdgcn_readfirstlane(r.xmaj);
        const int nl = xmaj ? g.nx : g.ny, nq = xmaj ? g.ny : g.nx;
        const unsigned pz = (unsigned)(g.nz + 2 * kCPad) * (4 * NE);
        const unsigned px = (unsigned)(g.nx + 2 * kCPad) * pz;
        const unsigned sl = xmaj ? pz : px, sh = xmaj ? px : pz;  // plane and line, in bytes
        // the planes between which the ray crosses the lines -1 .. nq (one more each side)
        int i0 = 0, i1 = nl;
        {
            const double A = (double)a, K = (double)k;
            const double t0 = (-kTwo32c - A) / K, t1 = (nq * kTwo32c - A) / K;
            if (k != 0) {
                i0 = (int)fmin(fmax(floor(fmin(t0, t1)) - 1.0, 0.0), (double)nl);
                i1 = (int)fmin(fmax(ceil(fmax(t0, t1)) + 2.0, 0.0), (double)nl);
            }
            i0 = __builtin_amdgcn_readfirstlane(i0) & ~3;  // whole groups of four planes
            i1 = __builtin_amdgcn_readfirstlane(i1);
        }
        int64_t q = a + k * i0;
        int64_t qz = r.az + r.kz * i0;
        unsigned plane = (unsigned)(i0 + kCPad) * sl + kCPad * sh;
        double acc[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[e] = 0.0;
        auto sample = [&](float (&s)[NE]) {
            const int h = min(max((int)(q >> 32), -2), nq);
            unsigned line = plane + (unsigned)h * sh;
            asm("" : "+s"(line));  // keeps the address arithmetic in 32 bits
            const char *line0 = (const char *)vp + line, *line1 = line0 + sh;
            int hz;  // the height's voxel, clamped to [-2, nz]
            asm("v_med3_i32 %0, %1, -2, %2" : "=v"(hz) : "v"((int)(qz >> 32)), "s"(g.nz));
            const float wa = (float)(uint32_t)q * kTwoM32c;
            const float wz = (float)(uint32_t)qz * kTwoM32c;
            const unsigned off = (unsigned)(hz + kCPad) * (4u * NE);
            const P p0 = *(const P *)(line0 + off), p1 = *(const P *)(line1 + off);
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const float lo = fmaf(wa, p1[e] - p0[e], p0[e]);
                const float hi = fmaf(wa, p1[NE + e] - p0[NE + e], p0[NE + e]);
                s[e] += fmaf(wz, hi - lo, lo);
            }
            q += k;
            qz += r.kz;
            plane += sl;
            asm("" : "+s"(q), "+v"(qz), "+s"(plane));  // one running value each
        };
        int i = i0;
        if constexpr (LINE) {
            float(&buf)[kFZUnroll][kFZSlices + 2 * kCPad] = line[wid];
            if (lane < 2 * kCPad)  // the borders that no lane's slice covers
#pragma unroll
                for (int u = 0; u < kFZUnroll; ++u)
                    buf[u][lane < kCPad ? lane : kFZSlices + lane] = 0.f;
            // the lane's slice; past the last one the zero border's first
            const unsigned mine = (unsigned)(min(lane, g.nz) + kCPad) * (4u * NE);
            for (; i + kFZUnroll <= min(nl, i1 + 3); i += kFZUnroll) {
                unsigned at_z = mine;
                asm("" : "+v"(at_z));  // stays an offset to the lines' scalar addresses
                float p0[kFZUnroll], p1[kFZUnroll], wa[kFZUnroll], wz[kFZUnroll];
                int hz[kFZUnroll];
#pragma unroll
                for (int u = 0; u < kFZUnroll; ++u) {
                    const int h = min(max((int)(q >> 32), -2), nq);
                    unsigned at = plane + (unsigned)h * sh;
                    asm("" : "+s"(at));  // keeps the address arithmetic in 32 bits
                    const char *line0 = (const char *)vp + at, *line1 = line0 + sh;
                    p0[u] = *(const float *)(line0 + at_z);
                    p1[u] = *(const float *)(line1 + at_z);
                    wa[u] = (float)(uint32_t)q * kTwoM32c;
                    asm("v_med3_i32 %0, %1, -2, %2" : "=v"(hz[u]) : "v"((int)(qz >> 32)), "s"(g.nz));
                    wz[u] = (float)(uint32_t)qz * kTwoM32c;
                    q += k;
                    qz += r.kz;
                    plane += sl;
                    asm("" : "+s"(q), "+v"(qz), "+s"(plane));  // one running value each
                }
                wave_order();  // the reads of the lines before are done (LDS is in order)
#pragma unroll
                for (int u = 0; u < kFZUnroll; ++u) buf[u][lane + kCPad] = fmaf(wa[u], p1[u] - p0[u], p0[u]);
                wave_order();
                float s = 0.f;
#pragma unroll
                for (int u = 0; u < kFZUnroll; ++u) {
                    const float lo = buf[u][hz[u] + kCPad], hi = buf[u][hz[u] + kCPad + 1];
                    s += fmaf(wz[u], hi - lo, lo);
                }
                acc[0] += (double)s;
            }
        }
        for (; !LINE && i + 4 <= min(nl, i1 + 3); i += 4) {
            float s[NE] = {};
#pragma unroll
            for (int u = 0; u < 4; ++u) sample(s);
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[e] += (double)s[e];
        }
        if (i < i1) {
            float s[NE] = {};
            for (; i < nl; ++i) sample(s);
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[e] += (double)s[e];
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) out[e][lane][wid] = acc[e] * (double)r.L;
    }
    __syncthreads();
    // stored along the bins; as in k_cone_fwd, with its rounding error where asked
    const int t = threadIdx.x;
    for (int n = t; n < nj * kFZWaves; n += kFZWaves * 64) {
        const int jj = n / kFZWaves, w = n % kFZWaves;
        if (bb + w >= g.B) continue;
        const size_t o = ((size_t)v * g.J + j0 + jj) * g.B + bb + w;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const double x = out[e][jj][w];
            const float hi = (float)x;
            (e ? proj1 : proj0)[o] = hi;
            float *lo = e ? lo1 : lo0;
            if (lo) lo[o] = (float)(x - (double)hi);
        }
    }
}

// Per (view, bin): the ray's 32.32 in-plane coordinate at plane 0 and its
// step (as in the forward walk), its class, and the height coefficients:
// at plane p the ray's height is qz = w * (g0 + g1 p) + (nz - 1)/2 voxels,
// w the row's height on the panel.
struct ConeTab {
    int64_t a, k;
    double g0, g1;
    int32_t xmaj, pad;
};

__global__ __launch_bounds__(256) void k_cone_tab(ConeDev g, ConeTab *__restrict__ tab)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= g.V * g.B) return;
    const int v = i / g.B, b = i % g.B;
    const ConeRay r = cone_ray(g, v, 0, b);  // in-plane terms do not depend on the row
    const double ct = g.cs[2 * v], st = g.cs[2 * v + 1];
    const double u = (b - (g.B - 1) / 2.0) * g.bin + g.off;
    const double sx = g.sod * ct, sy = g.sod * st;
    const double dx = -(g.sdd - g.sod) * ct - u * st - sx;
    const double dy = -(g.sdd - g.sod) * st + u * ct - sy;
    const double dp = r.xmaj ? dx : dy, sp = r.xmaj ? sx : sy;
    const int np = r.xmaj ? g.nx : g.ny;
    ConeTab t;
    t.a = r.a;
    t.k = r.k;
    t.g0 = ((0 - (np - 1) / 2.0) * g.voxel - sp) / (dp * g.voxel);
    t.g1 = 1.0 / dp;
    t.xmaj = r.xmaj;
    t.pad = 0;
    tab[i] = t;
}

// yl = L * proj (NE = 2: both projections interleaved), L the forward
// walk's path length per plane of each ray.
template <int NE>
__global__ __launch_bounds__(256) void k_cone_scale(ConeDev g, const float *__restrict__ proj0,
                                                    const float *__restrict__ proj1,
                                                    float *__restrict__ yl)
{
    const size_t nray = (size_t)g.V * g.J * g.B;
    const size_t rid = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (rid >= nray) return;
    const int b = (int)(rid % g.B), j = (int)(rid / g.B % g.J), v = (int)(rid / ((size_t)g.B * g.J));
    const float L = cone_ray(g, v, j, b).L;
    yl[rid * NE] = proj0[rid] * L;
    if constexpr (NE == 2) yl[rid * 2 + 1] = proj1[rid] * L;
}

#ifndef DECT_CONE_ZC
#define DECT_CONE_ZC 4
#endif
constexpr int kZC = DECT_CONE_ZC;  // slices per gather thread

// vol = A3^T proj in gather form.  Thread: voxel column (x, y), slices
// [z0, z0 + kZC); lanes along x.  Per view, the rays that can reach the
// column cross the segments (x, y -+ 1) (x-major rays, on plane x) or
// (x -+ 1, y) (y-major rays, on plane y); their bins lie between the
// panel positions of those four points.  Every candidate's in-plane weight
// comes from its exact 32.32 coordinate (the forward's interpolation
// weight); the rows reaching slice z are those whose height on the ray's
// plane lies within one voxel of z, the height taken in FP64 at the first
// such row and stepped in FP32 (a few rows).  Per-view sums in FP32,
// accumulated over views in FP64.
template <int NE>
__global__ __launch_bounds__(256) void k_cone_gather(ConeDev g, const ConeTab *__restrict__ tab,
                                                     const float *__restrict__ yl,
                                                     float *__restrict__ vol0,
                                                     float *__restrict__ vol1)
{
    const int x = blockIdx.x * 64 + (threadIdx.x & 63);
    const int y = blockIdx.y;
    const int z0 = (blockIdx.z * 4 + (threadIdx.x >> 6)) * kZC;
    if (x >= g.nx || z0 >= g.nz) return;
    const float vox = (float)g.voxel;
    const float px = (x - (g.nx - 1) * 0.5f) * vox, py = (y - (g.ny - 1) * 0.5f) * vox;
    const float R = (float)g.sod, D = (float)g.sdd;
    const float ibin = (float)(1.0 / g.bin), bc = (float)((g.B - 1) / 2.0 - g.off / g.bin);
    const double cz = (g.nz - 1) / 2.0, jc = (g.J - 1) / 2.0;
    const size_t JB = (size_t)g.J * g.B;
    double acc[kZC][NE];
#pragma unroll
    for (int t = 0; t < kZC; ++t)
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[t][e] = 0.0;
    for (int v = 0; v < g.V; ++v) {
        const float ct = (float)g.cs[2 * v], st = (float)g.cs[2 * v + 1];
        const float sx = R * ct, sy = R * st;
        // continuous bin of the ray through (qx, qy)
        auto bin_of = [&](float qx, float qy) {
            const float rx = qx - sx, ry = qy - sy;
            return -D * (ry * ct - rx * st) / (rx * ct + ry * st) * ibin + bc;
        };
        const float b1 = bin_of(px, py - vox), b2 = bin_of(px, py + vox);
        const float b3 = bin_of(px - vox, py), b4 = bin_of(px + vox, py);
        const float bmin = fminf(fminf(b1, b2), fminf(b3, b4));
        const float bmax = fmaxf(fmaxf(b1, b2), fmaxf(b3, b4));
        // clamped before conversion (bounds only; the exact test below decides)
        const int bl = max(0, (int)ceilf(fminf(fmaxf(bmin - 1e-3f, -1.f), (float)g.B)));
        const int bh = min(g.B - 1, (int)floorf(fminf(fmaxf(bmax + 1e-3f, -1.f), (float)g.B)));
        float part[kZC][NE];
#pragma unroll
        for (int t = 0; t < kZC; ++t)
#pragma unroll
            for (int e = 0; e < NE; ++e) part[t][e] = 0.f;
        const ConeTab *tv = tab + (size_t)v * g.B;
        const float *yv = yl + (size_t)v * JB * NE;
        for (int b = bl; b <= bh; ++b) {
            const ConeTab tb = tv[b];
            const int pl = tb.xmaj ? x : y, c = tb.xmaj ? y : x;
            // bilinear weights are the tent 1 - |q - c| (in-plane, exact in
            // 32.32 as in the forward walk) times 1 - |qz - z| (height)
            const int64_t dq = tb.a + tb.k * pl - ((int64_t)c << 32);
            const uint64_t adq = (uint64_t)(dq < 0 ? -dq : dq);
            if (adq >= (1ull << 32)) continue;
            const float wi = 1.f - (float)(uint32_t)adq * kTwoM32c;
            const double sb = (tb.g0 + tb.g1 * pl) * g.row;  // height step per row (> 0)
            const double qz0 = cz - jc * sb;                  // height of row 0
            const float sbf = (float)sb, isb = 1.f / sbf;
            const float lo0 = (float)(z0 - 1 - qz0) * isb;
            const float *yb = yv + (size_t)b * NE;
#pragma unroll
            for (int t = 0; t < kZC; ++t) {
                // rows with |qz - z| < 1: j in (lo, lo + 2/sb)
                const float lo = lo0 + t * isb, hi = lo + 2.f * isb;
                const int j0 = max(0, (int)floorf(fminf(fmaxf(lo, -1.f), (float)g.J)) + 1);
                const int j1 = min(g.J - 1, (int)ceilf(fminf(fmaxf(hi, -1.f), (float)g.J)) - 1);
                const float e0 = (float)(qz0 + j0 * sb - (z0 + t));  // qz - z at row j0
                float s[NE];
#pragma unroll
                for (int e = 0; e < NE; ++e) s[e] = 0.f;
                for (int j = j0; j <= j1; ++j) {
                    const float w = fmaxf(0.f, 1.f - fabsf(fmaf((float)(j - j0), sbf, e0)));
                    if constexpr (NE == 1) {
                        s[0] = fmaf(w, yb[(size_t)j * g.B], s[0]);
                    } else {
                        const c2 yy = *(const c2 *)(yb + (size_t)j * g.B * 2);
                        s[0] = fmaf(w, yy.x, s[0]);
                        s[1] = fmaf(w, yy.y, s[1]);
                    }
                }
#pragma unroll
                for (int e = 0; e < NE; ++e) part[t][e] = fmaf(wi, s[e], part[t][e]);
            }
        }
#pragma unroll
        for (int t = 0; t < kZC; ++t)
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[t][e] += (double)part[t][e];
    }
    const size_t plane = (size_t)g.nx * g.ny;
#pragma unroll
    for (int t = 0; t < kZC; ++t)
        if (z0 + t < g.nz) {
            const size_t o = (size_t)(z0 + t) * plane + (size_t)y * g.nx + x;
            vol0[o] = (float)acc[t][0];
            if constexpr (NE == 2) vol1[o] = (float)acc[t][1];
        }
}

// yl[v][b][JP][NE] = L * proj with the rows of a bin contiguous and zero rows
// around them (padlo before row 0): the layout k_cone_gather_z reads.  One
// 32 x 32 tile of (padded row, bin) per block, turned through LDS.
template <int NE>
__global__ __launch_bounds__(256) void k_cone_scale_z(ConeDev g, const float *__restrict__ proj0,
                                                      const float *__restrict__ proj1, int JP,
                                                      int padlo, float *__restrict__ yl)
{
    __shared__ float tile[NE][32][33];
    const int b0 = blockIdx.x * 32, p0 = blockIdx.y * 32, v = blockIdx.z;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const float *proj[2] = {proj0, proj1};
    for (int r = ty; r < 32; r += 8) {
        const int b = b0 + tx, j = p0 + r - padlo;
        const bool in = b < g.B && j >= 0 && j < g.J;
        const float L = in ? cone_ray(g, v, j, b).L : 0.f;
#pragma unroll
        for (int e = 0; e < NE; ++e)
            tile[e][r][tx] = in ? proj[e][((size_t)v * g.J + j) * g.B + b] * L : 0.f;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int b = b0 + r, jp = p0 + tx;
        if (b < g.B && jp < JP) {
            const size_t o = (((size_t)v * g.B + b) * JP + jp) * NE;
#pragma unroll
            for (int e = 0; e < NE; ++e) yl[o + e] = tile[e][tx][r];
        }
    }
}

// vol = A3^T proj with lanes along z: the gather for volumes of enough slices.
//
// A block owns an 8 x 8 tile of voxel columns over up to 64 slices (lane =
// slice).  Wavefront w first takes the x-major rays on plane x0 + w, lines
// y0 .. y0 + 7, then the y-major rays on plane y0 + w, lines x0 .. x0 + 7.
// On one plane a view's rays are ordered, so they are walked in the order of
// their line: a ray's height resampling u(z) (the rows whose height lies
// within one voxel of z) is formed once and given to its two columns, h
// with 1 - w and h + 1 with w, in a two-column FP32 window that slides along
// the lines; when the window leaves a column, its sum over this view is added
// to the column's FP64 sum in LDS (read when the window arrived there).
// Everything that does not depend on z (the exact 32.32 tap line and weight,
// the height step, the first row) is evaluated for the rays of four views at
// once, one ray per lane, and broadcast ray by ray through LDS (two 16-byte
// reads; a readlane per value is VALU work), so control flow is uniform.
//
// The first row's height over slice z is k_cone_gather's (FP64, rounded once)
// to a few 1e-9 voxel: the step and the height of a row near the chunk's middle
// are split in a multiple of 2^-18 (kGGrid), whose sums below 2^6 are exact, and
// a rest below 2^-19 as FP16 units of 2^-18.  The rows after it take the step in
// FP32, as there.  (With both in two FP32 parts, three instructions instead of
// four, a height loses the bits of the distance between rows: A^T's error at
// rows 20 voxels apart was 1.5e-7, 2.8e-8 now and with k_cone_gather.)
//
// Bound by VALU issue (88% of it, by the counters): 23 vector, 15 scalar and 3
// LDS instructions per (ray, plane) of 64 slices, against 50 to 60 vector ones
// per voxel and view of k_cone_gather, which finds a column's rays and rows again
// for every 4 slices.  512 x 512 x 64, 360 x 64 x 736: 5.6 ms (18.0 ms with k_cone_gather),
// 170 cycles per ray and SIMD; a pair on 320 x 289 x 40, 240 x 40 x 460:
// 2.06 ms (3.94 ms).  Rays in flight (kGBatch): 2, 3, 6 and 8 take 3, 2, 19
// and 21% longer than 4 (registers against latency).  Eight wavefronts per
// SIMD instead of six are no faster.
constexpr int kGT = 8;            // tile of columns per block side
constexpr int kGSlots = 16;       // ray slots per view of the broadcast set-up
constexpr int kGViews = 64 / kGSlots;
constexpr int kGMaxRows = 8;      // rows within one voxel of a slice, at most
// Slices per chunk from which the gather along z is the faster one: it takes
// 5.6 ms for a chunk of 16 to 64 slices of the size above, k_cone_gather 4.65
// ms for 16 and 0.29 ms more per slice.  Small volumes, with fewer blocks than
// CUs, gain as well: 20 slices of 16^2, 48^2 and 128^2 at 180 views 0.61, 0.55 and
// 0.60 -> 0.32 ms (16^2 to 192^2 by 20 to 64 slices: 1.3 to 2.7 times).
constexpr int kGMinSlices = 20;
constexpr int kGBatch = 4;         // rays whose rows are loaded together
constexpr int kGStride = 64;      // doubles per column in LDS
constexpr float kGGrid = 262144.f;
constexpr double kGMaxStep = 30.0;  // voxels between rows at most, for the exact sums

constexpr int kGSum = kGT * kGT * kGStride;  // doubles per volume in LDS

struct GatherView {
    int v;
    float ct, st;
    int pad;
};

// The views in the order of their axis' angle to the x axis: those with x-major
// rays are the first nx_views of them, those with y-major rays the last
// ny_views.
struct GatherPlan {
    int JP, padlo;  // padded rows per bin, rows before row 0
    int nx_views, ny_views;
    const GatherView *views;  // [V]
};

// a * b, and zero where either is zero (also for a non-finite other factor)
__device__ __forceinline__ float mul_zero(float a, float b)
{
    float r;
    asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

typedef float c4f __attribute__((ext_vector_type(4)));
typedef float c3a4 __attribute__((ext_vector_type(3), aligned(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));

template <int NE>
__global__ __launch_bounds__(kGT * 64, NE == 1 ? 6 : 4) void k_cone_gather_z(ConeDev g, GatherPlan gp,
                                                            const ConeTab *__restrict__ tab,
                                                            const float *__restrict__ yl, int zper,
                                                            float *__restrict__ vol0,
                                                            float *__restrict__ vol1)
{
    __shared__ double sum[NE][kGSum];
    __shared__ c4f bcast[kGT][2][64];
    const unsigned item = xcd_order(block_linear(), grid_blocks());
    const int x0 = (int)(item % gridDim.x) * kGT;
    const int y0 = (int)(item / gridDim.x % gridDim.y) * kGT;
    const int z0 = (int)(item / (gridDim.x * gridDim.y)) * zper;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nzc = min(zper, g.nz - z0);
    // slices relative to the chunk's middle (lanes past its end repeat the last slice)
    const double zc = z0 + (zper >> 1);
    const float dz = (float)(min(lane, nzc - 1) - (zper >> 1));
    const float vox = (float)g.voxel, R = (float)g.sod, D = (float)g.sdd;
    const float dbin = (float)(g.sdd / g.bin), bc = (float)((g.B - 1) / 2.0 - g.off / g.bin);
    const float margin = 0.02f + 1e-5f * (float)g.B;
    const double cz = (g.nz - 1) / 2.0, jc = (g.J - 1) / 2.0;
    const int slot = lane % kGSlots;
    // column (x0 + a, y0 + b) of the tile is entry a * 8 + b of `sum`
    auto phase = [&](const int cls) {
        const int cstride = (cls ? kGT : 1) * kGStride;
        double *const mine = &sum[0][(cls ? wid : wid * kGT) * kGStride + lane];
        // the sum of a line code's column (16 codes per view); columns of a neighbour tile
        // have none
        auto load = [&](int line, double (&v)[NE]) {
            const int c = line & 15;
            if (c < kGT)
#pragma unroll
                for (int e = 0; e < NE; ++e) v[e] = mine[c * cstride + e * kGSum];
        };
        auto store = [&](int line, const double (&v)[NE], const float (&add)[NE]) {
            const int c = line & 15;
            if (c < kGT)
#pragma unroll
                for (int e = 0; e < NE; ++e) mine[c * cstride + e * kGSum] = v[e] + (double)add[e];
        };
        const int pl = (cls ? y0 : x0) + wid, c0 = cls ? x0 : y0;
        const int npl = cls ? g.ny : g.nx, nq = cls ? g.nx : g.ny;
        const int nv = cls ? gp.ny_views : gp.nx_views;
        const GatherView *views = gp.views + (cls ? g.V - nv : 0);
        if (pl >= npl || nv == 0) return;
        const float pp = (pl - (npl - 1) * 0.5f) * vox;
        const float q1 = (c0 - 1 - (nq - 1) * 0.5f) * vox, q2 = q1 + (kGT + 1) * vox;
        GatherView vw = views[min(lane / kGSlots, nv - 1)];
        for (int v0 = 0; v0 < nv; v0 += kGViews) {
            // ---- one ray per lane: slot `slot` of view v0 + lane / kGSlots
            bool ok = v0 + lane / kGSlots < nv;
            const int v = vw.v;
            auto bin_of = [&](float qq) {
                const float rx = (cls ? qq : pp) - R * vw.ct, ry = (cls ? pp : qq) - R * vw.st;
                return (rx * vw.st - ry * vw.ct) * __builtin_amdgcn_rcpf(rx * vw.ct + ry * vw.st) *
                           dbin + bc;
            };
            // the bins whose rays cross the plane between the lines c0 - 1 and c0 + 8
            // (bounds only; the exact test below decides), in the order of their line
            const float b1 = bin_of(q1), b2 = bin_of(q2), lim = (float)g.B;
            const int bl = max(0, (int)ceilf(fminf(fmaxf(fminf(b1, b2) - margin, -1.f), lim)));
            const int bh = min(g.B - 1,
                               (int)floorf(fminf(fmaxf(fmaxf(b1, b2) + margin, -1.f), lim)));
            const int b = b2 > b1 ? bl + slot : bh - slot;
            ok = ok && slot <= bh - bl;
            const unsigned vb = (unsigned)(v * g.B + (ok ? b : 0));
            const ConeTab t = tab[vb];
            vw = views[min(v0 + kGViews + lane / kGSlots, nv - 1)];
            const int64_t q = t.a + t.k * pl;
            const int hq = (int)(q >> 32);
            const float w = (float)(uint32_t)q * kTwoM32c;
            ok = ok && t.xmaj == (cls == 0) && hq >= c0 - 1 && hq <= min(c0 + kGT, nq) - 1;
            // the line relative to the tile's, plus 16 per view of the group
            const int h = hq - c0 + (lane / kGSlots) * 16;
            const double sb = fma(t.g1, (double)pl, t.g0) * g.row;  // height step per row (> 0)
            const double sbg = rint(sb * kGGrid);
            const float sbh = (float)sbg * (1.f / kGGrid), sbf = (float)sb;
            const float isb = __builtin_amdgcn_rcpf(sbf);
            // a row near the chunk's middle; heights are taken relative to it
            const double dq0 = (cz - zc) - jc * sb;  // height of row 0 over it
            const float jm = floorf(-(float)dq0 * isb);
            const double qcs = fma((double)jm, sb, dq0) * kGGrid, qcg = rint(qcs);
            const float qc = (float)qcg * (1.f / kGGrid);
            const h2 rest = {(_Float16)(float)(sb * kGGrid - sbg), (_Float16)(float)(qcs - qcg)};
            const float first = 1.f - (qc + 1.f) * isb;
            const unsigned row =
                (vb * (unsigned)gp.JP + (unsigned)(gp.padlo + (ok ? (int)jm : 0))) * (4u * NE);

            uint64_t rem = __ballot(ok);
            if (!rem) continue;
            const uint64_t close = __ballot(sbf < 1.f), closer = __ballot(sbf < 2.f / 3.f + 1e-6f);
            wave_order();  // the rays of the views before have been read
            if (ok) {
                bcast[wid][0][lane] =
                    c4f{first, qc, __builtin_bit_cast(float, rest), __uint_as_float(row)};
                bcast[wid][1][lane] = c4f{isb, sbh, sbf, w};
            }
            wave_order();
            // rays in the order of view and line, kGBatch at a time (past the last one the
            // last is repeated, and not taken): their rows are loaded together
            int pos = __builtin_amdgcn_readlane(h, __builtin_ctzll(rem));
            float cur[NE], nxt[NE];  // the window: columns pos, pos + 1 of the view
            double s0[NE] = {}, s1[NE] = {};  // and their sums over the views before it
#pragma unroll
            for (int e = 0; e < NE; ++e) cur[e] = nxt[e] = 0.f;
            load(pos, s0);
            load(pos + 1, s1);
            while (rem) {
                float y[kGBatch][3][NE];  // the first rows within one voxel of the slice
                float t[kGBatch], sf[kGBatch];  // the first one's height over it, the step
                unsigned off[kGBatch];
                int at[kGBatch];
                uint64_t left = rem;
#pragma unroll
                for (int k = 0; k < kGBatch; ++k) {
                    at[k] = left ? __builtin_ctzll(left) : at[k > 0 ? k - 1 : 0];
                    left &= left - 1;
                }
                float ws[kGBatch];
                c4f cst[kGBatch], csu[kGBatch];
#pragma unroll
                for (int k = 0; k < kGBatch; ++k) {
                    cst[k] = bcast[wid][0][at[k]];
                    csu[k] = bcast[wid][1][at[k]];
                }
#pragma unroll
                for (int k = 0; k < kGBatch; ++k) {
                    sf[k] = csu[k].z;
                    ws[k] = csu[k].w;
                    const float dj = floorf(fmaf(dz, csu[k].x, cst[k].x));
                    off[k] = ((unsigned)(int)dj) * (4u * NE) + __float_as_uint(cst[k].w);
                    const float packed = cst[k].z;
                    const h2 rest = __builtin_bit_cast(h2, packed);
                    t[k] = fmaf(fmaf(dj, (float)rest.x, (float)rest.y), 1.f / kGGrid,
                                fmaf(dj, csu[k].y, -dz) + cst[k].y);
                    asm volatile("" : "+v"(t[k]));
                    const char *p = (const char *)yl + off[k];
                    if constexpr (NE == 1) {
                        const c3a4 r = *(const c3a4 *)p;
                        y[k][0][0] = r.x;
                        y[k][1][0] = r.y;
                        y[k][2][0] = r.z;
                    } else {
                        const c4a8 r = *(const c4a8 *)p;
                        const c2 d = *(const c2 *)(p + 16);
                        y[k][0][0] = r.x;
                        y[k][0][NE - 1] = r.y;
                        y[k][1][0] = r.z;
                        y[k][1][NE - 1] = r.w;
                        y[k][2][0] = d.x;
                        y[k][2][NE - 1] = d.y;
                    }
                }
#pragma unroll
                for (int k = 0; k < kGBatch; ++k) {
                    if (!rem) break;
                    rem &= rem - 1;
                    // a zero weight takes nothing, not even from a non-finite row
                    float u[NE];
                    auto weight = [](float tt) {
                        return __builtin_amdgcn_fmed3f(1.f - fabsf(tt), 0.f, 1.f);
                    };
                    const float w0 = weight(t[k]), w1 = weight(t[k] + sf[k]);
#pragma unroll
                    for (int e = 0; e < NE; ++e)
                        u[e] = mul_zero(w0, y[k][0][e]) + mul_zero(w1, y[k][1][e]);
                    if (close >> at[k] & 1) {  // rows closer than one voxel
                        const float w2 = weight(fmaf(2.f, sf[k], t[k]));
#pragma unroll
                        for (int e = 0; e < NE; ++e) u[e] += mul_zero(w2, y[k][2][e]);
                        if (closer >> at[k] & 1) {  // and than 2/3
                            const int rows =
                                __builtin_amdgcn_readfirstlane((int)ceilf(2.f / sf[k]));
                            for (int j = 3; j < rows; ++j) {
                                const float wr = weight(fmaf((float)j, sf[k], t[k]));
                                const unsigned at_j = off[k] + (unsigned)j * (4u * NE);
#pragma unroll
                                for (int e = 0; e < NE; ++e)
                                    u[e] += mul_zero(wr, *(const float *)((const char *)yl + (at_j + 4u * e)));
                            }
                        }
                    }
                    const int hs = __builtin_amdgcn_readlane(h, at[k]);
                    if (hs != pos) {  // the window moves on: its first column is complete
                        store(pos, s0, cur);
                        if (hs == pos + 1) {
#pragma unroll
                            for (int e = 0; e < NE; ++e) {
                                s0[e] = s1[e];
                                cur[e] = nxt[e];
                            }
                        } else {
                            store(pos + 1, s1, nxt);
                            load(hs, s0);
#pragma unroll
                            for (int e = 0; e < NE; ++e) cur[e] = 0.f;
                        }
                        load(hs + 1, s1);
#pragma unroll
                        for (int e = 0; e < NE; ++e) nxt[e] = 0.f;
                        pos = hs;
                    }
#pragma unroll
                    for (int e = 0; e < NE; ++e) {
                        cur[e] = fmaf(1.f - ws[k], u[e], cur[e]);
                        nxt[e] += mul_zero(ws[k], u[e]);
                    }
                }
            }
            store(pos, s0, cur);
            store(pos + 1, s1, nxt);
        }
    };

    for (int i = threadIdx.x; i < NE * kGSum; i += kGT * 64) (&sum[0][0])[i] = 0.0;
    __syncthreads();
    phase(0);
    __syncthreads();
    phase(1);
    __syncthreads();
    for (int i = threadIdx.x; i < kGT * kGT * nzc; i += kGT * 64) {
        const int a = i % kGT, b = i / kGT % kGT, z = i / (kGT * kGT);
        const int x = x0 + a, y = y0 + b;
        if (x < g.nx && y < g.ny) {
            const size_t o = ((size_t)(z0 + z) * g.ny + y) * g.nx + x;
#pragma unroll
            for (int e = 0; e < NE; ++e)
                (e ? vol1 : vol0)[o] = (float)sum[e][(a * kGT + b) * kGStride + z];
        }
    }
}

struct ConeWork {
    DevBuf vx, vy, cs, yl, tab;
    DevBuf rows, views;           // of the gather along z
    std::vector<double> cs_host;  // what cs holds
    std::vector<double> tilt;     // angle to the x axis of the views in `views` (ascending)
};

std::mutex g_cone_mu;
std::vector<std::pair<std::pair<int, hipStream_t>, std::unique_ptr<ConeWork>>> g_cone_ws;

ConeWork *cone_workspace(hipStream_t s)
{
    int dev = 0;
    (void)hipGetDevice(&dev);
    for (auto &p : g_cone_ws)
        if (p.first.first == dev && p.first.second == s) return p.second.get();
    g_cone_ws.emplace_back(std::make_pair(dev, s), std::make_unique<ConeWork>());
    return g_cone_ws.back().second.get();
}

dect_status cone_setup(const dect_cone_geometry *g, ConeDev &d, ConeWork *w, hipStream_t s)
{
    if (!g) return fail(DECT_ERR_INVALID_ARG, "cone geometry is NULL");
    if (g->nx <= 0 || g->ny <= 0 || g->nz <= 0 || g->n_views <= 0 || g->n_bins <= 0 ||
        g->n_rows <= 0)
        return fail(DECT_ERR_INVALID_ARG, "cone geometry sizes must be positive");
    if (g->nx > 4096 || g->ny > 4096 || g->nz > 4096 || g->n_bins > 16384 || g->n_rows > 16384 ||
        g->n_views > 65536)
        return fail(DECT_ERR_INVALID_ARG, "cone geometry sizes exceed the supported maximum");
    if (!(g->voxel_mm > 0.0) || !(g->bin_mm > 0.0) || !(g->row_mm > 0.0) ||
        !std::isfinite(g->det_offset_mm))
        return fail(DECT_ERR_INVALID_ARG, "voxel, bin and row sizes must be positive");
    const double hx = 0.5 * g->nx * g->voxel_mm, hy = 0.5 * g->ny * g->voxel_mm;
    if (!(g->sod_mm > std::sqrt(hx * hx + hy * hy)) || !std::isfinite(g->sod_mm))
        return fail(DECT_ERR_GEOMETRY, "source orbit (SOD) must lie outside the volume");
    if (!(g->sdd_mm > g->sod_mm) || !std::isfinite(g->sdd_mm))
        return fail(DECT_ERR_GEOMETRY, "SDD must exceed SOD");
    const double hu = 0.5 * g->n_bins * g->bin_mm + std::fabs(g->det_offset_mm);
    const double hv = 0.5 * g->n_rows * g->row_mm;
    if (!(std::atan(hu / g->sdd_mm) < 0.25 * M_PI))
        return fail(DECT_ERR_GEOMETRY, "fan angle must be below 90 degrees");
    // the height never becomes the driving axis: |dz| < |d_in-plane| on every ray
    if (!(hv < 0.5 * g->sdd_mm))
        return fail(DECT_ERR_GEOMETRY, "cone half-angle must be below atan(1/2)");
    std::vector<double> cs(2 * (size_t)g->n_views);
    for (int v = 0; v < g->n_views; ++v) {
        const double th = g->angles_rad ? g->angles_rad[v] : 2.0 * M_PI * v / g->n_views;
        if (!std::isfinite(th)) return fail(DECT_ERR_INVALID_ARG, "view angles must be finite");
        cs[2 * v] = std::cos(th);
        cs[2 * v + 1] = std::sin(th);
    }
    if (cs != w->cs_host) {
        // kernels in flight on this stream may still read the old table
        DECT_HIP(hipStreamSynchronize(s));
        dect_status st = w->cs.ensure(cs.size() * 8);
        if (st) return st;
        DECT_HIP(hipMemcpy(w->cs.ptr, cs.data(), cs.size() * 8, hipMemcpyHostToDevice));
        w->cs_host = cs;
        w->tilt.clear();
    }
    d = ConeDev{g->nx, g->ny, g->nz, g->n_views, g->n_rows, g->n_bins, g->voxel_mm, g->bin_mm,
                g->row_mm, g->det_offset_mm, g->sod_mm, g->sdd_mm, (const double *)w->cs.ptr};
    return DECT_OK;
}

// The padded rows k_cone_gather_z needs, or false where its limits do not
// hold (the gather along x then takes the call): at most kGMaxRows rows
// within one voxel of a slice, at most kGSlots rays of a view across nine
// lines, and a padded copy of at most about 8 times the projections and of
// less than 4 GiB (32-bit byte offsets), and rows at most kGMaxStep voxels apart.
// Bounds over the points within one voxel of
// the volume: the fraction of the way from the source's plane to the panel's
// is at least tmin there.
bool gather_plan(const ConeDev &d, int ne, GatherPlan &gp)
{
    const double rx = 0.5 * d.nx * d.voxel + d.voxel, ry = 0.5 * d.ny * d.voxel + d.voxel;
    const double r = std::sqrt(rx * rx + ry * ry);
    const double tmin = (d.sod - r) / d.sdd;
    if (!(tmin > 0.0)) return false;
    const double sb = d.row / d.voxel * tmin * (1.0 - 1e-6);
    const double slope = std::sqrt(1.0 + r * r / (d.sod * d.sod - r * r));
    const double margin = 0.02 + 1e-5 * d.B;
    if (std::ceil(2.0 / sb) > kGMaxRows || d.row / d.voxel * (d.sod + r) / d.sdd > kGMaxStep ||
        (kGT + 1) * d.voxel / (d.bin * tmin) * slope + 2.0 * margin + 1.0 > kGSlots)
        return false;
    // rows from the first one of slice 0 to the last one of slice nz - 1
    const double jc = 0.5 * (d.J - 1), reach = (0.5 * (d.nz - 1) + 1.0) / sb + 2.0;
    const int lo = std::max(0, (int)std::ceil(reach - jc) + 1);
    const int hi = std::max(0, (int)std::ceil(jc + reach) + kGMaxRows - (d.J - 1));
    const double jp = (double)d.J + lo + hi;
    if (jp * d.V * d.B * 4.0 * ne >= 4294967296.0 || jp > 8.0 * d.J + 64.0) return false;
    gp.JP = d.J + lo + hi;
    gp.padlo = lo;
    return true;
}

bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone;
}

// The buffers of the gather along z, or false where they cannot be had: under a
// caller's workspace (sized for the buffers of k_cone_gather, which are
// smaller), out of memory, or in a capture that no call has prepared.  The
// call then takes k_cone_gather.
bool gather_buffers(const ConeDev &d, int ne, ConeWork *w, GatherPlan &gp, hipStream_t s)
{
    if (caller_workspace()) return false;
    const size_t need = (size_t)d.V * d.B * gp.JP * 4 * ne;
    if ((w->rows.bytes < need || w->tilt.empty()) && capturing(s)) return false;
    if (w->rows.bytes < need || w->views.bytes < d.V * sizeof(GatherView)) {
        if (hipStreamSynchronize(s) != hipSuccess || w->rows.ensure(need) ||
            w->views.ensure(d.V * sizeof(GatherView))) {
            (void)hipGetLastError();
            set_error("");  // the call goes on without them
            return false;
        }
        w->tilt.clear();
    }
    const std::vector<double> &cs = w->cs_host;
    auto angle = [&](int v) { return std::atan2(std::fabs(cs[2 * v + 1]), std::fabs(cs[2 * v])); };
    if (w->tilt.empty()) {
        std::vector<int> order(d.V);
        for (int v = 0; v < d.V; ++v) order[v] = v;
        std::stable_sort(order.begin(), order.end(),
                         [&](int a, int b) { return angle(a) < angle(b); });
        std::vector<GatherView> views(d.V);
        std::vector<double> tilt(d.V);
        for (int i = 0; i < d.V; ++i) {
            const int v = order[i];
            views[i] = GatherView{v, (float)cs[2 * v], (float)cs[2 * v + 1], 0};
            tilt[i] = angle(v);
        }
        // kernels in flight on this stream may still read the old list
        if (hipStreamSynchronize(s) != hipSuccess ||
            hipMemcpy(w->views.ptr, views.data(), views.size() * sizeof(GatherView),
                      hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        w->tilt = tilt;
    }
    // a ray is within the half fan angle of its view's axis, and x-major within 45 degrees
    // of the x axis
    const double fan = std::atan((0.5 * d.B * d.bin + std::fabs(d.off)) / d.sdd) + 1e-6;
    const auto b = w->tilt.begin(), e = w->tilt.end();
    gp.nx_views = (int)(std::upper_bound(b, e, 0.25 * M_PI + fan) - b);
    gp.ny_views = (int)(e - std::lower_bound(b, e, 0.25 * M_PI - fan));
    gp.views = (const GatherView *)w->views.ptr;
    return true;
}

// Both projectors for NE volumes (1 or 2) sharing one geometry.
// lo: NULL, or NE buffers for the rounding errors of the FP32 results.
template <int NE>
dect_status cone_project_n(const dect_cone_geometry *g, const float *const *vol,
                           float *const *proj, float *const *lo, hipStream_t s)
{
    for (int e = 0; e < NE; ++e)
        if (!vol[e] || !proj[e]) return fail(DECT_ERR_INVALID_ARG, "dect_cone_project: null buffer");
    std::lock_guard<std::mutex> lk(g_cone_mu);
    ConeWork *w = cone_workspace(s);
    ConeDev d;
    dect_status st = cone_setup(g, d, w, s);
    if (st) return st;
    const int chunks = (d.J + 63) / 64, rper = (d.J + chunks - 1) / chunks;
    const size_t copy = (size_t)(d.nx + 2 * kCPad) * (d.ny + 2 * kCPad) * (d.nz + 2 * kCPad);
    const size_t need = copy * 4 * NE;  // of k_cone_fwd_z
    const size_t pz = d.nz + 2 * kCPad;
    const size_t nxb = (size_t)d.nx * pz * (d.ny + 2 * kCPad) * 4;  // of k_cone_fwd, per volume
    const size_t nyb = (size_t)d.ny * pz * (d.nx + 2 * kCPad) * 4;
    const bool by_line = NE == 1 && d.nz <= kFZSlices;
    // (a caller's workspace was sized for the two copies of k_cone_fwd and keeps them)
    const bool can_z = need < (size_t(1) << 32) && !caller_workspace();
    bool along_rows = can_z && rper >= (by_line ? kFZMinRowsLine : kFZMinRows);
    const bool have_z = can_z && w->vx.bytes >= need;
    const bool have_xy = w->vx.bytes >= nxb * NE && w->vy.bytes >= nyb * NE;
    // a capture that a call of other rows has prepared takes that call's buffers
    if (!(along_rows ? have_z : have_xy) && (along_rows ? have_xy : have_z) && capturing(s))
        along_rows = !along_rows;
    if (along_rows) {
        const size_t px = d.nx + 2 * kCPad, py = d.ny + 2 * kCPad, pzn = d.nz + 2 * kCPad;
        if (w->vx.bytes < need) {
            DECT_HIP(hipStreamSynchronize(s));
            if ((st = w->vx.ensure(need))) return st;
        }
        hipLaunchKernelGGL(k_cone_pad_z<NE>,
                           dim3((unsigned)((px + 31) / 32), (unsigned)((pzn + 31) / 32),
                                (unsigned)py),
                           dim3(256), 0, s, vol[0], vol[NE - 1], d.nx, d.ny, d.nz,
                           (float *)w->vx.ptr);
        DECT_HIP(hipGetLastError());
        hipLaunchKernelGGL((by_line ? k_cone_fwd_z<NE, NE == 1> : k_cone_fwd_z<NE, false>),
                           dim3((unsigned)((d.B + kFZWaves - 1) / kFZWaves), (unsigned)d.V,
                                (unsigned)chunks),
                           dim3(kFZWaves * 64), 0, s, d, (const float *)w->vx.ptr, rper, proj[0],
                           proj[NE - 1], lo ? lo[0] : (float *)nullptr,
                           lo ? lo[NE - 1] : (float *)nullptr);
        DECT_HIP(hipGetLastError());
        return DECT_OK;
    }
    if (w->vx.bytes < nxb * NE || w->vy.bytes < nyb * NE) {
        DECT_HIP(hipStreamSynchronize(s));
        if ((st = w->vx.ensure(nxb * NE)) || (st = w->vy.ensure(nyb * NE))) return st;
    }
    hipLaunchKernelGGL(k_cone_pad_x<NE>,
                       dim3((unsigned)((d.nx + 31) / 32), (unsigned)((d.ny + 2 * kCPad + 31) / 32),
                            (unsigned)pz),
                       dim3(256), 0, s, vol[0], vol[NE - 1], d.nx, d.ny, d.nz, (float *)w->vx.ptr);
    hipLaunchKernelGGL(k_cone_pad_y<NE>, dim3((unsigned)((nyb / 4 + 255) / 256)), dim3(256), 0, s,
                       vol[0], vol[NE - 1], d.nx, d.ny, d.nz, (float *)w->vy.ptr);
    DECT_HIP(hipGetLastError());
    const size_t nray = (size_t)d.V * d.J * d.B;
    hipLaunchKernelGGL(k_cone_fwd<NE>, dim3((unsigned)((nray + 255) / 256)), dim3(256), 0, s, d,
                       (const float *)w->vx.ptr, (const float *)w->vy.ptr, proj[0], proj[NE - 1],
                       lo ? lo[0] : (float *)nullptr, lo ? lo[NE - 1] : (float *)nullptr);
    DECT_HIP(hipGetLastError());
    return DECT_OK;
}

template <int NE>
dect_status cone_backproject_n(const dect_cone_geometry *g, const float *const *proj,
                               float *const *vol, hipStream_t s)
{
    for (int e = 0; e < NE; ++e)
        if (!vol[e] || !proj[e])
            return fail(DECT_ERR_INVALID_ARG, "dect_cone_backproject: null buffer");
    std::lock_guard<std::mutex> lk(g_cone_mu);
    ConeWork *w = cone_workspace(s);
    ConeDev d;
    dect_status st = cone_setup(g, d, w, s);
    if (st) return st;
    const size_t ntab = (size_t)d.V * d.B;
    const int chunks = (d.nz + 63) / 64, zper = (d.nz + chunks - 1) / chunks;
    GatherPlan gp{};
    const bool along_z =
        zper >= kGMinSlices && gather_plan(d, NE, gp) && gather_buffers(d, NE, w, gp, s);
    const size_t nray = ntab * d.J;
    // the gather along z scales into `rows`, the other into `yl`, or into `rows` too where
    // those are there (of a call along z that prepared a capture)
    DevBuf &scaled =
        along_z || (w->yl.bytes < nray * 4 * NE && w->rows.bytes >= nray * 4 * NE) ? w->rows : w->yl;
    if (scaled.bytes < nray * 4 * NE || w->tab.bytes < ntab * sizeof(ConeTab)) {
        DECT_HIP(hipStreamSynchronize(s));
        if ((st = scaled.ensure(nray * 4 * NE)) || (st = w->tab.ensure(ntab * sizeof(ConeTab))))
            return st;
    }
    hipLaunchKernelGGL(k_cone_tab, dim3((unsigned)((ntab + 255) / 256)), dim3(256), 0, s, d,
                       (ConeTab *)w->tab.ptr);
    DECT_HIP(hipGetLastError());
    if (along_z) {
        hipLaunchKernelGGL(k_cone_scale_z<NE>,
                           dim3((unsigned)((d.B + 31) / 32), (unsigned)((gp.JP + 31) / 32),
                                (unsigned)d.V),
                           dim3(256), 0, s, d, proj[0], proj[NE - 1], gp.JP, gp.padlo,
                           (float *)w->rows.ptr);
        hipLaunchKernelGGL(k_cone_gather_z<NE>,
                           dim3((unsigned)((d.nx + kGT - 1) / kGT),
                                (unsigned)((d.ny + kGT - 1) / kGT), (unsigned)chunks),
                           dim3(kGT * 64), 0, s, d, gp, (const ConeTab *)w->tab.ptr,
                           (const float *)w->rows.ptr, zper, vol[0], vol[NE - 1]);
        DECT_HIP(hipGetLastError());
        return DECT_OK;
    }
    hipLaunchKernelGGL(k_cone_scale<NE>, dim3((unsigned)((nray + 255) / 256)), dim3(256), 0, s, d,
                       proj[0], proj[NE - 1], (float *)scaled.ptr);
    DECT_HIP(hipGetLastError());
    const int nzc = (d.nz + kZC - 1) / kZC;
    hipLaunchKernelGGL(k_cone_gather<NE>, dim3((unsigned)((d.nx + 63) / 64), (unsigned)d.ny,
                                               (unsigned)((nzc + 3) / 4)),
                       dim3(256), 0, s, d, (const ConeTab *)w->tab.ptr, (const float *)scaled.ptr,
                       vol[0], vol[NE - 1]);
    DECT_HIP(hipGetLastError());
    return DECT_OK;
}

}  // namespace

dect_status cone_project(const dect_cone_geometry *g, const float *vol, float *proj,
                         hipStream_t s)
{
    return cone_project_n<1>(g, &vol, &proj, nullptr, s);
}

dect_status cone_backproject(const dect_cone_geometry *g, const float *proj, float *vol,
                             hipStream_t s)
{
    return cone_backproject_n<1>(g, &proj, &vol, s);
}

dect_status cone_project2(const dect_cone_geometry *g, const float *const vol[2],
                          float *const proj[2], hipStream_t s)
{
    return cone_project_n<2>(g, vol, proj, nullptr, s);
}

dect_status cone_project2_lo(const dect_cone_geometry *g, const float *const vol[2],
                             float *const proj[2], float *const lo[2], hipStream_t s)
{
    return cone_project_n<2>(g, vol, proj, lo, s);
}

dect_status cone_backproject2(const dect_cone_geometry *g, const float *const proj[2],
                              float *const vol[2], hipStream_t s)
{
    return cone_backproject_n<2>(g, proj, vol, s);
}

void release_cone_work()
{
    std::lock_guard<std::mutex> lk(g_cone_mu);
    g_cone_ws.clear();
}

}  // namespace dect
