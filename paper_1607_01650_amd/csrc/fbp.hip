// Fan-beam filtered back-projection on gfx950: the analytic reconstruction
// the paper compares its method with (Sec. 3), for the flat detector over a
// full turn of equally spaced views, in the textbook form for equally spaced
// collinear detectors:
//   k_fbp_filter : the views are weighted by R / sqrt(R^2 + s_b^2) (s_b the
//                  bin position scaled to a virtual detector through the
//                  isocentre, spacing ds = du R / D), convolved with the
//                  band-limited ramp kernel of spacing ds and halved (a full
//                  turn sees every line twice).  Output: each pair's filtered
//                  views, interleaved and zero-padded by kQPad bins per side.
//   k_fbp_bp_win, k_fbp_bp : per pixel of a pair, all views: the filtered
//                  views at the virtual-detector position where the ray from
//                  the source through the pixel meets it (linear
//                  interpolation between both images' taps), weighted by
//                  R^2 / (R - p . e_s)^2, times 2 pi / V.
// All are gathers with no atomics.
#include <cmath>
#include <mutex>
#include <vector>

#include "common.h"
#include "proj_device.h"
#include "reduce.h"
#include "xcd.h"

namespace dect {
namespace {

constexpr int kQPad = 2;           // zero bins on each side of a filtered view
// Bins, at most: the entry point's range (the direct sums grow with the square of the
// bins; no buffer depends on it).
constexpr int kFbpMaxBins = 6144;

// The ramp's nonzero taps off the centre have odd distances, so the even bins
// are filtered from the odd ones and the odd bins from the even ones: two
// Toeplitz products per row, [rows] x [B / 2] x [B / 2], which run on the
// matrix cores in FP64 (the sums' precision).  grid (64-bin chunks, groups of
// 8 views, pairs): the 16 rows of a block are 8 views of both images; wavefront
// w forms the 16 outputs 2 (m0 + n) + (w & 1), m0 the chunk's first half bin
// plus 16 (w >> 1).  The weighted rows are staged kFKc bins at a time, the two
// parities apart (row stride 4 mod 64 dwords: a fragment's 16 rows x 4 bins
// lie in distinct banks), with the taps 1 / (pi^2 k^2), k odd, between them and
// the chunk's outputs.
// 720 rows x 736 bins (390 MFLOP): 17.5 us traced, 55 for the direct sums on
// the vector units (bound by their FP64 conversions and adds); the matrix
// cores are busy for 5 us of it, the rest is the staging of 16 rows per block
// and the launch.  Staging 768 bins at a time measured the same to 5% slower.
constexpr int kFKc = 512;
constexpr int kFTaps = 32 + kFKc / 2;  // taps between a chunk's outputs and the staged bins
constexpr int kFRow = kFKc / 2 + 4;
typedef double d4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float fbp_weight(int b, float r_sod, float u_to_s, float u0, float du_v)
{
    // virtual-detector position s_b = u_b R / D, weight R / sqrt(R^2 + s_b^2)
    const float s = (u0 + b * du_v) * u_to_s;
    return r_sod * rsqrtf(fmaf(s, s, r_sod * r_sod));
}

__global__ __launch_bounds__(256) void k_fbp_filter(const float *__restrict__ sino, int batch,
                                                    int V, int B, float r_sod, float u_to_s,
                                                    float u0, float du_v, float inv2ds,
                                                    f2v *__restrict__ q)
{
    __shared__ double tap[2][kFTaps];     // [parity of the output][half-bin distance]
    __shared__ float rows[2][16][kFRow];  // [parity][2 view + image][half bin]
    const int v0 = blockIdx.y * 8, pr = blockIdx.z, e0 = 2 * pr;
    const size_t M = (size_t)V * B;
    const double kPi2 = 9.869604401089358;  // pi^2
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int par = wid & 1, m0 = blockIdx.x * 32 + (wid >> 1) * 16;
    const int n = lane & 15, kk = lane >> 4;
    d4v acc = {0.0, 0.0, 0.0, 0.0};
    for (int b0 = 0; b0 < B; b0 += kFKc) {
        __syncthreads();
        float t[kFKc / 256][16];
#pragma unroll
        for (int i = 0; i < kFKc / 256; ++i)  // unconditional loads, all in flight
#pragma unroll
            for (int r = 0; r < 16; ++r)
                t[i][r] = sino[(size_t)min(e0 + (r & 1), batch - 1) * M +
                               (size_t)min(v0 + (r >> 1), V - 1) * B +
                               min(b0 + 256 * i + (int)threadIdx.x, B - 1)];
        // tap i: half bin j = b0 / 2 + kFKc / 2 - 1 - k seen from output m = 32 x + l, i = k + l;
        // their distance 2 (m - j) + 1 (odd outputs) or 2 (m - j) - 1
        for (int i = threadIdx.x; i < 2 * kFTaps; i += 256) {
            const int p = i >= kFTaps, o = i - p * kFTaps;
            const int d = (int)blockIdx.x * 32 - b0 / 2 - (kFKc / 2 - 1) + o;
            const double k = 2.0 * d + (p ? 1.0 : -1.0);
            tap[p][o] = 1.0 / (kPi2 * k * k);
        }
#pragma unroll
        for (int i = 0; i < kFKc / 256; ++i) {
            const int o = 256 * i + threadIdx.x, b = b0 + o;
            const float w = fbp_weight(b, r_sod, u_to_s, u0, du_v);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool in = b < B && v0 + (r >> 1) < V && e0 + (r & 1) < batch;
                rows[o & 1][r][o >> 1] = in ? w * t[i][r] : 0.f;
            }
        }
        __syncthreads();
        const int half = (min(kFKc, B - b0 + 1) / 2 + 15) & ~15;  // half bins (zeros past the row)
        const float *a = &rows[1 - par][n][kk];
        const double *h = &tap[par][m0 - (int)blockIdx.x * 32 + n + kFKc / 2 - 1 - kk];
        for (int j = 0; j < half; j += 16) {  // four steps' operands in flight
            double x[4], t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = (double)a[j + 4 * u];
                t[u] = h[-(j + 4 * u)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u], t[u], acc, 0, 0, 0);
        }
    }
    const int stride = B + 2 * kQPad;
    const int c = 2 * (m0 + n) + par;
#pragma unroll
    for (int r = 0; r < 4; ++r) {  // row 4 r + kk of the product, column n
        const int row = 4 * r + kk, v = v0 + (row >> 1), e = e0 + (row & 1);
        if (c < B && v < V) {
            float o = 0.f;
            if (e < batch) {
                const float p = fbp_weight(c, r_sod, u_to_s, u0, du_v) *
                                sino[(size_t)e * M + (size_t)v * B + c];
                o = (float)((0.25 * (double)p - acc[r]) * (double)inv2ds);
            }
            ((float *)q)[(((size_t)pr * V + v) * stride + c + kQPad) * 2 + (row & 1)] = o;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < 8 * 2 * kQPad) {  // the zero bins of the 8 views
        const int v = v0 + threadIdx.x / (2 * kQPad), k = threadIdx.x % (2 * kQPad);
        if (v < V) q[((size_t)pr * V + v) * stride + (k < kQPad ? k : B + k)] = f2v(0.f);
    }
}

// The detector position of a tile's centre (xm, ym) at a view, in FP64: the bin
// it falls on, the position relative to that bin, and its derivative, so that
// the position of the pixel at (dx, dy) from the centre is off + (dx ax + dy
// ay) / (distance from the source along the axis) past the bin.  The centre is that of the tile's part
// of the image: a whole tile's may lie at the source, where it has no position.
struct TilePos {
    int bin;
    float off, ax, ay;
};

__device__ __forceinline__ TilePos tile_pos(const ViewInfo &vi, double xm, double ym, double sod,
                                            double sdd_over_du, double b0)
{
    const double ct = (double)vi.ct + (double)vi.ctl, st = (double)vi.st + (double)vi.stl;
    const double m = (ym * ct - xm * st) * sdd_over_du / (sod - (xm * ct + ym * st));
    const double fl = floor(m + b0);
    TilePos o;
    o.bin = (int)fmin(fmax(fl, -1e6), 1e6);
    o.off = (float)(m + b0 - fl);
    o.ax = (float)(m * ct - sdd_over_du * st);
    o.ay = (float)(m * st + sdd_over_du * ct);
    return o;
}

__device__ __forceinline__ float lane_f(float v, int i)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i));
}

// The general form, for tiles that may see more bins than a window of
// k_fbp_bp_win holds: one 16-byte load for both taps of both images per pixel
// and view, positions relative to the tile's centre as there.  512 x 512, 360
// views, 2048 bins of 0.85 mm: the call takes 142 us (428 us with the direct
// filter and the positions from the isocentre).  grid (tiles, pairs) of 16 x
// 16 pixels, XCD-ordered.  TILE false: positions from the isocentre, for orbits
// so close to the image that a tile may see half the detector (the rounding of
// a position is that of the bins it is the sum of).  A block has S wavefronts per
// 64 pixels, with an S-th of the views each, their sums added in FP64 in order:
// four where there are few tiles (a wavefront then waits for its taps, group by
// group, with nothing else on its SIMD), 360 views of 4 bins per pixel: 16^2 46
// -> 30 us, 64^2 61 -> 33, 256^2 101 -> 69; but 16 views at 384^2 26 -> 31, 360 at
// 1024^2 745 -> 830.
constexpr size_t kBpFew = 400;  // tiles, at most
template <bool TILE, int S>
__global__ __launch_bounds__(256 * S) void k_fbp_bp(const f2v *__restrict__ q,
                                                const ViewInfo *__restrict__ views, int batch,
                                                int nx, int ny, int V, int B, float pixel,
                                                double sod_d, double sdd_over_du, double b0,
                                                float scale, float *__restrict__ img)
{
    const float sod = (float)sod_d;
    const unsigned item = xcd_order(block_linear(), grid_blocks());
    const int ntx = (nx + 15) / 16, nty = (ny + 15) / 16;
    const int pr = (int)(item / (unsigned)(ntx * nty));
    const int tile = (int)(item % (unsigned)(ntx * nty));
    const int x0 = (tile % ntx) * 16, y0 = (tile / ntx) * 16;
    const int c = x0 + (threadIdx.x & 15), r = y0 + (threadIdx.x >> 4 & 15);
    const int lane = threadIdx.x & 63;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    // the tile's part of the image: lanes past it repeat its last column and row
    const int cl = min(c, nx - 1), rl = min(r, ny - 1);
    const float hx = 0.5f * (min(16, nx - x0) - 1), hy = 0.5f * (min(16, ny - y0) - 1);
    const float x = (cl - 0.5f * (nx - 1)) * pixel, y = (rl - 0.5f * (ny - 1)) * pixel;
    const float dx = (cl - x0 - hx) * pixel, dy = (rl - y0 - hy) * pixel;
    const double xm = (x0 + hx - 0.5 * (nx - 1)) * pixel, ym = (y0 + hy - 0.5 * (ny - 1)) * pixel;
    const int stride = B + 2 * kQPad;
    const char *base = (const char *)(q + (size_t)pr * V * stride);
    // n views from v (lane u of tp): their taps' loads first, then the sums
    auto group = [&](auto n_tag, int v, const TilePos &tp, int u, float &s0, float &s1) {
        constexpr int n = decltype(n_tag)::value;
        f4a8 t[n];
        float w[n], g[n];
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const ViewInfo vi = views[v + k];
            const float inv = __builtin_amdgcn_rcpf(sod - fmaf(x, vi.ct, y * vi.st));
            float bf;
            if constexpr (TILE)
                bf = fmaf(fmaf(dy, lane_f(tp.ay, u + k), dx * lane_f(tp.ax, u + k)), inv,
                          lane_f(tp.off, u + k));
            else
                bf = fmaf(fmaf(-x, vi.st, y * vi.ct) * inv, (float)sdd_over_du, (float)b0);
            const float fl = floorf(bf);
            // taps h, h + 1 of the padded row; beyond the detector both are zero
            const int o = TILE ? __builtin_amdgcn_readlane(tp.bin, u + k) : 0;
            const int h = min(max((int)fl + o, -kQPad), B);
            const char *rowp = base + (size_t)(v + k) * stride * 8;
            t[k] = *(const f4a8 *)(rowp + (unsigned)(h + kQPad) * 8u);
            w[k] = bf - fl;
            g[k] = inv * inv;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < n; ++k) {
            s0 = fmaf(g[k], fmaf(w[k], t[k].z - t[k].x, t[k].x), s0);
            s1 = fmaf(g[k], fmaf(w[k], t[k].w - t[k].y, t[k].y), s1);
        }
    };
    // groups of 8 views (their loads in flight together) summed in FP32,
    // the group sums in FP64
    double acc0 = 0.0, acc1 = 0.0;
    const int v_end = (int)((int64_t)V * (part + 1) / S);
    for (int vb = (int)((int64_t)V * part / S); vb < v_end; vb += 64) {
        // the tile's centre at 64 views, one per lane
        const TilePos tp =
            tile_pos(views[min(vb + lane, V - 1)], xm, ym, sod_d, sdd_over_du, b0);
        for (int v0 = vb; v0 < min(v_end, vb + 64); v0 += 8) {
            float s0 = 0.f, s1 = 0.f;
            if (v0 + 8 <= v_end)
                group(std::integral_constant<int, 8>{}, v0, tp, v0 - vb, s0, s1);
            else
                for (int v = v0; v < v_end; ++v)
                    group(std::integral_constant<int, 1>{}, v, tp, v - vb, s0, s1);
            acc0 += (double)s0;
            acc1 += (double)s1;
        }
    }
    if constexpr (S > 1) {
        __shared__ double sum[S][2][256];
        const int t = threadIdx.x & 255;
        sum[part][0][t] = acc0;
        sum[part][1][t] = acc1;
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int k = 1; k < S; ++k) {
            acc0 += sum[k][0][t];
            acc1 += sum[k][1][t];
        }
    }
    if (c >= nx || r >= ny) return;
    const size_t N = (size_t)nx * ny, i = (size_t)r * nx + c;
    const int e0 = 2 * pr;
    img[(size_t)e0 * N + i] = (float)(acc0 * (double)scale);
    if (e0 + 1 < batch) img[(size_t)(e0 + 1) * N + i] = (float)(acc1 * (double)scale);
}

// The back-projection with the views' samples in LDS: a block's tile of TX x
// 16 pixels sees at most 60 bins of a view (checked by the host), so a
// wavefront reads a 64-bin window of both images with one coalesced load per
// view and every pixel takes its taps from there.  The eight wavefronts of a
// block hold the same pixels, PX per lane, and an eighth of the views each, in
// groups of eight whose windows are loaded while the group before is walked.
// Sums: eight views in FP32, groups in FP64, the eighths in FP64 in wave order.
//
// Bound by VALU issue: 14 instructions per pixel and view plus 10 per window.
// k_fbp_bp's 16-byte load per pixel and view kept the L1 busy (0.94 accesses
// per cycle) beside 23 VALU instructions.  512 x 512, 360 views, both images: 48
// us traced (55 with k_fbp_bp), the call with its filter 104 -> 60 us; at 128 x
// 128, 90 views 18 -> 13 us.  The error of that 512 x 512 image against FP64 fell from
// 4.9e-6 to 7e-7.  Tiles of 32 columns (eight pixels per lane) where there are
// enough of them to fill the chip: the call took 67 against 72 us with 16 columns
// at that size when the rule was set; four wavefronts per block instead of eight
// 73 us.
constexpr int kBpWin = 64, kBpGroup = 8, kBpWaves = 8;
constexpr size_t kBpWide = 1024;  // 16 x 16 tiles from which tiles of 32 columns are taken

template <int TX>
__global__ __launch_bounds__(kBpWaves * 64) void k_fbp_bp_win(
    const f2v *__restrict__ q, const ViewInfo *__restrict__ views, int batch, int nx, int ny, int V,
    int B, float pixel, double sod_d, double sdd_over_du, double b0, float scale,
    float *__restrict__ img)
{
    constexpr int PX = TX / 4;  // rows of a lane; the lanes are TX columns x 64 / TX row groups
    __shared__ union {
        f2v win[kBpWaves][kBpGroup][kBpWin];
        double sum[kBpWaves][PX][64];
    } sh;
    const float sod = (float)sod_d;
    const unsigned item = xcd_order(block_linear(), grid_blocks());
    const int ntx = (nx + TX - 1) / TX, nty = (ny + 15) / 16;
    const int pr = (int)(item / (unsigned)(ntx * nty));
    const int tile = (int)(item % (unsigned)(ntx * nty));
    const int x0 = (tile % ntx) * TX, y0 = (tile / ntx) * 16;
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = x0 + lane % TX, r = y0 + lane / TX * PX;
    // a pixel's position (x, y), and from the centre of the tile's part of the image
    // (dx, dy; exact); lanes past that part repeat its last column and row
    const int cl = min(c, nx - 1);
    const float hx = 0.5f * (min(TX, nx - x0) - 1), hy = 0.5f * (min(16, ny - y0) - 1);
    const float x = (cl - 0.5f * (nx - 1)) * pixel, dx = (cl - x0 - hx) * pixel;
    float y[PX], dy[PX];
#pragma unroll
    for (int i = 0; i < PX; ++i) {
        const int rl = min(r + i, ny - 1);
        y[i] = (rl - 0.5f * (ny - 1)) * pixel;
        dy[i] = (rl - y0 - hy) * pixel;
    }
    const double xm = (x0 + hx - 0.5 * (nx - 1)) * pixel;
    const double ym = (y0 + hy - 0.5 * (ny - 1)) * pixel;
    const int stride = B + 2 * kQPad;
    const f2v *base = q + (size_t)pr * V * stride + kQPad;
    const int v_begin = V * wid / kBpWaves, v_end = V * (wid + 1) / kBpWaves;
    f2v(*win)[kBpWin] = sh.win[wid];
    double acc[PX][2] = {};
    // views v .. v + 63, one per lane; a window starts 31 bins before the tile centre's
    auto windows = [&](int v) {
        TilePos o = tile_pos(views[min(v + lane, V - 1)], xm, ym, sod_d, sdd_over_du, b0);
        o.bin -= kBpWin / 2 - 1;
        o.off += (float)(kBpWin / 2 - 1);
        return o;
    };
    f2v pre[kBpGroup];
    auto load = [&](int v, int fb, int k) {  // (bins off the detector read its zero bins)
#pragma unroll
        for (int u = 0; u < kBpGroup; ++u) {
            const int b = __builtin_amdgcn_readlane(fb, k + u) + lane;
            const f2v *row = base + (size_t)min(v + u, V - 1) * stride - 1;
            pre[u] = row[(unsigned)(min(max(b, -1), B) + 1)];
        }
    };
    TilePos nw = windows(v_begin);
    load(v_begin, nw.bin, 0);
    TilePos cw = nw;  // of the group being walked: lanes k ..
    for (int v = v_begin; v < v_end; v += kBpGroup) {
        const int k = (v - v_begin) & 63, kn = (k + kBpGroup) & 63;
        wave_order();  // the group before has been read
#pragma unroll
        for (int u = 0; u < kBpGroup; ++u) win[u][lane] = pre[u];
        wave_order();
        if (k == 0) cw = nw;
        if (v + kBpGroup < v_end) {
            if (kn == 0) nw = windows(v + kBpGroup);
            load(v + kBpGroup, nw.bin, kn);
        }
        float s[PX][2] = {};
        auto view = [&](int u) {
            const ViewInfo vi = views[v + u];
            const float off = lane_f(cw.off, k + u), ay = lane_f(cw.ay, k + u);
            const float ex = fmaf(-x, vi.ct, sod), px = dx * lane_f(cw.ax, k + u);
#pragma unroll
            for (int i0 = 0; i0 < PX; i0 += 4) {
                f2v t0[4], t1[4];
                float w[4], g[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // the distance, then the position in the window (1 .. 62)
                    const float inv = __builtin_amdgcn_rcpf(fmaf(-y[i0 + i], vi.st, ex));
                    const float bf = fmaf(fmaf(dy[i0 + i], ay, px), inv, off);
                    const unsigned h = (unsigned)bf;
                    w[i] = __builtin_amdgcn_fractf(bf);
                    g[i] = inv * inv;
                    t0[i] = win[u][h];
                    t1[i] = win[u][h + 1];
                }
                __builtin_amdgcn_sched_barrier(0);  // the four pixels' reads in flight together
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float(&si)[2] = s[i0 + i];
                    si[0] = fmaf(g[i], fmaf(w[i], t1[i].x - t0[i].x, t0[i].x), si[0]);
                    si[1] = fmaf(g[i], fmaf(w[i], t1[i].y - t0[i].y, t0[i].y), si[1]);
                }
            }
        };
        if (v + kBpGroup <= v_end) {
#pragma unroll
            for (int u = 0; u < kBpGroup; ++u) view(u);
        } else {
            for (int u = 0; v + u < v_end; ++u) view(u);
        }
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            acc[i][0] += (double)s[i][0];
            acc[i][1] += (double)s[i][1];
        }
    }
    const size_t N = (size_t)nx * ny;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PX; ++i) sh.sum[wid][i][lane] = acc[i][e];
        __syncthreads();
        const int t = threadIdx.x, tx = t % TX, ty = t / TX;
        if (t < TX * 16 && x0 + tx < nx && y0 + ty < ny && 2 * pr + e < batch) {
            double a = 0.0;
#pragma unroll
            for (int k = 0; k < kBpWaves; ++k) a += sh.sum[k][ty % PX][ty / PX * TX + tx];
            img[(size_t)(2 * pr + e) * N + (size_t)(y0 + ty) * nx + x0 + tx] =
                (float)(a * (double)scale);
        }
    }
}

std::mutex g_fbp_mu;
std::vector<std::pair<std::pair<int, hipStream_t>, std::unique_ptr<DevBuf>>> g_fbp_ws;

DevBuf *fbp_workspace(hipStream_t s)
{
    int dev = 0;
    (void)hipGetDevice(&dev);
    for (auto &p : g_fbp_ws)
        if (p.first.first == dev && p.first.second == s) return p.second.get();
    g_fbp_ws.emplace_back(std::make_pair(dev, s), std::make_unique<DevBuf>());
    return g_fbp_ws.back().second.get();
}

}  // namespace

// Bytes of the filtered, padded sinograms of `batch` items (pairs).
static size_t fbp_work_bytes(const dect_geometry *g, int batch)
{
    return (size_t)pairs_of(batch) * g->n_views * (g->n_bins + 2 * kQPad) * sizeof(f2v);
}

// The work buffer dect_fbp allocates for `batch` sinograms on one stream,
// for a dry run under a SizingScope.
dect_status fbp_size_run(const dect_geometry *g, int batch)
{
    DevBuf w;
    return w.ensure(fbp_work_bytes(g, batch));
}

dect_status fbp(const dect_geometry *g, const float *sino, float *img, int batch, hipStream_t s)
{
    if (!sino || !img || batch <= 0)
        return fail(DECT_ERR_INVALID_ARG, "dect_fbp: null buffer or batch <= 0");
    dect_status st = validate_geometry(g);
    if (st != DECT_OK) return st;
    if (g->angles_rad)
        return fail(DECT_ERR_INVALID_ARG, "dect_fbp: needs the equally spaced full turn (angles_rad NULL)");
    if (g->n_bins > kFbpMaxBins)
        return fail(DECT_ERR_INVALID_ARG, "dect_fbp: at most 6144 detector bins");
    GeomTables *t = nullptr;
    if ((st = get_tables(g, &t)) != DECT_OK) return st;
    const int V = g->n_views, B = g->n_bins, pairs = pairs_of(batch);
    const size_t qbytes = fbp_work_bytes(g, batch);
    std::lock_guard<std::mutex> lk(g_fbp_mu);
    DevBuf *w = fbp_workspace(s);
    if (w->bytes < qbytes) {
        DECT_HIP(hipStreamSynchronize(s));
        if ((st = w->ensure(qbytes)) != DECT_OK) return st;
    }
    const double R = g->sod_mm, D = g->sdd_mm, du = g->bin_mm;
    const double ds = du * R / D;
    hipLaunchKernelGGL(k_fbp_filter, dim3((unsigned)((B + 63) / 64), (unsigned)((V + 7) / 8), pairs),
                       dim3(256), 0, s, sino, batch, V, B,
                       (float)R, (float)(R / D), (float)(-(B - 1) / 2.0 * du + g->det_offset_mm),
                       (float)du, (float)(0.5 / ds), (f2v *)w->ptr);
    DECT_HIP(hipGetLastError());
    const int ntx = (g->nx + 15) / 16, nty = (g->ny + 15) / 16;
    const double b0 = (B - 1) / 2.0 - g->det_offset_mm / du;
    // bins between a tile's centre and its corners, at most: half the tile's diagonal times
    // the gradient of the detector position over the image and its overhanging tiles
    const double rm = 0.5 * g->pixel_mm * std::hypot((double)g->nx + 32.0, (double)g->ny + 16.0);
    const double grad = rm < R ? g->pixel_mm * (D / (R - rm)) / du *
                                     std::sqrt(1.0 + rm * rm / (R * R - rm * rm))
                               : INFINITY;
    const double room = kBpWin / 2 - 2.5;
    const float scale = (float)(2.0 * M_PI / V * R * R);  // (the weights are 1 / distance^2)
    const auto windowed = [&](auto kern, int tx) {
        hipLaunchKernelGGL(kern, dim3((g->nx + tx - 1) / tx * nty, pairs), dim3(kBpWaves * 64), 0, s,
                           (const f2v *)w->ptr, (const ViewInfo *)t->views, batch, g->nx, g->ny, V,
                           B, (float)g->pixel_mm, R, D / du, b0, scale, img);
    };
    if (std::hypot(15.5, 7.5) * grad <= room && (size_t)ntx * nty * pairs >= kBpWide) {
        windowed(k_fbp_bp_win<32>, 32);
        DECT_HIP(hipGetLastError());
        return DECT_OK;
    }
    if (std::hypot(7.5, 7.5) * grad <= room) {
        windowed(k_fbp_bp_win<16>, 16);
        DECT_HIP(hipGetLastError());
        return DECT_OK;
    }
    // bins between a tile's centre and its corners where the image comes closest to the source
    const double rc = 0.5 * g->pixel_mm * std::hypot((double)g->nx - 1.0, (double)g->ny - 1.0);
    const double across = std::hypot(7.5, 7.5) * g->pixel_mm * (D / (R - rc)) / du *
                          std::sqrt(1.0 + rc * rc / (R * R - rc * rc));
    const bool rel = across < 0.5 * B, few = (size_t)ntx * nty * pairs <= kBpFew;
    const auto bp = few ? (rel ? k_fbp_bp<true, 4> : k_fbp_bp<false, 4>)
                        : (rel ? k_fbp_bp<true, 1> : k_fbp_bp<false, 1>);
    hipLaunchKernelGGL(bp, dim3(ntx * nty, pairs), dim3(few ? 1024 : 256), 0, s, (const f2v *)w->ptr,
                       (const ViewInfo *)t->views, batch, g->nx, g->ny, V, B, (float)g->pixel_mm,
                       R, D / du, b0, scale, img);
    DECT_HIP(hipGetLastError());
    return DECT_OK;
}

void release_fbp_work()
{
    std::lock_guard<std::mutex> lk(g_fbp_mu);
    g_fbp_ws.clear();
}

}  // namespace dect
