// One unrolled ADM-TV step (Eq. 10 with a given step alpha in place of the
// BB step) and its vector-Jacobian product, for a batch of images that
// share one size.  The data term h = mu A^T (A f - g) comes from the
// projector pair (the caller forms A f, r = A f - g with k_unr_resid, and
// A^T r); everything else runs here:
//   z  = shrink(grad f - lambda / rho, 1 / rho)                      (Eq. 8)
//   G  = mu hb + grad^T (rho (grad f - z) - lambda)                  (Eq. 9)
//   f' = f - alpha G
//   lambda' = lambda - xi (grad f' - z)                              (Eq. 7)
// with grad the backward differences of Eq. 2 (zero on the first column and
// row), grad^T its exact adjoint and shrink the isotropic shrinkage with
// |v| evaluated as sqrt(max(|v|^2, 1e-30)) so that value and derivative stay
// finite at v = 0.  Images are [batch][ny][nx] FP32; (mu, rho, xi, alpha)
// are read from device memory, so learnable step parameters never leave the
// device.  Per-pixel arithmetic in FP32; the parameter gradients are FP64
// per-block partial sums reduced in a fixed order by one block (bitwise
// reproducible).
#include <cmath>
#include <mutex>
#include <vector>

#include "common.h"
#include "reduce.h"
#include "xcd.h"

namespace dect {
namespace {

constexpr int kUnrBlocks = 2048;  // grid of the residual kernel (grid-stride)
enum { P_MU, P_RHO, P_XI, P_ALPHA, P_COUNT };

// The step and its backward pass run on tiles of kUX x kUY pixels of one
// image, 256 threads, with everything the neighbours share in LDS: the z-step
// is formed once on the tile and one pixel around it (W region), f' once on
// the tile and the pixels before it, and the intermediate images of the
// backward pass (G, f', f'~, G~, d~) never leave the block.  A thread keeps
// the same W-region pixels (at most kUK) through every phase.  8 x 512^2:
// forward 33 -> 16 us (its seven arrays take 11 at 5.1 TB/s), backward 90 -> 52
// (eleven arrays, 18; then bound by its divisions), against passes per pixel
// with 64-bit index divisions, three z-steps each and six intermediate images.
constexpr int kUX = 32, kUY = 16;
constexpr int kUWX = kUX + 2, kUWY = kUY + 2;  // W region: rows / columns -1 .. tile
constexpr int kUFX = kUX + 3, kUFY = kUY + 3;  // f region: -2 .. tile
constexpr int kUK = (kUWX * kUWY + 255) / 256;
static_assert(kUFX * kUFY <= 256 * kUK, "the f region takes as many loads as the W region");
constexpr unsigned kUnrGrid = 4096;  // blocks at most (each then takes several tiles)

struct Img {
    int nx, ny;
    int tx, ty;      // tiles along x and y
    int64_t ntiles;  // of the batch
    size_t N, T;     // pixels per image, pixels of the batch
};

struct Prm {
    float mu, rho, xi, alpha;
};

__device__ __forceinline__ Prm load_prm(const float *__restrict__ p)
{
    return Prm{p[0], p[1], p[2], p[3]};
}

// The z-step: v = grad f - lambda / rho, n = |v| (floored), the shrink factor
// s and z = s v; also W = rho (grad f - z) - lambda.
struct ZW {
    float dx, dy, vx, vy, n, zx, zy, wx, wy;
};

__device__ __forceinline__ ZW zstep(float dx, float dy, float lxi, float lyi, float rho)
{
    ZW o;
    o.dx = dx;
    o.dy = dy;
    o.vx = o.dx - lxi / rho;
    o.vy = o.dy - lyi / rho;
    o.n = sqrtf(fmaxf(o.vx * o.vx + o.vy * o.vy, 1e-30f));
    const float t = 1.0f / rho;
    const float s = fmaxf(o.n - t, 0.f) / o.n;
    o.zx = s * o.vx;
    o.zy = s * o.vy;
    o.wx = rho * (o.dx - o.zx) - lxi;
    o.wy = rho * (o.dy - o.zy) - lyi;
    return o;
}

// A thread's pixel k of the W region: its place rr, cc in the region (tile
// pixels at 1 .. kUY, 1 .. kUX), row r and column c and offset o in the image;
// in: it exists and lies in the image (else o = 0, an element that is loaded
// and not used).
struct Px {
    int rr, cc, r, c;
    size_t o;
    bool in;
    __device__ bool own() const { return in && rr >= 1 && rr <= kUY && cc >= 1 && cc <= kUX; }
    __device__ bool before() const { return in && rr <= kUY && cc <= kUX; }  // tile and pixels before it
};

__device__ __forceinline__ Px px_at(const Img &d, int r0, int c0, int k)
{
    const int i = threadIdx.x + 256 * k;
    Px p;
    p.rr = i / kUWX;
    p.cc = i % kUWX;
    p.r = r0 - 1 + p.rr;
    p.c = c0 - 1 + p.cc;
    p.in = i < kUWX * kUWY && p.r >= 0 && p.r < d.ny && p.c >= 0 && p.c < d.nx;
    p.o = p.in ? (size_t)p.r * d.nx + p.c : 0;
    return p;
}

// f on its region, from registers loaded by f_load
__device__ __forceinline__ void f_load(const Img &d, const float *__restrict__ f, int r0, int c0,
                                       float (&v)[kUK])
{
#pragma unroll
    for (int k = 0; k < kUK; ++k) {
        const int i = threadIdx.x + 256 * k, r = r0 - 2 + i / kUFX, c = c0 - 2 + i % kUFX;
        const bool in = i < kUFX * kUFY && r >= 0 && r < d.ny && c >= 0 && c < d.nx;
        v[k] = f[in ? (size_t)r * d.nx + c : 0];
    }
}

__device__ __forceinline__ void f_store(const float (&v)[kUK], float (&sf)[kUFY][kUFX])
{
#pragma unroll
    for (int k = 0; k < kUK; ++k) {
        const int i = threadIdx.x + 256 * k;
        if (i < kUFX * kUFY) sf[i / kUFX][i % kUFX] = v[k];
    }
}

// Backward differences of Eq. 2 at a W-region pixel from a W-region array.
__device__ __forceinline__ void grad_w(const Px &p, const float (&s)[kUWY][kUWX], float own, float &gx,
                                       float &gy)
{
    gx = p.c >= 1 ? own - s[p.rr][p.cc - 1] : 0.f;
    gy = p.r >= 1 ? own - s[p.rr - 1][p.cc] : 0.f;
}

// grad^T of the field (sx, sy) at a W-region pixel
__device__ __forceinline__ float grad_t(const Img &d, const Px &p, const float (&sx)[kUWY][kUWX],
                                        const float (&sy)[kUWY][kUWX])
{
    float s = 0.f;
    if (p.c >= 1) s += sx[p.rr][p.cc];
    if (p.c + 1 <= d.nx - 1) s -= sx[p.rr][p.cc + 1];
    if (p.r >= 1) s += sy[p.rr][p.cc];
    if (p.r + 1 <= d.ny - 1) s -= sy[p.rr + 1][p.cc];
    return s;
}

// The z-steps of the W region (wx, wy to swx, swy) from f in sf.
__device__ __forceinline__ void z_region(const Px (&px)[kUK], const float (&sf)[kUFY][kUFX],
                                         const float (&lx)[kUK], const float (&ly)[kUK], float rho,
                                         ZW (&z)[kUK], float (&swx)[kUWY][kUWX],
                                         float (&swy)[kUWY][kUWX])
{
#pragma unroll
    for (int k = 0; k < kUK; ++k) {
        const Px &p = px[k];
        if (!p.in) continue;
        const float f = sf[p.rr + 1][p.cc + 1];
        z[k] = zstep(p.c >= 1 ? f - sf[p.rr + 1][p.cc] : 0.f, p.r >= 1 ? f - sf[p.rr][p.cc + 1] : 0.f,
                     lx[k], ly[k], rho);
        swx[p.rr][p.cc] = z[k].wx;
        swy[p.rr][p.cc] = z[k].wy;
    }
}

// Tile t: its image's first pixel and the tile's first row and column.
__device__ __forceinline__ size_t tile_at(const Img &d, int64_t t, int &r0, int &c0)
{
    const int per = d.tx * d.ty;
    const int64_t img = t / per;
    const int q = (int)(t - img * per);
    r0 = q / d.tx * kUY;
    c0 = q % d.tx * kUX;
    return (size_t)img * d.N;
}

// r = p - g (r may be p)
__global__ __launch_bounds__(256) void k_unr_resid(const float *p, const float *__restrict__ g,
                                                   size_t n, float *r)
{
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
        r[i] = p[i] - g[i];
}

// f' = f - alpha G and lambda' = lambda - xi (grad f' - z).
__global__ __launch_bounds__(256) void k_unr_fwd(Img d, const float *__restrict__ f,
                                                 const float *__restrict__ lx,
                                                 const float *__restrict__ ly,
                                                 const float *__restrict__ hb,
                                                 const float *__restrict__ prm,
                                                 float *__restrict__ fo, float *__restrict__ lxo,
                                                 float *__restrict__ lyo)
{
    __shared__ float sf[kUFY][kUFX], swx[kUWY][kUWX], swy[kUWY][kUWX], sfo[kUWY][kUWX];
    const Prm p = load_prm(prm);
    const unsigned b0 = gridDim.x == d.ntiles ? xcd_order(blockIdx.x, gridDim.x) : blockIdx.x;
    for (int64_t t = b0; t < d.ntiles; t += gridDim.x) {
        int r0, c0;
        const size_t im = tile_at(d, t, r0, c0);
        Px px[kUK];
        float vf[kUK], vlx[kUK], vly[kUK], vh[kUK];
        f_load(d, f + im, r0, c0, vf);
#pragma unroll
        for (int k = 0; k < kUK; ++k) {
            px[k] = px_at(d, r0, c0, k);
            vlx[k] = lx[im + px[k].o];
            vly[k] = ly[im + px[k].o];
            vh[k] = hb[im + px[k].o];
        }
        __syncthreads();  // the tile before is done with the LDS
        f_store(vf, sf);
        __syncthreads();
        ZW z[kUK];
        z_region(px, sf, vlx, vly, p.rho, z, swx, swy);
        __syncthreads();
        float fn[kUK];
#pragma unroll
        for (int k = 0; k < kUK; ++k) {
            const Px &q = px[k];
            if (!q.before()) continue;
            const float G = p.mu * vh[k] + grad_t(d, q, swx, swy);
            fn[k] = sf[q.rr + 1][q.cc + 1] - p.alpha * G;
            sfo[q.rr][q.cc] = fn[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kUK; ++k) {
            const Px &q = px[k];
            if (!q.own()) continue;
            float gx, gy;
            grad_w(q, sfo, fn[k], gx, gy);
            fo[im + q.o] = fn[k];
            lxo[im + q.o] = vlx[k] - p.xi * (gx - z[k].zx);
            lyo[im + q.o] = vly[k] - p.xi * (gy - z[k].zy);
        }
    }
}

// Backward, given the cotangents gfo of f' and glx, gly of lambda' (G, f' and
// z formed again, bitwise as in the forward):
//   the multiplier step: d(grad f')~ = -xi glam', xi~ = -<glam', grad f' - z>;
//   f'~ = gfo + grad^T d(grad f')~;
//   G~ = -alpha f'~, alpha~ = -<f'~, G>; hb~ = mu G~, mu~ = <G~, hb>;
//   W~ = grad G~ (grad^T's adjoint), then through W = rho (d - z) - lambda,
//   the shrinkage and v = d - lambda / rho:
//   z~ = xi glam' - rho W~;
//   v~ = z~ - t (z~ / n - v <v, z~> / n^3), t~ = -<z~, v> / n  where n > t
//        (z = v - t v / n), else 0;
//   d~ = rho W~ + v~, lambda~ = glam' - W~ - v~ / rho;
//   rho~ = <W~, d - z> + <v~, lambda> / rho^2 - t~ / rho^2;
//   f~ = f'~ + grad^T d~.
// The parameter gradients leave as one partial sum per block each.
__global__ __launch_bounds__(256) void k_unr_bwd(Img d, const float *__restrict__ f,
                                                 const float *__restrict__ lx,
                                                 const float *__restrict__ ly,
                                                 const float *__restrict__ hb,
                                                 const float *__restrict__ prm,
                                                 const float *__restrict__ gfo,
                                                 const float *__restrict__ glxo,
                                                 const float *__restrict__ glyo,
                                                 float *__restrict__ gf, float *__restrict__ glx,
                                                 float *__restrict__ gly, float *__restrict__ ghb,
                                                 double *__restrict__ part, size_t stride)
{
    // W and then d~ in swx, swy
    __shared__ float sf[kUFY][kUFX], swx[kUWY][kUWX], swy[kUWY][kUWX], sfo[kUWY][kUWX];
    // glam' on the W region and the column / row after it; G~
    __shared__ float sax[kUWY][kUWX + 1], say[kUWY + 1][kUWX], sgb[kUWY][kUWX];
    const Prm p = load_prm(prm);
    const float t = 1.0f / p.rho;
    double sum[P_COUNT] = {0.0, 0.0, 0.0, 0.0};
    double srho2 = 0.0;  // the terms of rho~ over rho^2
    const unsigned b0 = gridDim.x == d.ntiles ? xcd_order(blockIdx.x, gridDim.x) : blockIdx.x;
    for (int64_t tile = b0; tile < d.ntiles; tile += gridDim.x) {
        int r0, c0;
        const size_t im = tile_at(d, tile, r0, c0);
        Px px[kUK];
        float vf[kUK], vlx[kUK], vly[kUK], vh[kUK], vg[kUK], vax[kUK], vay[kUK];
        f_load(d, f + im, r0, c0, vf);
#pragma unroll
        for (int k = 0; k < kUK; ++k) {
            px[k] = px_at(d, r0, c0, k);
            const size_t o = im + px[k].o;
            vlx[k] = lx[o];
            vly[k] = ly[o];
            vh[k] = hb[o];
            vg[k] = gfo[o];
            vax[k] = glxo[o];
            vay[k] = glyo[o];
        }
        // the column after the W region of glx, the row after it of gly
        const int er = r0 - 1 + (int)threadIdx.x, ec = c0 + kUX + 1;
        const bool ein = (int)threadIdx.x < kUWY && er >= 0 && er < d.ny && ec < d.nx;
        const float eax = glxo[im + (ein ? (size_t)er * d.nx + ec : 0)];
        const int fr = r0 + kUY + 1, fc = c0 - 1 + (int)threadIdx.x;
        const bool fin = (int)threadIdx.x < kUWX && fc >= 0 && fc < d.nx && fr < d.ny;
        const float eay = glyo[im + (fin ? (size_t)fr * d.nx + fc : 0)];
        __syncthreads();  // the tile before is done with the LDS
        f_store(vf, sf);
#pragma unroll
        for (int k = 0; k < kUK; ++k)
            if (px[k].in) {
                sax[px[k].rr][px[k].cc] = vax[k];
                say[px[k].rr][px[k].cc] = vay[k];
            }
        if (ein) sax[threadIdx.x][kUWX] = eax;
        if (fin) say[kUWY][threadIdx.x] = eay;
        __syncthreads();
        ZW z[kUK];
        z_region(px, sf, vlx, vly, p.rho, z, swx, swy);
        // f'~ and G~ on the W region
        float ft[kUK], gb[kUK];
#pragma unroll
        for (int k = 0; k < kUK; ++k) {
            const Px &q = px[k];
            if (!q.in) continue;
            float u = 0.f;  // grad^T of -xi glam'
            if (q.c >= 1) u += -p.xi * vax[k];
            if (q.c + 1 <= d.nx - 1) u -= -p.xi * sax[q.rr][q.cc + 1];
            if (q.r >= 1) u += -p.xi * vay[k];
            if (q.r + 1 <= d.ny - 1) u -= -p.xi * say[q.rr + 1][q.cc];
            ft[k] = vg[k] + u;
            gb[k] = -p.alpha * ft[k];
            sgb[q.rr][q.cc] = gb[k];
        }
        __syncthreads();
        float G[kUK], fn[kUK];
#pragma unroll
        for (int k = 0; k < kUK; ++k) {
            const Px &q = px[k];
            if (!q.before()) continue;
            G[k] = p.mu * vh[k] + grad_t(d, q, swx, swy);
            fn[k] = sf[q.rr + 1][q.cc + 1] - p.alpha * G[k];
            sfo[q.rr][q.cc] = fn[k];
        }
        __syncthreads();  // W has been read: d~ takes its place
#pragma unroll
        for (int k = 0; k < kUK; ++k) {
            const Px &q = px[k];
            if (!q.in || q.rr < 1 || q.cc < 1) continue;  // the tile and the pixels after it
            float wbx, wby;
            grad_w(q, sgb, gb[k], wbx, wby);
            const float zbx = p.xi * vax[k] - p.rho * wbx, zby = p.xi * vay[k] - p.rho * wby;
            float vbx = 0.f, vby = 0.f, tb = 0.f;
            if (z[k].n > t) {
                const float vz = z[k].vx * zbx + z[k].vy * zby;
                const float n3 = z[k].n * z[k].n * z[k].n;
                vbx = zbx - t * (zbx / z[k].n - z[k].vx * vz / n3);
                vby = zby - t * (zby / z[k].n - z[k].vy * vz / n3);
                tb = -vz / z[k].n;
            }
            swx[q.rr][q.cc] = p.rho * wbx + vbx;
            swy[q.rr][q.cc] = p.rho * wby + vby;
            if (!q.own()) continue;
            const size_t o = im + q.o;
            glx[o] = vax[k] - wbx - vbx / p.rho;
            gly[o] = vay[k] - wby - vby / p.rho;
            ghb[o] = p.mu * gb[k];
            float gx, gy;
            grad_w(q, sfo, fn[k], gx, gy);
            sum[P_MU] += (double)gb[k] * vh[k];
            sum[P_RHO] += (double)wbx * (z[k].dx - z[k].zx) + (double)wby * (z[k].dy - z[k].zy);
            srho2 += ((double)vbx * vlx[k] + (double)vby * vly[k]) - (double)tb;
            sum[P_XI] -= (double)vax[k] * (gx - z[k].zx) + (double)vay[k] * (gy - z[k].zy);
            sum[P_ALPHA] -= (double)ft[k] * G[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kUK; ++k)
            if (px[k].own()) gf[im + px[k].o] = ft[k] + grad_t(d, px[k], swx, swy);
    }
    sum[P_RHO] += srho2 / ((double)p.rho * p.rho);
    __shared__ double tot[P_COUNT];
    block_sum<P_COUNT>(sum, tot);
    if (threadIdx.x < P_COUNT) part[threadIdx.x * stride + blockIdx.x] = tot[threadIdx.x];
}

// The four parameter gradients (mu, rho, xi, alpha), one block each, from the
// partial sums in a fixed order, rounded to FP32.
__global__ __launch_bounds__(256) void k_unr_bwd_prm(const double *__restrict__ part,
                                                     size_t stride, int nb,
                                                     float *__restrict__ gprm)
{
    __shared__ double tot[1];
    double v[1] = {0.0};
    const double *q = part + blockIdx.x * stride;
    constexpr int kU = kUnrGrid / 256;  // loads in flight: all of them
    double u[kU];
#pragma unroll
    for (int k = 0; k < kU; ++k) {
        const int b = threadIdx.x + 256 * k;
        u[k] = b < nb ? q[b] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < kU; ++k) v[0] += u[k];
    block_sum<1>(v, tot);
    if (threadIdx.x == 0) gprm[blockIdx.x] = (float)tot[0];
}

// The partial sums of a backward call, kept per device and stream: calls on two
// streams may overlap.  A buffer holds the largest grid's sums, so none grows
// under a graph that has recorded it.
struct UnrWork {
    int dev;
    hipStream_t stream;
    bool spare;  // of no stream yet
    DevBuf part;
};

std::mutex g_unr_mu;
std::vector<std::unique_ptr<UnrWork>> g_unr;

// The buffer of at least `bytes` for stream s.  Where an allocation must not be
// made, in a capture that no call on this stream has prepared, it takes the
// device's spare one, which an eager call leaves behind.
dect_status unr_work(hipStream_t s, size_t bytes, double **part)
{
    int dev = 0;
    DECT_HIP(hipGetDevice(&dev));
    const bool arena = caller_workspace();
    const size_t size = arena ? bytes : (size_t)P_COUNT * kUnrGrid * 8;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const bool capturing =
        !arena && (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone);
    UnrWork *mine = nullptr, *spare = nullptr, *any = nullptr;
    for (auto &w : g_unr) {
        if (w->dev != dev) continue;
        if (w->spare) spare = w.get();
        else if (w->stream == s) mine = w.get();
        else any = w.get();
    }
    if (!mine && capturing) {
        if ((mine = spare)) {
            mine->spare = false;
            mine->stream = s;
        } else if (any) {  // (all handed out: the stream's calls must not overlap its owner's)
            mine = any;
        }
    }
    auto make = [&](bool is_spare) -> UnrWork * {
        g_unr.push_back(std::make_unique<UnrWork>());
        UnrWork *w = g_unr.back().get();
        w->dev = dev;
        w->stream = s;
        w->spare = is_spare;
        return w;
    };
    if (!mine) mine = make(false);
    dect_status st = mine->part.ensure(size);
    if (st) return st;
    if (!capturing && !arena && !spare && (st = make(true)->part.ensure(size))) return st;
    *part = (double *)mine->part.ptr;
    return DECT_OK;
}

dect_status check_img(int nx, int ny, int batch, Img &d)
{
    if (nx <= 0 || ny <= 0 || batch < 0 || (int64_t)nx * ny > (int64_t)1 << 30 ||
        (int64_t)nx * ny * batch > (int64_t)1 << 34)
        return fail(DECT_ERR_INVALID_ARG, "unrolled step: bad image size or batch");
    d.nx = nx;
    d.ny = ny;
    d.N = (size_t)nx * ny;
    d.T = d.N * (size_t)batch;
    d.tx = (nx + kUX - 1) / kUX;
    d.ty = (ny + kUY - 1) / kUY;
    d.ntiles = (int64_t)d.tx * d.ty * batch;
    return DECT_OK;
}

unsigned grid_of(size_t n) { return (unsigned)std::min<size_t>(kUnrBlocks, (n + 255) / 256); }

unsigned tile_grid(const Img &d) { return (unsigned)std::min<int64_t>(kUnrGrid, d.ntiles); }

bool overlaps(const void *a, const void *b, size_t bytes)
{
    const char *x = (const char *)a, *y = (const char *)b;
    return x < y + bytes && y < x + bytes;
}

}  // namespace

void release_unrolled_work()
{
    std::lock_guard<std::mutex> lk(g_unr_mu);
    g_unr.clear();
}

dect_status unrolled_residual(int64_t n, const float *p, const float *g, float *r, hipStream_t s)
{
    if (n < 0) return fail(DECT_ERR_INVALID_ARG, "dect_unrolled_residual: n < 0");
    if (n == 0) return DECT_OK;
    if (!p || !g || !r) return fail(DECT_ERR_INVALID_ARG, "dect_unrolled_residual: null buffer");
    hipLaunchKernelGGL(k_unr_resid, dim3(grid_of((size_t)n)), dim3(256), 0, s, p, g, (size_t)n,
                       r);
    DECT_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status unrolled_step(int nx, int ny, int batch, const float *f, const float *lx,
                          const float *ly, const float *hb, const float *prm, float *fo,
                          float *lxo, float *lyo, hipStream_t s)
{
    Img d;
    dect_status st = check_img(nx, ny, batch, d);
    if (st) return st;
    if (d.T == 0) return DECT_OK;
    if (!f || !lx || !ly || !hb || !prm || !fo || !lxo || !lyo)
        return fail(DECT_ERR_INVALID_ARG, "dect_unrolled_step: null buffer");
    const size_t bytes = d.T * 4;
    const void *in[4] = {f, lx, ly, hb};
    const void *out[3] = {fo, lxo, lyo};
    for (const void *o : out)
        for (const void *i : in)
            if (overlaps(o, i, bytes))
                return fail(DECT_ERR_INVALID_ARG, "dect_unrolled_step: outputs overlap inputs");
    if (overlaps(fo, lxo, bytes) || overlaps(fo, lyo, bytes) || overlaps(lxo, lyo, bytes))
        return fail(DECT_ERR_INVALID_ARG, "dect_unrolled_step: outputs overlap each other");
    hipLaunchKernelGGL(k_unr_fwd, dim3(tile_grid(d)), dim3(256), 0, s, d, f, lx, ly, hb, prm, fo, lxo,
                       lyo);
    DECT_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status unrolled_step_backward(int nx, int ny, int batch, const float *f, const float *lx,
                                   const float *ly, const float *hb, const float *prm,
                                   const float *gfo, const float *glxo, const float *glyo,
                                   float *gf, float *glx, float *gly, float *ghb, float *gprm,
                                   hipStream_t s)
{
    Img d;
    dect_status st = check_img(nx, ny, batch, d);
    if (st) return st;
    if (!gprm) return fail(DECT_ERR_INVALID_ARG, "dect_unrolled_step_backward: gprm is NULL");
    if (d.T == 0) {  // an empty batch: zero parameter gradients
        hipLaunchKernelGGL(k_unr_bwd_prm, dim3(P_COUNT), dim3(256), 0, s, (const double *)nullptr,
                           (size_t)0, 0, gprm);
        DECT_HIP(hipGetLastError());
        return DECT_OK;
    }
    if (!f || !lx || !ly || !hb || !prm || !gfo || !glxo || !glyo || !gf || !glx || !gly || !ghb)
        return fail(DECT_ERR_INVALID_ARG, "dect_unrolled_step_backward: null buffer");
    const size_t bytes = d.T * 4;
    const void *in[8] = {f, lx, ly, hb, gfo, glxo, glyo, prm};
    const void *out[4] = {gf, glx, gly, ghb};
    for (const void *o : out)
        for (int k = 0; k < 8; ++k)
            if (overlaps(o, in[k], k == 7 ? 16 : bytes))
                return fail(DECT_ERR_INVALID_ARG,
                            "dect_unrolled_step_backward: outputs overlap inputs");
    for (int a = 0; a < 4; ++a)
        for (int b = a + 1; b < 4; ++b)
            if (overlaps(out[a], out[b], bytes))
                return fail(DECT_ERR_INVALID_ARG,
                            "dect_unrolled_step_backward: outputs overlap each other");
    const unsigned g = tile_grid(d);
    std::lock_guard<std::mutex> lk(g_unr_mu);
    double *part = nullptr;
    if ((st = unr_work(s, (size_t)P_COUNT * g * 8, &part))) return st;
    hipLaunchKernelGGL(k_unr_bwd, dim3(g), dim3(256), 0, s, d, f, lx, ly, hb, prm, gfo, glxo, glyo, gf,
                       glx, gly, ghb, part, (size_t)g);
    DECT_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_unr_bwd_prm, dim3(P_COUNT), dim3(256), 0, s, (const double *)part, (size_t)g,
                       (int)g, gprm);
    DECT_HIP(hipGetLastError());
    return DECT_OK;
}

}  // namespace dect
