// Penalised least-squares image-domain decomposition (Eqs. 11-15) on gfx950.
//
//   dinv   : b = D^{-1} x per pixel (closed-form 2x2, Eq. 12); u starts at b.
//   prewitt: m2 = fmaf(gx, gx, gy*gy) of the Prewitt responses (fixed FP32
//            operation order, no contraction), per-block maxima.
//   weights: e_ik = eps where either pixel is an edge (m2 > tau^2 max m2),
//            1 otherwise (Eq. 14's edge weights after Sec. 2.3).
//   PCG    : (I + gamma L) u = b per material (Eq. 15 with grad R = 2L),
//            Jacobi preconditioner, two kernels per iteration, both materials
//            per launch.  Scalars are reduced redundantly by every block in
//            a fixed order, so every block takes the same decision.
#include <cmath>
#include <mutex>
#include <vector>

#include "common.h"
#include "reduce.h"

namespace dect {
namespace {

constexpr int kPix = 4;  // pixels per thread in the streaming kernels

// The sums of NV arrays of n doubles (one per block of a launch), in a fixed
// order, to every thread: all arrays' loads go out together, and one block
// reduction serves all of them.
template <int NV>
__device__ __forceinline__ void reduce_arrays(const double *const (&a)[NV], int n,
                                              double (&sum)[NV])
{
    double v[NV] = {};
    for (int i = threadIdx.x; i < n; i += 256)
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] += a[k][i];
    __shared__ double out[NV];
    block_sum<NV>(v, out);
#pragma unroll
    for (int k = 0; k < NV; ++k) sum[k] = out[k];
}

// A thread's pixel j of kPix (stride 256): its index, clamped to the last
// pixel, the indices of its four neighbours (its own where there is none) and
// which of them exist.  I: an unsigned type that holds the launch's last index, up
// to kPix * 256 - 1 past N (small_index).
template <typename I>
struct Pix {
    I i, r, l, d, u;
    bool in, hr, hl, hd, hu;
};

constexpr bool small_index(size_t N) { return N <= 0x100000000ull - 256 * kPix; }
static_assert(small_index(0xFFFFFC00u) && !small_index(0xFFFFFC01u), "the last block's indices fit 32 bits");

template <typename I>
__device__ __forceinline__ Pix<I> pixel_at(int j, int nx, int ny, I N)
{
    Pix<I> p;
    const I i = ((I)blockIdx.x * kPix + (I)j) * 256 + threadIdx.x;
    p.in = i < N;
    p.i = p.in ? i : N - 1;
    const I row = p.i / (I)nx, c = p.i - row * (I)nx;
    p.hr = c + 1 < (I)nx;
    p.hl = c >= 1;
    p.hd = row + 1 < (I)ny;
    p.hu = row >= 1;
    p.r = p.hr ? p.i + 1 : p.i;
    p.l = p.hl ? p.i - 1 : p.i;
    p.d = p.hd ? p.i + (I)nx : p.i;
    p.u = p.hu ? p.i - (I)nx : p.i;
    return p;
}

// The pair weights of a pixel to its right, left, lower and upper neighbour
// (zero where there is none, whatever the map holds there).
struct PairW {
    float r, l, d, u;
};

template <typename I>
__device__ __forceinline__ PairW pair_weights(const Pix<I> &p, const float *__restrict__ er,
                                              const float *__restrict__ ed)
{
    const float r = er[p.i], l = er[p.l], d = ed[p.i], u = ed[p.u];
    return PairW{p.hr ? r : 0.f, p.hl ? l : 0.f, p.hd ? d : 0.f, p.hu ? u : 0.f};
}

__device__ __forceinline__ float weight_sum(const PairW &w)
{
    return ((w.r + w.l) + w.d) + w.u;
}

// Row and column of pixel i (a 32-bit division where i allows it).
__device__ __forceinline__ void coords(size_t i, int nx, int &r, int &c)
{
    if (i >> 32) {
        r = (int)(i / nx);
        c = (int)(i % nx);
    } else {
        r = (int)((unsigned)i / (unsigned)nx);
        c = (int)((unsigned)i - (unsigned)r * (unsigned)nx);
    }
}

struct PlsCoef {
    float i11, i12, i21, i22;  // D^{-1} = [[i11, i12], [i21, i22]]
};

__global__ __launch_bounds__(256) void k_dinv(const float *__restrict__ xh,
                                              const float *__restrict__ xl, PlsCoef c,
                                              float *__restrict__ u1, float *__restrict__ u2,
                                              float *__restrict__ b, size_t N)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    float h = xh[i], l = xl[i];
    float a = c.i11 * h + c.i12 * l;
    float d = c.i21 * h + c.i22 * l;
    u1[i] = a;
    u2[i] = d;
    b[i] = a;
    b[N + i] = d;
}

__global__ __launch_bounds__(256) void k_prewitt(const float *__restrict__ x,
                                                 float *__restrict__ m2,
                                                 float *__restrict__ pmax, int nx, int ny)
{
#pragma clang fp contract(off)
    const size_t N = (size_t)nx * ny;
    float mx = 0.f;
    for (int j = 0; j < kPix; ++j) {
        size_t i = ((size_t)blockIdx.x * kPix + j) * 256 + threadIdx.x;
        if (i < N) {
            int r, c;
            coords(i, nx, r, c);
            int ru = r > 0 ? r - 1 : 0, rd = r < ny - 1 ? r + 1 : ny - 1;
            int cl = c > 0 ? c - 1 : 0, cr = c < nx - 1 ? c + 1 : nx - 1;
#define X(rr, cc) x[(size_t)(rr) * nx + (cc)]
            float right = (X(ru, cr) + X(r, cr)) + X(rd, cr);
            float left = (X(ru, cl) + X(r, cl)) + X(rd, cl);
            float down = (X(rd, cl) + X(rd, c)) + X(rd, cr);
            float up = (X(ru, cl) + X(ru, c)) + X(ru, cr);
#undef X
            float gx = right - left, gy = down - up;
            float v = fmaf(gx, gx, gy * gy);
            m2[i] = v;
            mx = fmaxf(mx, v);
        }
    }
    __shared__ float sh[256];
    sh[threadIdx.x] = mx;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = fmaxf(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) pmax[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(256) void k_weights(const float *__restrict__ m2,
                                                 const float *__restrict__ pmax, int nblk,
                                                 float tau2, float eps, float *__restrict__ w,
                                                 int nx, int ny)
{
    __shared__ float sh[256];
    float mx = 0.f;
    for (int i = threadIdx.x; i < nblk; i += 256) mx = fmaxf(mx, pmax[i]);
    sh[threadIdx.x] = mx;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = fmaxf(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    const float thr = tau2 * sh[0];
    const size_t N = (size_t)nx * ny;
    for (int j = 0; j < kPix; ++j) {
        size_t i = ((size_t)blockIdx.x * kPix + j) * 256 + threadIdx.x;
        if (i < N) {
            int r, c;
            coords(i, nx, r, c);
            bool ei = m2[i] > thr;
            float wr = 0.f, wd = 0.f;
            if (c + 1 < nx) wr = (ei || m2[i + 1] > thr) ? eps : 1.0f;
            if (r + 1 < ny) wd = (ei || m2[i + nx] > thr) ? eps : 1.0f;
            w[i] = wr;
            w[N + i] = wd;
        }
    }
}

// A launch that ends the solve says which one it is: `since` is its number plus
// one (part A of iteration it is launch 2 it, part B 2 it + 1).  Only later
// launches leave on it, so that every wavefront of a block decides alike, also
// while block 0 of its own launch writes.
struct PcgStatus {
    int32_t done, iters;
    double relres;
    uint32_t since, pad;
};

__device__ __forceinline__ bool pcg_over(const PcgStatus *stat, unsigned launch)
{
    const unsigned since = stat->since;
    return since != 0 && since <= launch;
}

// The kernels of an iteration are bound by latency at image sizes (2 MB of
// vectors, 512 blocks): every load of a block -- the four pixels' stencils and
// the per-block partial sums of the launch before -- is issued before any is
// used, unconditionally (a neighbour that does not exist reads the pixel
// itself, with weight zero), and the sums are reduced together.  512 x 512,
// both materials, traced: k_pcg_a 7.1 -> 4.0 us, k_pcg_b 3.9 -> 3.5 us.

// Setup: res = b - (I + gamma L) b (u starts at b), z = M^{-1} res with the Jacobi
// preconditioner M = 1 + gamma sum_k e_ik, p_old = 0, partials rz, |res|^2, |b|^2.
template <typename I>
__global__ __launch_bounds__(256) void k_pcg_setup(
    const float *__restrict__ b, const float *__restrict__ w, float gamma,
    float *__restrict__ res, float *__restrict__ z, float *__restrict__ pold,
    float *__restrict__ minv, double *__restrict__ p_rz, double *__restrict__ p_rr,
    double *__restrict__ p_bb, PcgStatus *__restrict__ stat, int nx, int ny, int nblk)
{
    const int m = blockIdx.y;
    const I N = (I)nx * (I)ny;
    const float *bm = b + (size_t)m * N;
    Pix<I> px[kPix];
    PairW e[kPix];
    float bc[kPix][5];
#pragma unroll
    for (int j = 0; j < kPix; ++j) {
        px[j] = pixel_at<I>(j, nx, ny, N);
        e[j] = pair_weights(px[j], w, w + N);
        bc[j][0] = bm[px[j].i];
        bc[j][1] = bm[px[j].r];
        bc[j][2] = bm[px[j].l];
        bc[j][3] = bm[px[j].d];
        bc[j][4] = bm[px[j].u];
    }
    double v[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < kPix; ++j) {
        if (!px[j].in) continue;
        const size_t i = px[j].i;
        const float ui = bc[j][0];
        float lu = 0.f;
        lu += e[j].r * (ui - bc[j][1]);
        lu += e[j].l * (ui - bc[j][2]);
        lu += e[j].d * (ui - bc[j][3]);
        lu += e[j].u * (ui - bc[j][4]);
        const float rs = ui - (ui + gamma * lu);
        const float mi = 1.0f / (1.0f + gamma * weight_sum(e[j]));
        const float zz = mi * rs;
        res[(size_t)m * N + i] = rs;
        z[(size_t)m * N + i] = zz;
        pold[(size_t)m * N + i] = 0.f;
        if (m == 0) minv[i] = mi;
        v[0] += (double)rs * zz;
        v[1] += (double)rs * rs;
        v[2] += (double)ui * ui;
    }
    __shared__ double out[3];
    block_sum<3>(v, out);
    if (threadIdx.x == 0) {
        p_rz[(size_t)m * nblk + blockIdx.x] = out[0];
        p_rr[(size_t)m * nblk + blockIdx.x] = out[1];
        p_bb[(size_t)m * nblk + blockIdx.x] = out[2];
        if (blockIdx.x == 0) {
            stat[m].done = 0;
            stat[m].iters = 0;
            stat[m].relres = 0.0;
            stat[m].since = 0;
        }
    }
}

// The convergence test on the previous residual and beta of iteration it, from
// the partial sums of <res, z> now and before, |res|^2 and |b|^2.  False where
// the solve is done (block 0 records it).
__device__ __forceinline__ bool pcg_begin(const double *rz_cur, const double *rz_prev,
                                          const double *p_rr, const double *p_bb, int nblk, int it,
                                          double tol, PcgStatus *stat, double &beta)
{
    const double *const arr[4] = {p_rr, p_bb, rz_cur, rz_prev};
    double sum[4];
    reduce_arrays<4>(arr, nblk, sum);
    const double bn = sum[1] > 0.0 ? sqrt(sum[1]) : 1.0;
    const double rn = sum[1] > 0.0 ? sqrt(sum[0]) : 0.0;
    if (rn <= tol * bn) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            stat->done = 1;
            stat->iters = it;
            stat->relres = rn / bn;
            stat->since = 2u * (unsigned)it + 1u;
        }
        return false;
    }
    beta = it > 0 ? sum[2] / sum[3] : 0.0;
    return true;
}

// Iteration it, part A: convergence test on the previous residual, beta,
// p_new = z + beta p_old, q = (I + gamma L) p_new, partial <p_new, q>.
// rz_cur: partials of <res, z> of this iteration; rz_prev of the previous.
template <typename I>
__global__ __launch_bounds__(256) void k_pcg_a(
    const float *__restrict__ z, const float *__restrict__ pold, float *__restrict__ pnew,
    float *__restrict__ q, const float *__restrict__ w, float gamma,
    const double *__restrict__ rz_cur, const double *__restrict__ rz_prev,
    const double *__restrict__ p_rr, const double *__restrict__ p_bb,
    double *__restrict__ p_pq, PcgStatus *__restrict__ stat, int it, double tol, int nx, int ny,
    int nblk)
{
    const int m = blockIdx.y;
    if (pcg_over(stat + m, 2u * (unsigned)it)) return;
    const I N = (I)nx * (I)ny;
    const float *zm = z + (size_t)m * N, *pm = pold + (size_t)m * N;
    Pix<I> px[kPix];
    PairW e[kPix];
    float zc[kPix][5], pc[kPix][5];
#pragma unroll
    for (int j = 0; j < kPix; ++j) {
        px[j] = pixel_at<I>(j, nx, ny, N);
        e[j] = pair_weights(px[j], w, w + N);
        const I at[5] = {px[j].i, px[j].r, px[j].l, px[j].d, px[j].u};
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            zc[j][k] = zm[at[k]];
            pc[j][k] = pm[at[k]];
        }
    }
    const size_t mb = (size_t)m * nblk;
    double beta_d = 0.0;
    if (!pcg_begin(rz_cur + mb, rz_prev + mb, p_rr + mb, p_bb + mb, nblk, it, tol, stat + m,
                   beta_d))
        return;
    const float beta = (float)beta_d;
    double v[1] = {0.0};
#pragma unroll
    for (int j = 0; j < kPix; ++j) {
        if (!px[j].in) continue;
        const float pi = zc[j][0] + beta * pc[j][0];
        float lp = 0.f;
        lp += e[j].r * (pi - (zc[j][1] + beta * pc[j][1]));
        lp += e[j].l * (pi - (zc[j][2] + beta * pc[j][2]));
        lp += e[j].d * (pi - (zc[j][3] + beta * pc[j][3]));
        lp += e[j].u * (pi - (zc[j][4] + beta * pc[j][4]));
        const float qi = pi + gamma * lp;
        pnew[(size_t)m * N + px[j].i] = pi;
        q[(size_t)m * N + px[j].i] = qi;
        v[0] += (double)pi * qi;
    }
    __shared__ double out[1];
    block_sum<1>(v, out);
    if (threadIdx.x == 0) p_pq[mb + blockIdx.x] = out[0];
}

// Part B: a = rz / <p, q>, u += a p, res -= a q, z = M^{-1} res; partials of
// the next <res, z> and |res|^2.
__global__ __launch_bounds__(256) void k_pcg_b(
    float *__restrict__ u1, float *__restrict__ u2, float *__restrict__ res,
    float *__restrict__ z, const float *__restrict__ pnew, const float *__restrict__ q,
    const float *__restrict__ minv, const double *__restrict__ rz_cur,
    const double *__restrict__ p_pq, double *__restrict__ rz_next, double *__restrict__ p_rr,
    PcgStatus *__restrict__ stat, int it, int nx, int ny, int nblk)
{
    const int m = blockIdx.y;
    const unsigned launch = 2u * (unsigned)it + 1u;
    if (pcg_over(stat + m, launch)) return;
    const size_t N = (size_t)nx * ny;
    float *um = m == 0 ? u1 : u2;
    size_t at[kPix];
    float uc[kPix], pc[kPix], rc[kPix], qc[kPix], mc[kPix];
#pragma unroll
    for (int j = 0; j < kPix; ++j) {
        const size_t i = ((size_t)blockIdx.x * kPix + j) * 256 + threadIdx.x;
        at[j] = i < N ? i : N - 1;
        uc[j] = um[at[j]];
        pc[j] = pnew[m * N + at[j]];
        rc[j] = res[m * N + at[j]];
        qc[j] = q[m * N + at[j]];
        mc[j] = minv[at[j]];
    }
    const double *const arr[2] = {p_pq + (size_t)m * nblk, rz_cur + (size_t)m * nblk};
    double sum[2];
    reduce_arrays<2>(arr, nblk, sum);
    if (!(sum[0] > 0.0)) {  // breakdown: stop with the current iterate
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            stat[m].done = 2;
            stat[m].since = launch + 1u;
        }
        return;
    }
    const float a = (float)(sum[1] / sum[0]);
    double v[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < kPix; ++j) {
        if (((size_t)blockIdx.x * kPix + j) * 256 + threadIdx.x >= N) continue;
        um[at[j]] = uc[j] + a * pc[j];
        const float rs = rc[j] - a * qc[j];
        const float zz = mc[j] * rs;
        res[m * N + at[j]] = rs;
        z[m * N + at[j]] = zz;
        v[0] += (double)rs * zz;
        v[1] += (double)rs * rs;
    }
    __shared__ double out[2];
    block_sum<2>(v, out);
    if (threadIdx.x == 0) {
        rz_next[(size_t)m * nblk + blockIdx.x] = out[0];
        p_rr[(size_t)m * nblk + blockIdx.x] = out[1];
    }
}

// After the last iteration: final residual of materials still running.
__global__ __launch_bounds__(256) void k_pcg_final(const double *__restrict__ p_rr,
                                                   const double *__restrict__ p_bb,
                                                   PcgStatus *__restrict__ stat, int iters,
                                                   double tol, int nblk)
{
    const int m = blockIdx.x;
    if (stat[m].done) return;
    const double *const arr[2] = {p_rr + (size_t)m * nblk, p_bb + (size_t)m * nblk};
    double sum[2];
    reduce_arrays<2>(arr, nblk, sum);
    if (threadIdx.x != 0) return;
    const double rr = sum[0], bb = sum[1];
    const double bn = bb > 0.0 ? sqrt(bb) : 1.0;
    const double rn = bb > 0.0 ? sqrt(rr) : 0.0;
    stat[m].iters = iters;
    stat[m].relres = rn / bn;
    stat[m].done = rn <= tol * bn ? 1 : 3;  // 3: stopped at the cap
}

// ---------------------------------------------- attenuation-space PLS ---
// (D^T D (x) I + gamma I (x) L) u = D^T x (|x - Du|^2 + gamma R(u)): both
// materials of a pixel in one thread, so the per-pixel 2 x 2 coupling D^T D
// and the block-Jacobi preconditioner (D^T D + gamma diag(L)) apply in place;
// joint scalars over both materials.  D^T D has the condition number of D
// squared (~740 for water and bone), so vectors and arithmetic are FP64.
struct AttCoef {
    double g11, g12, g22;       // D^T D
    double e1h, e2h, e1l, e2l;  // D
};

// z = P^{-1} res at one pixel, P = D^T D + gamma diag(L) I.
__device__ __forceinline__ void att_precond(const AttCoef &k, double gamma, double d,
                                            const double (&rs)[2], double (&z)[2])
{
    const double a11 = k.g11 + gamma * d, a22 = k.g22 + gamma * d;
    const double dt = a11 * a22 - k.g12 * k.g12;
    z[0] = (a22 * rs[0] - k.g12 * rs[1]) / dt;
    z[1] = (a11 * rs[1] - k.g12 * rs[0]) / dt;
}

// (gamma L v) + D^T D v at a pixel from both materials' values at it and its
// neighbours (c[m][k], k = 0 the pixel, then right, left, below, above).
__device__ __forceinline__ void att_apply(const double (&c)[2][5], const PairW &e,
                                          const AttCoef &k, double gamma, double (&out)[2])
{
    double lv[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        double l = 0.0;
        l += (double)e.r * (c[m][0] - c[m][1]);
        l += (double)e.l * (c[m][0] - c[m][2]);
        l += (double)e.d * (c[m][0] - c[m][3]);
        l += (double)e.u * (c[m][0] - c[m][4]);
        lv[m] = l;
    }
    const double a = c[0][0], b = c[1][0];
    out[0] = k.g11 * a + k.g12 * b + gamma * lv[0];
    out[1] = k.g12 * a + k.g22 * b + gamma * lv[1];
}

// Setup from u = D^{-1} x (u1, u2): u64 = u, res = D^T x - A u, z = P^{-1} res,
// p_old = 0; partials <res, z>, |res|^2, |D^T x|^2 in slot 0.
template <typename I>
__global__ __launch_bounds__(256) void k_apcg_setup(
    const float *__restrict__ xh, const float *__restrict__ xl, const float *__restrict__ u1,
    const float *__restrict__ u2, const float *__restrict__ w, double gamma, AttCoef k,
    double *__restrict__ u, double *__restrict__ res, double *__restrict__ z,
    double *__restrict__ pold, double *__restrict__ p_rz, double *__restrict__ p_rr,
    double *__restrict__ p_bb, PcgStatus *__restrict__ stat, int nx, int ny)
{
    const I N = (I)nx * (I)ny;
    const float *const um[2] = {u1, u2};
    double v[3] = {0.0, 0.0, 0.0};
    for (int j = 0; j < kPix; ++j) {
        const Pix<I> px = pixel_at<I>(j, nx, ny, N);
        const PairW e = pair_weights(px, w, w + N);
        const I at[5] = {px.i, px.r, px.l, px.d, px.u};
        double c[2][5];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int t = 0; t < 5; ++t) c[m][t] = um[m][at[t]];
        const double h = xh[px.i], l = xl[px.i];
        if (!px.in) continue;
        const size_t i = px.i;
        const double c0 = k.e1h * h + k.e1l * l, c1 = k.e2h * h + k.e2l * l;
        double au[2], zz[2];
        att_apply(c, e, k, gamma, au);
        double rs[2] = {c0 - au[0], c1 - au[1]};
        att_precond(k, gamma, (double)weight_sum(e), rs, zz);
        u[i] = c[0][0];
        u[N + i] = c[1][0];
        res[i] = rs[0];
        res[N + i] = rs[1];
        z[i] = zz[0];
        z[N + i] = zz[1];
        pold[i] = 0.0;
        pold[N + i] = 0.0;
        v[0] += rs[0] * zz[0] + rs[1] * zz[1];
        v[1] += rs[0] * rs[0] + rs[1] * rs[1];
        v[2] += c0 * c0 + c1 * c1;
    }
    __shared__ double out[3];
    block_sum<3>(v, out);
    if (threadIdx.x == 0) {
        p_rz[blockIdx.x] = out[0];
        p_rr[blockIdx.x] = out[1];
        p_bb[blockIdx.x] = out[2];
        if (blockIdx.x == 0) {
            stat[0].done = 0;
            stat[0].iters = 0;
            stat[0].relres = 0.0;
            stat[0].since = 0;
        }
    }
}

// Part A: convergence test, beta, p_new = z + beta p_old, q = A p_new, partial
// <p_new, q>.  One kernel (the neighbours' p_new are formed again from z and
// p_old) in place of one for p and one for q: with the loads as above, 500
// iterations at 512 x 512 take 9.6 ms in place of 14.7.
template <typename I>
__global__ __launch_bounds__(256) void k_apcg_a(
    const double *__restrict__ z, const double *__restrict__ pold, double *__restrict__ pnew,
    double *__restrict__ q, const float *__restrict__ w, double gamma, AttCoef k,
    const double *__restrict__ rz_cur, const double *__restrict__ rz_prev,
    const double *__restrict__ p_rr, const double *__restrict__ p_bb, double *__restrict__ p_pq,
    PcgStatus *__restrict__ stat, int it, double tol, int nx, int ny, int nblk)
{
    if (pcg_over(stat, 2u * (unsigned)it)) return;
    const I N = (I)nx * (I)ny;
    double beta = 0.0;
    if (!pcg_begin(rz_cur, rz_prev, p_rr, p_bb, nblk, it, tol, stat, beta)) return;
    double v[1] = {0.0};
    for (int j = 0; j < kPix; ++j) {
        const Pix<I> px = pixel_at<I>(j, nx, ny, N);
        const PairW e = pair_weights(px, w, w + N);
        const I at[5] = {px.i, px.r, px.l, px.d, px.u};
        double zc[2][5], c[2][5];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                zc[m][t] = z[(size_t)m * N + at[t]];
                c[m][t] = pold[(size_t)m * N + at[t]];
            }
        if (!px.in) continue;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int t = 0; t < 5; ++t) c[m][t] = zc[m][t] + beta * c[m][t];
        double qq[2];
        att_apply(c, e, k, gamma, qq);
        const size_t i = px.i;
        pnew[i] = c[0][0];
        pnew[N + i] = c[1][0];
        q[i] = qq[0];
        q[N + i] = qq[1];
        v[0] += c[0][0] * qq[0] + c[1][0] * qq[1];
    }
    __shared__ double out[1];
    block_sum<1>(v, out);
    if (threadIdx.x == 0) p_pq[blockIdx.x] = out[0];
}

// Part B: a = rz / <p, q>, u += a p, res -= a q, z = P^{-1} res; partials of
// the next <res, z> and |res|^2.
template <typename I>
__global__ __launch_bounds__(256) void k_apcg_b(
    double *__restrict__ u, double *__restrict__ res, double *__restrict__ z,
    const double *__restrict__ pnew, const double *__restrict__ q, const float *__restrict__ w,
    double gamma, AttCoef k, const double *__restrict__ rz_cur, const double *__restrict__ p_pq,
    double *__restrict__ rz_next, double *__restrict__ p_rr, PcgStatus *__restrict__ stat,
    int it, int nx, int ny, int nblk)
{
    const unsigned launch = 2u * (unsigned)it + 1u;
    if (pcg_over(stat, launch)) return;
    const double *const arr[2] = {p_pq, rz_cur};
    double sum[2];
    reduce_arrays<2>(arr, nblk, sum);
    if (!(sum[0] > 0.0)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            stat[0].done = 2;
            stat[0].since = launch + 1u;
        }
        return;
    }
    const double a = sum[1] / sum[0];
    const I N = (I)nx * (I)ny;
    double v[2] = {0.0, 0.0};
    for (int j = 0; j < kPix; ++j) {
        const Pix<I> px = pixel_at<I>(j, nx, ny, N);
        const PairW e = pair_weights(px, w, w + N);
        const size_t i = px.i;
        double uc[2], pc[2], rs[2], qc[2], zz[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            uc[m] = u[(size_t)m * N + i];
            pc[m] = pnew[(size_t)m * N + i];
            rs[m] = res[(size_t)m * N + i];
            qc[m] = q[(size_t)m * N + i];
        }
        if (!px.in) continue;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            u[(size_t)m * N + i] = uc[m] + a * pc[m];
            rs[m] -= a * qc[m];
        }
        att_precond(k, gamma, (double)weight_sum(e), rs, zz);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            res[(size_t)m * N + i] = rs[m];
            z[(size_t)m * N + i] = zz[m];
        }
        v[0] += rs[0] * zz[0] + rs[1] * zz[1];
        v[1] += rs[0] * rs[0] + rs[1] * rs[1];
    }
    __shared__ double out[2];
    block_sum<2>(v, out);
    if (threadIdx.x == 0) {
        rz_next[blockIdx.x] = out[0];
        p_rr[blockIdx.x] = out[1];
    }
}

__global__ __launch_bounds__(256) void k_apcg_out(const double *__restrict__ u,
                                                  float *__restrict__ u1, float *__restrict__ u2,
                                                  size_t N)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    u1[i] = (float)u[i];
    u2[i] = (float)u[N + i];
}

struct PlsWork {
    DevBuf b, res, z, p0, p1, q, minv, w, m2, pmax, prz0, prz1, prr, pbb, ppq, stat, u64;
    StreamOrder order;
};

// Device buffers of one image-space decomposition of N pixels (nblk
// reduction blocks): D^{-1} x (both materials), PCG vectors, the Jacobi
// inverse, edge weights and the Prewitt map, per-block partial sums.
struct PlsBufs {
    float *b, *res, *z, *p0, *p1, *q, *minv, *w, *m2, *pmax;
    double *prz0, *prz1, *prr, *pbb, *ppq;
    PcgStatus *stat;
};

std::mutex g_pls_mu;
std::vector<std::pair<int, std::unique_ptr<PlsWork>>> g_pls;

PlsWork *pls_work()
{
    int dev = 0;
    (void)hipGetDevice(&dev);
    for (auto &p : g_pls)
        if (p.first == dev) return p.second.get();
    g_pls.emplace_back(dev, std::make_unique<PlsWork>());
    return g_pls.back().second.get();
}

dect_status edges_run(int nx, int ny, const float *x, double tau, double eps, float *w,
                      float *m2, float *pmax, hipStream_t s)
{
    const size_t N = (size_t)nx * ny;
    const int nblk = (int)((N + 256 * kPix - 1) / (256 * kPix));
    hipLaunchKernelGGL(k_prewitt, dim3(nblk), dim3(256), 0, s, x, m2, pmax, nx, ny);
    DECT_HIP(hipGetLastError());
    const float tau2 = (float)(tau * tau);
    hipLaunchKernelGGL(k_weights, dim3(nblk), dim3(256), 0, s, (const float *)m2,
                       (const float *)pmax, nblk, tau2, (float)eps, w, nx, ny);
    DECT_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status edges_into(int nx, int ny, const float *x, double tau, double eps, float *w,
                       PlsWork *W, hipStream_t s)
{
    const size_t N = (size_t)nx * ny;
    const int nblk = (int)((N + 256 * kPix - 1) / (256 * kPix));
    dect_status st;
    if ((st = W->m2.ensure(N * 4)) || (st = W->pmax.ensure((size_t)nblk * 4))) return st;
    return edges_run(nx, ny, x, tau, eps, w, (float *)W->m2.ptr, (float *)W->pmax.ptr, s);
}

dect_status check_pls_args(int nx, int ny, const float *xh, const float *xl,
                           const dect_pls_params *P, float *u1, float *u2, const char *who)
{
    if (nx <= 0 || ny <= 0 || !xh || !xl || !P || !u1 || !u2)
        return fail(DECT_ERR_INVALID_ARG, std::string(who) + ": bad size or null argument");
    const double det = P->eta_water_high * P->eta_bone_low - P->eta_bone_high * P->eta_water_low;
    if (!std::isfinite(det) || det == 0.0)
        return fail(DECT_ERR_INVALID_ARG, std::string(who) + ": singular decomposition matrix");
    if (!(P->gamma >= 0.0) || !std::isfinite(P->gamma) || P->max_iter < 0 || !(P->tol >= 0.0))
        return fail(DECT_ERR_INVALID_ARG, std::string(who) + ": bad gamma/max_iter/tol");
    if (P->mode != DECT_PLS_IMAGE && P->mode != DECT_PLS_ATTENUATION)
        return fail(DECT_ERR_INVALID_ARG, std::string(who) + ": unknown mode");
    return DECT_OK;
}

// D^{-1} x into u1, u2 and B.b (both materials).
void dinv_run(int nx, int ny, const float *xh, const float *xl, const dect_pls_params *P,
              float *u1, float *u2, float *b, hipStream_t s)
{
    const size_t N = (size_t)nx * ny;
    const double det = P->eta_water_high * P->eta_bone_low - P->eta_bone_high * P->eta_water_low;
    PlsCoef c;
    c.i11 = (float)(P->eta_bone_low / det);
    c.i12 = (float)(-P->eta_bone_high / det);
    c.i21 = (float)(-P->eta_water_low / det);
    c.i22 = (float)(P->eta_water_high / det);
    hipLaunchKernelGGL(k_dinv, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, xh, xl, c, u1,
                       u2, b, N);
}

// Jacobi-PCG of the image-space system (I + gamma L) u_m = b_m for both
// materials, from u = b (already in u1, u2), on the pair weights w.
dect_status pcg_image_run(int nx, int ny, const dect_pls_params *P, const float *w, float *u1,
                          float *u2, dect_report *rep, const PlsBufs &B, hipStream_t s)
{
    const size_t N = (size_t)nx * ny;
    const int nblk = (int)((N + 256 * kPix - 1) / (256 * kPix));
    const float gamma = (float)P->gamma;
    PcgStatus *stat = B.stat;
    float *pbuf[2] = {B.p0, B.p1};
    double *rzb[2] = {B.prz0, B.prz1};
    // 32-bit pixel indices where the image allows them
    const bool small = small_index(N);
    const auto setup = small ? k_pcg_setup<unsigned> : k_pcg_setup<size_t>;
    const auto part_a = small ? k_pcg_a<unsigned> : k_pcg_a<size_t>;
    hipLaunchKernelGGL(setup, dim3(nblk, 2), dim3(256), 0, s, (const float *)B.b, w, gamma,
                       B.res, B.z, pbuf[0], B.minv, rzb[0], B.prr, B.pbb, stat, nx, ny, nblk);
    DECT_HIP(hipGetLastError());
    int it = 0;
    const int check_every = 16;
    for (; it < P->max_iter; ++it) {
        float *pold = pbuf[it & 1], *pnew = pbuf[(it + 1) & 1];
        const double *rz_prev = rzb[(it + 1) & 1];
        hipLaunchKernelGGL(part_a, dim3(nblk, 2), dim3(256), 0, s, (const float *)B.z,
                           (const float *)pold, pnew, B.q, w, gamma, (const double *)rzb[it & 1],
                           rz_prev, (const double *)B.prr, (const double *)B.pbb, B.ppq, stat, it,
                           P->tol, nx, ny, nblk);
        DECT_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_pcg_b, dim3(nblk, 2), dim3(256), 0, s, u1, u2, B.res, B.z,
                           (const float *)pnew, (const float *)B.q, (const float *)B.minv,
                           (const double *)rzb[it & 1], (const double *)B.ppq, rzb[(it + 1) & 1],
                           B.prr, stat, it, nx, ny, nblk);
        DECT_HIP(hipGetLastError());
        if ((it + 1) % check_every == 0) {
            PcgStatus hs[2];
            DECT_HIP(hipMemcpyAsync(hs, stat, sizeof(hs), hipMemcpyDeviceToHost, s));
            DECT_HIP(hipStreamSynchronize(s));
            if (hs[0].done && hs[1].done) {
                ++it;
                break;
            }
        }
    }
    hipLaunchKernelGGL(k_pcg_final, dim3(2), dim3(256), 0, s, (const double *)B.prr,
                       (const double *)B.pbb, stat, it, P->tol, nblk);
    DECT_HIP(hipGetLastError());
    if (rep) {
        PcgStatus hs[2];
        DECT_HIP(hipMemcpyAsync(hs, stat, sizeof(hs), hipMemcpyDeviceToHost, s));
        DECT_HIP(hipStreamSynchronize(s));
        rep->iters = std::max(hs[0].iters, hs[1].iters);
        rep->pcg_residual = std::max(hs[0].relres, hs[1].relres);
        rep->objective = 0.0;
        rep->rel_change = 0.0;
        rep->status = (hs[0].done == 3 || hs[1].done == 3) ? DECT_WARN_MAXITER : DECT_OK;
        if (rep->status == DECT_WARN_MAXITER) {
            set_error("dect_pls_decompose: PCG reached max_iter above tolerance");
            return DECT_WARN_MAXITER;
        }
    }
    return DECT_OK;
}

}  // namespace

dect_status pls_edge_weights(int nx, int ny, const float *x, double tau, double eps, float *w,
                             hipStream_t s)
{
    if (nx <= 0 || ny <= 0 || !x || !w)
        return fail(DECT_ERR_INVALID_ARG, "dect_pls_edge_weights: bad size or null buffer");
    if (!(tau >= 0.0) || !std::isfinite(tau) || !std::isfinite(eps))
        return fail(DECT_ERR_INVALID_ARG, "dect_pls_edge_weights: bad tau/eps");
    std::lock_guard<std::mutex> lk(g_pls_mu);
    PlsWork *W = pls_work();
    StreamOrder::Call call(W->order, s);
    if (call.status()) return call.status();
    return edges_into(nx, ny, x, tau, eps, w, W, s);
}

// The image-space work buffers of N pixels in nblk reduction blocks.
static dect_status pls_prepare(PlsWork *W, size_t N, int nblk)
{
    dect_status st;
    if ((st = W->b.ensure(2 * N * 4)) || (st = W->res.ensure(2 * N * 4)) ||
        (st = W->z.ensure(2 * N * 4)) || (st = W->p0.ensure(2 * N * 4)) ||
        (st = W->p1.ensure(2 * N * 4)) || (st = W->q.ensure(2 * N * 4)) ||
        (st = W->minv.ensure(N * 4)) || (st = W->prz0.ensure((size_t)2 * nblk * 8)) ||
        (st = W->prz1.ensure((size_t)2 * nblk * 8)) || (st = W->prr.ensure((size_t)2 * nblk * 8)) ||
        (st = W->pbb.ensure((size_t)2 * nblk * 8)) || (st = W->ppq.ensure((size_t)2 * nblk * 8)) ||
        (st = W->stat.ensure(2 * sizeof(PcgStatus))))
        return st;
    return DECT_OK;
}

// The FP64 vectors of the attenuation-space solve (they replace the FP32
// ones of the same names).
static dect_status pls_prepare_att(PlsWork *W, size_t N)
{
    dect_status st;
    if ((st = W->u64.ensure(2 * N * 8)) || (st = W->res.ensure(2 * N * 8)) ||
        (st = W->z.ensure(2 * N * 8)) || (st = W->p0.ensure(2 * N * 8)) ||
        (st = W->p1.ensure(2 * N * 8)) || (st = W->q.ensure(2 * N * 8)))
        return st;
    return DECT_OK;
}

// The work buffers of a decomposition of N pixels in both modes with the
// edges detected, in the order the calls allocate them (image mode first),
// for a dry run under a SizingScope.
dect_status pls_size_run(size_t N)
{
    const int nblk = (int)((N + 256 * kPix - 1) / (256 * kPix));
    PlsWork W;
    dect_status st;
    if ((st = pls_prepare(&W, N, nblk)) || (st = W.w.ensure(2 * N * 4)) ||
        (st = W.m2.ensure(N * 4)) || (st = W.pmax.ensure((size_t)nblk * 4)) ||
        (st = pls_prepare_att(&W, N)))
        return st;
    return DECT_OK;
}

// The attenuation-space system, from u = D^{-1} x already in u1, u2.
dect_status pls_attenuation(int nx, int ny, const float *xh, const float *xl,
                            const dect_pls_params *P, const float *w, float *u1, float *u2,
                            dect_report *rep, PlsWork *W, int nblk, hipStream_t s)
{
    const size_t N = (size_t)nx * ny;
    dect_status st;
    if ((st = pls_prepare_att(W, N))) return st;
    AttCoef k;
    k.e1h = P->eta_water_high;
    k.e2h = P->eta_bone_high;
    k.e1l = P->eta_water_low;
    k.e2l = P->eta_bone_low;
    k.g11 = k.e1h * k.e1h + k.e1l * k.e1l;
    k.g12 = k.e1h * k.e2h + k.e1l * k.e2l;
    k.g22 = k.e2h * k.e2h + k.e2l * k.e2l;
    const double gamma = P->gamma;
    PcgStatus *stat = (PcgStatus *)W->stat.ptr;
    double *u = (double *)W->u64.ptr, *res = (double *)W->res.ptr, *z = (double *)W->z.ptr;
    double *q = (double *)W->q.ptr;
    double *pbuf[2] = {(double *)W->p0.ptr, (double *)W->p1.ptr};
    double *rzb[2] = {(double *)W->prz0.ptr, (double *)W->prz1.ptr};
    const bool small = small_index(N);  // 32-bit pixel indices where the image allows them
    const auto setup = small ? k_apcg_setup<unsigned> : k_apcg_setup<size_t>;
    const auto part_a = small ? k_apcg_a<unsigned> : k_apcg_a<size_t>;
    const auto part_b = small ? k_apcg_b<unsigned> : k_apcg_b<size_t>;
    hipLaunchKernelGGL(setup, dim3(nblk), dim3(256), 0, s, xh, xl, (const float *)u1,
                       (const float *)u2, w, gamma, k, u, res, z, pbuf[0], rzb[0],
                       (double *)W->prr.ptr, (double *)W->pbb.ptr, stat, nx, ny);
    DECT_HIP(hipGetLastError());
    int it = 0;
    const int check_every = 16;
    for (; it < P->max_iter; ++it) {
        const double *pold = pbuf[it & 1];
        double *pnew = pbuf[(it + 1) & 1];
        hipLaunchKernelGGL(part_a, dim3(nblk), dim3(256), 0, s, (const double *)z, pold, pnew, q,
                           w, gamma, k, (const double *)rzb[it & 1],
                           (const double *)rzb[(it + 1) & 1], (const double *)W->prr.ptr,
                           (const double *)W->pbb.ptr, (double *)W->ppq.ptr, stat, it, P->tol, nx,
                           ny, nblk);
        DECT_HIP(hipGetLastError());
        hipLaunchKernelGGL(part_b, dim3(nblk), dim3(256), 0, s, u, res, z, (const double *)pnew,
                           (const double *)q, w, gamma, k, (const double *)rzb[it & 1],
                           (const double *)W->ppq.ptr, rzb[(it + 1) & 1], (double *)W->prr.ptr,
                           stat, it, nx, ny, nblk);
        DECT_HIP(hipGetLastError());
        if ((it + 1) % check_every == 0) {
            PcgStatus hs;
            DECT_HIP(hipMemcpyAsync(&hs, stat, sizeof(hs), hipMemcpyDeviceToHost, s));
            DECT_HIP(hipStreamSynchronize(s));
            if (hs.done) {
                ++it;
                break;
            }
        }
    }
    hipLaunchKernelGGL(k_pcg_final, dim3(1), dim3(256), 0, s, (const double *)W->prr.ptr,
                       (const double *)W->pbb.ptr, stat, it, P->tol, nblk);
    DECT_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_apcg_out, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s,
                       (const double *)u, u1, u2, N);
    DECT_HIP(hipGetLastError());
    if (rep) {
        PcgStatus hs;
        DECT_HIP(hipMemcpyAsync(&hs, stat, sizeof(hs), hipMemcpyDeviceToHost, s));
        DECT_HIP(hipStreamSynchronize(s));
        rep->iters = hs.iters;
        rep->pcg_residual = hs.relres;
        rep->objective = 0.0;
        rep->rel_change = 0.0;
        rep->status = hs.done == 3 ? DECT_WARN_MAXITER : DECT_OK;
        if (rep->status == DECT_WARN_MAXITER) {
            set_error("dect_pls_decompose: PCG reached max_iter above tolerance");
            return DECT_WARN_MAXITER;
        }
    }
    return DECT_OK;
}

dect_status pls_decompose(int nx, int ny, const float *xh, const float *xl,
                          const dect_pls_params *P, const float *ew, float *u1, float *u2,
                          dect_report *rep, hipStream_t s)
{
    dect_status st = check_pls_args(nx, ny, xh, xl, P, u1, u2, "dect_pls_decompose");
    if (st) return st;
    std::lock_guard<std::mutex> lk(g_pls_mu);
    PlsWork *W = pls_work();
    StreamOrder::Call call(W->order, s);
    if ((st = call.status())) return st;
    const size_t N = (size_t)nx * ny;
    const int nblk = (int)((N + 256 * kPix - 1) / (256 * kPix));
    if ((st = pls_prepare(W, N, nblk))) return st;
    dinv_run(nx, ny, xh, xl, P, u1, u2, (float *)W->b.ptr, s);
    DECT_HIP(hipGetLastError());
    const float *w = ew;
    if (!w) {
        if ((st = W->w.ensure(2 * N * 4))) return st;
        if ((st = edges_into(nx, ny, xl, P->edge_tau, P->edge_eps, (float *)W->w.ptr, W, s)))
            return st;
        w = (const float *)W->w.ptr;
    }
    // a report waits for the call's work
    auto finish = [&](dect_status run) {
        if (rep && (run == DECT_OK || run == DECT_WARN_MAXITER)) call.done();
        return run;
    };
    if (P->mode == DECT_PLS_ATTENUATION)
        return finish(pls_attenuation(nx, ny, xh, xl, P, w, u1, u2, rep, W, nblk, s));
    PlsBufs B;
    B.b = (float *)W->b.ptr;
    B.res = (float *)W->res.ptr;
    B.z = (float *)W->z.ptr;
    B.p0 = (float *)W->p0.ptr;
    B.p1 = (float *)W->p1.ptr;
    B.q = (float *)W->q.ptr;
    B.minv = (float *)W->minv.ptr;
    B.w = nullptr;
    B.m2 = nullptr;
    B.pmax = nullptr;
    B.prz0 = (double *)W->prz0.ptr;
    B.prz1 = (double *)W->prz1.ptr;
    B.prr = (double *)W->prr.ptr;
    B.pbb = (double *)W->pbb.ptr;
    B.ppq = (double *)W->ppq.ptr;
    B.stat = (PcgStatus *)W->stat.ptr;
    return finish(pcg_image_run(nx, ny, P, w, u1, u2, rep, B, s));
}

// ------------------------------------------------ allocation-free form ---
// The work memory of dect_pls_decompose_noalloc: one array per GPU, in the
// code object, sized for kNoAllocMaxPixels pixels.  Host code never passes
// its name to a kernel (on the host the name is not the device address):
// hipGetSymbolAddress gives each device's address once, kept in g_scratch.
constexpr size_t kNoAllocMaxPixels = (size_t)512 * 512;
constexpr size_t kNoAllocBlocks = (kNoAllocMaxPixels + 256 * kPix - 1) / (256 * kPix);
constexpr size_t kScratchBytes =
    16 * 4 * kNoAllocMaxPixels + 10 * 8 * kNoAllocBlocks + 4 * kNoAllocBlocks + (size_t)64 * 1024;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

std::mutex g_scratch_mu;
std::vector<void *> g_scratch;  // per device id: the array's device address

dect_status scratch_ptr(void **out)
{
    int dev = 0;
    DECT_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch.size() <= dev) g_scratch.resize((size_t)dev + 1, nullptr);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(DECT_ERR_HIP, std::string("dect_pls_decompose_noalloc: scratch address: ") +
                                          hipGetErrorString(e));
        g_scratch[dev] = p;
    }
    *out = g_scratch[dev];
    return DECT_OK;
}

// Consecutive 256-byte-aligned pieces of one buffer.
struct Carve {
    unsigned char *base;
    size_t off;
    template <class T>
    T *take(size_t n)
    {
        off = (off + 255) & ~(size_t)255;
        T *p = (T *)(base + off);
        off += n * sizeof(T);
        return p;
    }
};

}  // namespace

dect_status pls_decompose_noalloc(int nx, int ny, const float *xh, const float *xl,
                                  const dect_pls_params *P, const float *ew, float *u1,
                                  float *u2, dect_report *rep, hipStream_t s)
{
    dect_status st = check_pls_args(nx, ny, xh, xl, P, u1, u2, "dect_pls_decompose_noalloc");
    if (st) return st;
    if (P->mode != DECT_PLS_IMAGE)
        return fail(DECT_ERR_INVALID_ARG,
                    "dect_pls_decompose_noalloc: image-space mode (DECT_PLS_IMAGE) only");
    const size_t N = (size_t)nx * ny;
    if (N > kNoAllocMaxPixels)
        return fail(DECT_ERR_INVALID_ARG, "dect_pls_decompose_noalloc: at most " +
                                              std::to_string(kNoAllocMaxPixels) +
                                              " pixels, got " + std::to_string(N));
    void *sp = nullptr;
    if ((st = scratch_ptr(&sp))) return st;
    const size_t nblk = (N + 256 * kPix - 1) / (256 * kPix);
    Carve c{(unsigned char *)sp, 0};
    PlsBufs B;
    B.b = c.take<float>(2 * N);
    B.res = c.take<float>(2 * N);
    B.z = c.take<float>(2 * N);
    B.p0 = c.take<float>(2 * N);
    B.p1 = c.take<float>(2 * N);
    B.q = c.take<float>(2 * N);
    B.minv = c.take<float>(N);
    B.w = c.take<float>(2 * N);
    B.m2 = c.take<float>(N);
    B.pmax = c.take<float>(nblk);
    B.prz0 = c.take<double>(2 * nblk);
    B.prz1 = c.take<double>(2 * nblk);
    B.prr = c.take<double>(2 * nblk);
    B.pbb = c.take<double>(2 * nblk);
    B.ppq = c.take<double>(2 * nblk);
    B.stat = c.take<PcgStatus>(2);
    if (c.off > kScratchBytes)
        return fail(DECT_ERR_INVALID_ARG, "dect_pls_decompose_noalloc: scratch too small");
    dinv_run(nx, ny, xh, xl, P, u1, u2, B.b, s);
    DECT_HIP(hipGetLastError());
    const float *w = ew;
    if (!w) {
        if ((st = edges_run(nx, ny, xl, P->edge_tau, P->edge_eps, B.w, B.m2, B.pmax, s)))
            return st;
        w = B.w;
    }
    return pcg_image_run(nx, ny, P, w, u1, u2, rep, B, s);
}

void release_pls_work()
{
    std::lock_guard<std::mutex> lk(g_pls_mu);
    g_pls.clear();
}

}  // namespace dect
