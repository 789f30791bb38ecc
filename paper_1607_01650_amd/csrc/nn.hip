// BF16 MFMA convolution kernels (gfx950) and the small kernels of the U-Net
// that maps an early ADM iterate to a late one (learned warm start).
//
// Tensors are NHWC, activations and weights BF16, accumulation FP32 on the
// matrix cores (v_mfma_f32_16x16x32_bf16).  Convolutions are implicit GEMMs:
//   forward / dgrad : D[pixel][co] = sum_k A[pixel][k] B[k][co], k = (tap, ci)
//   wgrad           : D[co][ci]    = sum_p dZ[p][co] X[p + tap][ci] per tap
// dgrad is the forward kernel run on dZ with taps flipped and channels
// transposed; a 2x2 stride-2 transposed convolution is a 1x1 convolution to
// 4*Cout channels followed by depth-to-space.  Every reduction that crosses
// blocks goes through per-block partials summed in a fixed order.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <map>
#include <mutex>
#include <tuple>

#include "../../include/dect_nn.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16;

thread_local const char *g_nn_err = "";

dect_status nn_fail(dect_status st, const char *msg)
{
    g_nn_err = msg;
    return st;
}

#define NN_HIP(expr)                                                        \
    do {                                                                    \
        hipError_t e_ = (expr);                                             \
        if (e_ != hipSuccess) return nn_fail(DECT_ERR_HIP, hipGetErrorString(e_)); \
    } while (0)

__device__ __forceinline__ float bf2f(u16 v) { return __uint_as_float((uint32_t)v << 16); }

// float -> bf16, round to nearest even (NaN kept quiet)
__device__ __forceinline__ u16 f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u16)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (u16)(u >> 16);
}

union Frag {
    bf16x8 v;
    uint4 u;
};


// The thread's index, opaque to the compiler: addresses made from it are worked
// out again at each use, not kept in registers across a loop (which spills).
__device__ __forceinline__ int opaque_tid()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// ------------------------------------------------------------ conv fwd ---
// Block: 256 threads = 4 waves on a tile of TR x 32 output pixels of one
// image (TR = 2 MT).  Wave w owns the MT pixel tiles j = w MT .. w MT + MT - 1
// (tile j: row j / 2, columns 16 (j % 2) .. + 15) and every output-channel
// tile, so each weight fragment it loads feeds MT matrix-core steps.  The
// input window (TR + 2 rows x 34 columns with the halo for 3x3, TR x 32 for
// 1x1) is staged in LDS, at most 64 channels at a time, with 16-byte loads;
// the output tile goes back through LDS and leaves as 16-byte stores.
// X [N][H][W][Cin], Wk [taps][CoutP][Cin] (CoutP = 16 NT, zero padded),
// bias [CoutP] or null, Y [N][H][W][Cout] as bf16 or f32.
constexpr int kConvLds = 49152;  // bytes: max(window chunk, output tile)
constexpr int kConvChunk = 64;   // channels staged at a time

constexpr int conv_mt(int nt) { return nt <= 6 ? 4 : (nt <= 12 ? 2 : 1); }
static_assert(2 * conv_mt(6) * 32 * 96 * 2 <= kConvLds && 2 * conv_mt(12) * 32 * 192 * 2 <= kConvLds &&
                  2 * conv_mt(16) * 32 * 256 * 2 <= kConvLds,
              "a bf16 output tile must fit the LDS");
static_assert((2 * conv_mt(16) + 2) * 34 * (kConvChunk + 8) * 2 <= kConvLds &&
                  (2 * conv_mt(6) + 2) * 34 * (kConvChunk + 8) * 2 <= kConvLds,
              "the staged input window must fit the LDS");

// v with its elements zero where those of mk are not positive (bf16)
__device__ __forceinline__ uint4 relu_mask(uint4 v, uint4 mk)
{
    const u16 *em = (const u16 *)&mk;
    u16 *ev = (u16 *)&v;
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if (!(bf2f(em[q]) > 0.f)) ev[q] = 0;
    return v;
}

// The output tile [TR * 32 pixels][ps] staged in LDS (bf16, or FP32 with
// out_f32; ps >= Cout elements apart) to Y [.][H][W][Cout] as 16-byte stores
// where the channel count allows, zero where mask (when given) is not positive.
__device__ __forceinline__ void conv_store_tile(const unsigned char *lds_raw, int ps,
                                                void *__restrict__ Y, const u16 *__restrict__ mask,
                                                size_t img, int r0, int c0, int TR, int H, int W,
                                                int Cout, int out_f32)
{
    const int epv = out_f32 ? 4 : 8;  // elements per 16-byte store
    if (Cout % epv != 0) {            // channel counts off the 16-byte grid: one at a time
        for (int it = threadIdx.x; it < TR * 32 * Cout; it += 256) {
            const int p = it / Cout, e = it - p * Cout;
            const int rr = r0 + (p >> 5), cc = c0 + (p & 31);
            if (rr < H && cc < W) {
                const size_t o = (img + (size_t)rr * W + cc) * Cout + e;
                const bool keep = !mask || bf2f(mask[o]) > 0.f;
                if (out_f32) ((float *)Y)[o] = keep ? ((const float *)lds_raw)[p * ps + e] : 0.f;
                else ((u16 *)Y)[o] = keep ? ((const u16 *)lds_raw)[p * ps + e] : (u16)0;
            }
        }
        return;
    }
    const int vpp = Cout / epv;  // stores per pixel
    for (int it = threadIdx.x; it < TR * 32 * vpp; it += 256) {
        const int p = it / vpp, e = (it - p * vpp) * epv;
        const int rr = r0 + (p >> 5), cc = c0 + (p & 31);
        if (rr < H && cc < W) {
            const size_t o = (img + (size_t)rr * W + cc) * Cout + e;
            if (out_f32) {
                uint4 v = *(const uint4 *)((const float *)lds_raw + p * ps + e);
                if (mask) {
                    const uint2 mk = *(const uint2 *)(mask + o);
                    const u16 *em = (const u16 *)&mk;
                    uint32_t *ev = (uint32_t *)&v;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (!(bf2f(em[q]) > 0.f)) ev[q] = 0u;
                }
                *(uint4 *)((float *)Y + o) = v;
            } else {
                uint4 v = *(const uint4 *)((const u16 *)lds_raw + p * ps + e);
                if (mask) v = relu_mask(v, *(const uint4 *)(mask + o));
                *(uint4 *)((u16 *)Y + o) = v;
            }
        }
    }
}

template <int NT>
__global__ __launch_bounds__(256) void k_conv_fwd(const u16 *__restrict__ X,
                                                  const u16 *__restrict__ Wk,
                                                  const float *__restrict__ bias,
                                                  void *__restrict__ Y, int H, int W, int Cin,
                                                  int Cout, int ks, int relu, int out_f32,
                                                  const u16 *__restrict__ mask)
{
    constexpr int MT = conv_mt(NT);
    constexpr int TR = 2 * MT;
    constexpr int CoutP = NT * 16;
    // dynamic LDS, sized by the launch to this layer's window and output
    // tile (conv_fwd_lds): small layers keep more blocks per CU
    extern __shared__ __align__(16) unsigned char lds_raw[];
    u16 *win = (u16 *)lds_raw;
    const int n = blockIdx.z, r0 = blockIdx.y * TR, c0 = blockIdx.x * 32;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int m = lane & 15, grp = lane >> 4;
    const int halo = ks == 3 ? 1 : 0;
    const int HR = TR + 2 * halo, HC = 32 + 2 * halo;
    const size_t img = (size_t)n * H * W;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int cc0 = 0; cc0 < Cin; cc0 += kConvChunk) {
        const int CC = min(kConvChunk, Cin - cc0);  // a multiple of 8
        const int PS = CC + 8;                       // LDS pixel stride (bf16)
        const int c8n = CC / 8;
        __syncthreads();
        for (int it = threadIdx.x; it < HR * HC * c8n; it += 256) {
            const int px = it / c8n, c8 = (it - px * c8n) * 8;
            const int hr = px / HC, hc = px - hr * HC;
            const int rr = r0 - halo + hr, cc = c0 - halo + hc;
            uint4 v = make_uint4(0, 0, 0, 0);
            if (rr >= 0 && rr < H && cc >= 0 && cc < W)
                v = *(const uint4 *)(X + (img + (size_t)rr * W + cc) * Cin + cc0 + c8);
            *(uint4 *)(win + px * PS + c8) = v;
        }
        __syncthreads();
        if (CC % 32 == 0) {  // whole 32-channel K steps: no index division
            for (int tap = 0; tap < ks * ks; ++tap) {
                const int dr = ks == 3 ? tap / 3 : 0, dc = ks == 3 ? tap - 3 * (tap / 3) : 0;
                const u16 *wrow = Wk + ((size_t)tap * CoutP + m) * Cin + cc0 + 8 * grp;
                const u16 *arow = win + (dr * HC + dc) * PS + 8 * grp;
                for (int ci0 = 0; ci0 < CC; ci0 += 32) {
                    Frag b[NT];
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        b[t].u = *(const uint4 *)(wrow + (size_t)t * 16 * Cin + ci0);
#pragma unroll
                    for (int i = 0; i < MT; ++i) {
                        const int j = wid * MT + i;
                        const int orow = j >> 1, ocol = 16 * (j & 1) + m;
                        Frag a;
                        a.u = *(const uint4 *)(arow + (orow * HC + ocol) * PS + ci0);
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b[t].v,
                                                                                acc[i][t], 0, 0, 0);
                    }
                }
            }
            continue;
        }
        const int KT = ks * ks * CC;  // this chunk's K: (tap, channel), tap-major
        for (int kc = 0; kc < KT; kc += 32) {
            const int k = kc + 8 * grp;
            const bool kin = k < KT;
            const int tap = kin ? k / CC : 0;
            const int ci = kin ? k - tap * CC : 0;
            const int dr = ks == 3 ? tap / 3 : 0, dc = ks == 3 ? tap - 3 * (tap / 3) : 0;
            Frag b[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                b[t].u = make_uint4(0, 0, 0, 0);
                if (kin)
                    b[t].u = *(const uint4 *)(Wk + (((size_t)tap * CoutP + t * 16 + m) * Cin +
                                                    cc0 + ci));
            }
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int j = wid * MT + i;
                const int orow = j >> 1, ocol = 16 * (j & 1) + m;
                Frag a;
                a.u = make_uint4(0, 0, 0, 0);
                if (kin) a.u = *(const uint4 *)(win + ((orow + dr) * HC + ocol + dc) * PS + ci);
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b[t].v, acc[i][t], 0,
                                                                        0, 0);
            }
        }
    }
    // epilogue: D[pixel 4 grp + q of tile j][co = 16 t + m]
    if (out_f32 && (size_t)TR * 32 * CoutP * 4 > (size_t)kConvLds) {
        // an FP32 tile larger than the LDS: straight from the registers
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int co = t * 16 + m;
            const float bb = (bias && co < Cout) ? bias[co] : 0.f;
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int j = wid * MT + i;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int rr = r0 + (j >> 1), cc = c0 + 16 * (j & 1) + 4 * grp + q;
                    if (rr < H && cc < W && co < Cout) {
                        const size_t o = (img + (size_t)rr * W + cc) * Cout + co;
                        float v = acc[i][t][q] + bb;
                        if (relu) v = fmaxf(v, 0.f);
                        if (mask && !(bf2f(mask[o]) > 0.f)) v = 0.f;
                        ((float *)Y)[o] = v;
                    }
                }
            }
        }
        return;
    }
    // otherwise through LDS [pixel][co] (at most kConvLds bytes: bf16 tiles
    // are TR * 32 * CoutP * 2 <= 49152 bytes for every NT)
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int co = t * 16 + m;
        const float bb = (bias && co < Cout) ? bias[co] : 0.f;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int j = wid * MT + i;
            const int pbase = (j >> 1) * 32 + 16 * (j & 1) + 4 * grp;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v = acc[i][t][q] + bb;
                if (relu) v = fmaxf(v, 0.f);
                const int p = pbase + q;
                if (out_f32) ((float *)lds_raw)[p * CoutP + co] = v;
                else ((u16 *)lds_raw)[p * CoutP + co] = f2bf(v);
            }
        }
    }
    __syncthreads();
    conv_store_tile(lds_raw, CoutP, Y, mask, img, r0, c0, TR, H, W, Cout, out_f32);
}

// ------------------------------------------------------ conv fwd, 3x3 ---
// The 3x3 forward / input-gradient convolution for Cout <= 128 and Cin >= 16.  Block: 4
// waves on 8 x 32 output pixels of one image; wave w takes the column half
// w & 1 and the four rows 4 (w >> 1) .. of the tile.  Input channels go in
// chunks of 32 (zero beyond Cin): per chunk the block stages the input window
// (10 rows x 34 columns) and the chunk's weights of all nine taps in LDS.
// Then for each column shift dc a wave reads the six window-row fragments it
// needs once and uses each for the three kernel rows dr (output row i takes
// window row i + dr), so a window fragment feeds up to 3 NT matrix-core steps
// and a weight fragment four.  What bounds it is the latency of the windows at
// two blocks per CU (matrix cores and LDS are each a third busy): loading the
// next window behind the products took 8 x 512^2 64 -> 32 from 160 to 130 us
// and its input gradient (with the mask) from 285 to 170, a second window in
// flight to 113 and 163.  Again in one session, from graphs: 153 without either,
// 114 with both, 110 with the addresses in steps; with the mask 272, 137 and 136;
// at 5.1 TB/s their bytes take 78 and 131.
constexpr int kC3Chunk = 32;
constexpr int kC3Rows = 8, kC3MT = 4;                // tile rows, rows per wave
constexpr int kC3HR = kC3Rows + 2, kC3HC = 34;       // the staged window
constexpr int kC3Items = (kC3HR * kC3HC * 4 + 255) / 256;  // its 16-byte items per thread
constexpr int kC3Win = kC3Items * 256 * 16;          // its bytes in LDS, every item stored
// the 3x3 kernel up to 128 output channels from at least 16 input channels
// (its 32-channel chunks waste the matrix cores on fewer); its LDS (the
// weights and the FP32 tile of 128 output channels) fits the 160 KB of a CU
// and its offsets within a tile are 32-bit
inline bool conv3_use(int nt, int cin, int w)
{
    return cin >= 16 && nt <= 8 && (long long)(kC3HR + 1) * (w + kC3HC) * std::max(cin, 16 * nt) < 0x7fffffff;
}
constexpr size_t kC3LdsMax = 163840;

// bytes between the pixels of the output tile in LDS: 16 more where the
// pixels' own 32 NT bytes would put 16 of them on a quarter of the banks
__host__ __device__ constexpr int conv3_ps(int nt, int out_f32)
{
    return out_f32 ? 64 * nt + 16 : 32 * nt + (nt % 2 ? 0 : 16);
}

// LDS: bias, weights (of all nch chunks with wall, else of one), window; the
// output tile over the window, and over the weights too where they are staged
// again for each chunk
constexpr size_t conv3_lds(int nt, int nch, bool wall, int out_f32)
{
    const size_t w = (size_t)(wall ? nch : 1) * 9 * 16 * nt * kC3Chunk * 2;
    const size_t tile = (size_t)kC3Rows * 32 * conv3_ps(nt, out_f32);
    const size_t stage = wall ? w + std::max<size_t>(kC3Win, tile) : std::max(w + kC3Win, tile);
    return 64 * (size_t)nt + stage;
}
static_assert(conv3_lds(8, 1, false, 1) <= kC3LdsMax, "the 3x3 kernel's LDS must fit a CU");

// Window pixel (row hr, column hc) of a thread's items, 64 pixels apart.
struct WinPx {
    int hr, hc;
    __device__ __forceinline__ explicit WinPx(int tid)
    {
        const int px = tid >> 2;  // below 64: in the first two rows
        hr = px >= kC3HC;
        hc = px - hr * kC3HC;
    }
    __device__ __forceinline__ void next()
    {
        hr += 1;
        hc += 64 - kC3HC;
        if (hc >= kC3HC) {
            hr += 1;
            hc -= kC3HC;
        }
    }
};
static_assert(kC3HC <= 64 && 64 < 2 * kC3HC, "64 pixels on: one or two rows");

// Byte offset of the 16-byte piece c (0..3) of a staged 64-byte row: pieces
// are rotated by col, the row's window column or output channel, so that a
// fragment read (16 neighbouring rows, one piece each) touches every bank once
// and differs by a constant from row to row of the window and tap to tap.
__device__ __forceinline__ int c3_at(int row, int col, int c)
{
    return row * 64 + ((c ^ (col >> 1)) & 3) * 16;
}

// Blocks stay: block b of a grid of 8 g takes every g-th tile of the b % 8th
// eighth of the tiles (consecutive blocks go to different XCDs, so each XCD's
// L2 sees one run of neighbouring tiles and their shared halo rows).  The
// window of a (tile, chunk) is loaded into registers two steps before it is
// multiplied, and the mask of the output while the last chunk is, so a
// block's loads are in flight behind its matrix-core work; with the weights
// of every chunk held in LDS for the block's life (WALL) the windows are all
// that is staged.  WHOLE: a bf16 output of 16 NT channels, which leaves in
// whole 16-byte pieces; otherwise any channel count and FP32.
template <int NT, bool WALL, bool WHOLE>
__global__ __launch_bounds__(256, NT <= 4 ? 2 : 1) void k_conv3(
    const u16 *__restrict__ X, const u16 *__restrict__ Wk, const float *__restrict__ bias,
    void *__restrict__ Y, int H, int W, int Cin, int Cout, int relu, int out_f32,
    const u16 *__restrict__ mask, int tx, int ty, int ntile)
{
    constexpr int CoutP = 16 * NT, MT = kC3MT;
    constexpr int NWIN = kC3HR * kC3HC * 4, KW = kC3Items;  // 16-byte items
    constexpr int NWTS = 9 * CoutP * 4, KB = (NWTS + 255) / 256;
    constexpr int VPP = 2 * NT;  // 16-byte pieces of a bf16 output pixel
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int nch = (Cin + kC3Chunk - 1) / kC3Chunk;
    float *sb = (float *)lds_raw;
    unsigned char *wts = lds_raw + 64 * NT;  // [chunk][9][CoutP] rows of 64 bytes
    unsigned char *win = wts + (size_t)(WALL ? nch : 1) * NWTS * 16;  // [HR][HC] rows of 64 bytes
    unsigned char *out = WALL ? win : wts;                            // the output tile
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int m = lane & 15, grp = lane >> 4;
    const int h = wid & 1, rg = wid >> 1;
    const int s0 = (int)((long long)ntile * (blockIdx.x & 7) >> 3);
    const int s1 = (int)((long long)ntile * ((blockIdx.x & 7) + 1) >> 3);
    const int step = gridDim.x >> 3;
    const int first = s0 + (blockIdx.x >> 3);
    if (first >= s1) return;
    if ((int)threadIdx.x < CoutP)
        sb[threadIdx.x] = bias && (int)threadIdx.x < Cout ? bias[threadIdx.x] : 0.f;

    struct Window {
        uint4 v[KW];  // pixels and channels outside the image load its first element ...
        unsigned ok;  // ... and are stored as zero: bit k for item k
        int tile, c;  // tile >= s1: none
    };
    auto corner = [&](int t, int &n, int &r0, int &c0) {
        n = t / (tx * ty);
        const int q = t - n * (tx * ty);
        r0 = q / tx * kC3Rows;
        c0 = q % tx * 32;
    };
    auto window_load = [&](Window &w, int t, int c) {
        w.tile = t;
        w.c = c;
        int n, r0, c0;
        corner(t < s1 ? t : first, n, r0, c0);
        const int tid = opaque_tid();
        // may point before the image: only pixels inside it are dereferenced
        const u16 *Xt = X + (((long long)n * H + r0 - 1) * W + c0 - 1) * Cin + c * kC3Chunk;
        w.ok = 0;
        WinPx at(tid);
        const int ci = (tid & 3) * 8;
#pragma unroll
        for (int k = 0; k < KW; ++k, at.next()) {
            const int it = tid + 256 * k, hr = at.hr, hc = at.hc;
            const bool in = (256 * k + 256 <= NWIN || it < NWIN) &
                            ((unsigned)(r0 - 1 + hr) < (unsigned)H) &
                            ((unsigned)(c0 - 1 + hc) < (unsigned)W) & (c * kC3Chunk + ci < Cin);
            w.ok |= (unsigned)in << k;
            const u16 *p = Xt + (hr * W + hc) * Cin + ci;
            w.v[k] = *(const uint4 *)(in ? p : X);
        }
    };
    // item k of a thread lies 64 rows after item 0, in global memory and in LDS
    auto weights = [&](int c, unsigned char *dst) {
        const int tid = opaque_tid();
        const int row = tid >> 2, ci = c * kC3Chunk + (tid & 3) * 8;
        const bool in = ci < Cin;
        const u16 *src = Wk + (in ? row * Cin + ci : 0);
        dst += c3_at(row, row, tid & 3);
#pragma unroll
        for (int g = 0; g < KB; g += 8) {
            uint4 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool all = 256 * (g + k) + 256 <= NWTS;
                if (g + k < KB)
                    v[k] = *(const uint4 *)(all || tid + 256 * (g + k) < NWTS ? src + 64 * (g + k) * Cin : Wk);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool all = 256 * (g + k) + 256 <= NWTS;
                if (g + k < KB && (all || tid + 256 * (g + k) < NWTS))
                    *(uint4 *)(dst + 64 * 64 * (g + k)) = in ? v[k] : make_uint4(0, 0, 0, 0);
            }
        }
    };
    f32x4 acc[MT][NT];
    // multiplies the window of w, then (after the last chunk) stores the tile;
    // nt, nc: the tile and chunk two steps on, loaded into w meanwhile
    auto run = [&](Window &w, int nt, int nc) {
        const int tile = w.tile, c = w.c;
        const bool last = c + 1 == nch;
        int n, r0, c0;
        corner(tile, n, r0, c0);
        const size_t img = (size_t)n * H * W;
        __syncthreads();  // the chunk or tile before is done with the LDS
        {
            const int tid = opaque_tid();
            WinPx at(tid);
#pragma unroll
            for (int k = 0; k < KW; ++k, at.next()) {
                const unsigned keep = 0u - (w.ok >> k & 1u);
                const uint4 v = w.v[k];
                *(uint4 *)(win + c3_at((tid >> 2) + 64 * k, at.hc, tid & 3)) =
                    make_uint4(v.x & keep, v.y & keep, v.z & keep, v.w & keep);
            }
        }
        if constexpr (!WALL) weights(c, wts);
        uint4 mk[VPP];
        if (WHOLE && last && mask) {
            const int tid = opaque_tid();
            const u16 *mt = mask + (img + (size_t)r0 * W + c0) * CoutP;
#pragma unroll
            for (int k = 0; k < VPP; ++k) {
                const int it = tid + 256 * k;
                const int p = it / VPP, e = it % VPP * 8;
                const u16 *q = mt + ((p >> 5) * W + (p & 31)) * CoutP + e;
                mk[k] = *(const uint4 *)(((r0 + (p >> 5) < H) & (c0 + (p & 31) < W)) ? q : mask);
            }
        }
        __syncthreads();
        window_load(w, nt, nc);
        if (c == 0)
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        const unsigned char *wc = wts + (WALL ? c * NWTS * 16 : 0) + c3_at(m, m, grp);
#pragma unroll
        for (int dc = 0; dc < 3; ++dc) {
            const int hc = 16 * h + m + dc;
            const unsigned char *wr = win + c3_at(rg * MT * kC3HC + hc, hc, grp);
            Frag a[MT + 2];
#pragma unroll
            for (int r = 0; r < MT + 2; ++r) a[r].u = *(const uint4 *)(wr + r * kC3HC * 64);
#pragma unroll
            for (int dr = 0; dr < 3; ++dr) {
                Frag b[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    b[t].u = *(const uint4 *)(wc + ((3 * dr + dc) * CoutP + 16 * t) * 64);
                // D[co = 16 t + 4 grp + .][pixel m of row i]
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[t].v, a[i + dr].v,
                                                                            acc[i][t], 0, 0, 0);
            }
        }
        if (!last) return;
        // the tile through LDS [pixel][co] (pixel = row * 32 + column)
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const f32x4 bb = *(const f32x4 *)(sb + 16 * t + 4 * grp);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                f32x4 v = acc[i][t] + bb;
                if (relu)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
                const int p = (rg * MT + i) * 32 + 16 * h + m;
                if (!WHOLE && out_f32) *(f32x4 *)(out + p * conv3_ps(NT, 1) + 64 * t + 16 * grp) = v;
                else *(bf16x4 *)(out + p * conv3_ps(NT, 0) + 32 * t + 8 * grp) =
                    __builtin_convertvector(v, bf16x4);
            }
        }
        __syncthreads();
        if constexpr (!WHOLE) {
            conv_store_tile(out, out_f32 ? conv3_ps(NT, 1) / 4 : conv3_ps(NT, 0) / 2, Y, mask, img,
                            r0, c0, kC3Rows, H, W, Cout, out_f32);
            return;
        }
        const int tid = opaque_tid();
#pragma unroll
        for (int k = 0; k < VPP; ++k) {
            const int it = tid + 256 * k;
            const int p = it / VPP, e = it % VPP * 8;
            const int rr = r0 + (p >> 5), cc = c0 + (p & 31);
            uint4 v = *(const uint4 *)(out + p * conv3_ps(NT, 0) + e * 2);
            if (mask) v = relu_mask(v, mk[k]);
            if (rr < H && cc < W) *(uint4 *)((u16 *)Y + (img + (size_t)rr * W + cc) * CoutP + e) = v;
        }
    };
    int nt = first, nc = 0;  // the next (tile, chunk) to load
    auto advance = [&] {
        if (++nc == nch) {
            nc = 0;
            nt += step;
        }
    };
    Window wa, wb;
    window_load(wa, nt, nc);
    advance();
    window_load(wb, nt, nc);
    advance();
    if constexpr (WALL)
        for (int c = 0; c < nch; ++c) weights(c, wts + (size_t)c * NWTS * 16);
    while (wa.tile < s1) {
        run(wa, nt, nc);
        advance();
        if (wb.tile < s1) {
            run(wb, nt, nc);
            advance();
        } else {
            // the last step, with nothing left to wait for: without it the
            // compiler takes wa's loads for the newest ones on the way round
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
        }
    }
}

// ----------------------------------------------------------- conv wgrad ---
// Partial weight and bias gradients of one chunk: a strip of kWgPix columns
// (from c0) of image n over rows [r0, r0 + 4 kst), in steps of four rows.
// dZ [N][H][W][Cout], X [N][H][W][Cin] (channel counts multiples of 8).
// Block = 4 waves on TMS output-channel and TNS WN input-channel tiles: wave w
// takes the TNS input tiles (w % WN) TNS .. and WN of a step's rows, from
// (w / WN) WN.  Per step the block stages, transposed into LDS
// ([channel][column], bf16, zero outside the image), the four rows of dZ and
// the four rows of X (columns c0 - 1 .. c0 + kWgPix + 2 for 3x3) that it does
// not hold yet: X rows stay in a ring of six, so each is read once per chunk.
// A wave reads its dZ fragments and, for every X row that its rows reach, two
// 16-byte fragments and the next dword, which give the column shifts 0, 1 and
// 2 of three taps, and uses them for every (dZ row, kernel row) that meets
// there.  Threads t < 4 * 16 TMS of the ci-split 0 blocks also sum their dZ
// row and channel (the bias gradient).  At the end the row groups' sums are
// added in order through LDS and written to part[chunk][taps][CoutP][Cin], the
// bias to part[chunk][len + co] (len = taps CoutP Cin): every chunk's row is
// written whole by its split blocks.  split = sm * nsn + sn (co tiles sm
// TMS.., ci tiles sn TNS WN..), chunk = strip * nrc + row chunk.
// Bound by memory latency at two blocks per CU, then LDS.  8 x 512^2, 64 -> 32:
// 264 us with a wave per row and one input tile per block (dZ read four times,
// X in 32-byte pieces, X rows r - 1 and r + 4 twice; 192 of 340 k clocks lost to
// LDS bank conflicts of the transposed writes), 149 with every input tile in
// the block, 131 with the writes on all banks, 112 with each X row read from
// LDS once; its bytes take 78 at 5.1 TB/s.
constexpr int kWgPix = 64;  // two matrix-core steps
constexpr int kWgLD = kWgPix + 8;  // bf16 row stride of the staged arrays

__host__ __device__ constexpr int wg_xrows(int ks) { return ks == 3 ? 6 : 4; }

template <int KS, int TMS, int TNS, int WN>
__global__ __launch_bounds__(256, 2) void k_wgrad(const u16 *__restrict__ dZ,
                                               const u16 *__restrict__ X,
                                               float *__restrict__ part, int H, int W, int Cin,
                                               int Cout, int nstrip, int nstrip_n, int nrc, int kst,
                                               int nsn, int nsplit, int by_xcd, size_t len,
                                               size_t pstride)
{
    constexpr int T = KS * KS, XR = wg_xrows(KS), ZC = 16 * TMS, XC = 16 * TNS * WN;
    constexpr int WR = 4 / WN;
    constexpr int halo = KS == 3 ? 1 : 0;
    constexpr int K4X = (kWgPix + 4 * halo) / 4;  // 4-column groups of a staged X row
    extern __shared__ __align__(16) unsigned char lds_raw[];
    u16 *sZ = (u16 *)lds_raw;           // [4][ZC][kWgLD]
    u16 *sX = sZ + 4 * ZC * kWgLD;      // [XR][XC][kWgLD]: element k is column c0 - halo + k
    // by_xcd: the splits of a chunk, which read the same rows, eight blocks apart:
    // on one XCD (consecutive blocks go to different ones), whose L2 they share
    const int bq = by_xcd ? blockIdx.x >> 3 : blockIdx.x, split = bq % nsplit;
    const int chunk = by_xcd ? bq / nsplit * 8 + (blockIdx.x & 7) : bq / nsplit;
    if (chunk >= nstrip_n * nrc) return;
    const int sm = split / nsn, sn = split - sm * nsn;
    const int rc = chunk % nrc, strip = chunk / nrc;
    const int n = strip / nstrip, c0 = (strip - n * nstrip) * kWgPix;
    const int co0 = sm * ZC, ci0 = sn * XC;
    const int CoutP = (Cout + 15) / 16 * 16;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, grp = lane >> 4;
    const int wn = wid % WN, wr = wid / WN;
    const long long img = (long long)n * H * W;
    const bool bias = sn == 0;
    f32x4 acc[T][TMS][TNS];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < TMS; ++i)
#pragma unroll
            for (int j = 0; j < TNS; ++j) acc[t][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    // Staging items: four pixels by eight channels.  A step's loads are
    // unconditional (a pixel or channel outside the tensor loads dZ's first
    // element and is stored as zero), so they are in flight together, and the
    // next step's loads go out before this step's matrix-core work.
    constexpr int zrow = kWgPix / 4 * (ZC / 8), xrow = K4X * (XC / 8);  // items of a row
    constexpr int NZ = (4 * zrow + 255) / 256, NX = (4 * xrow + 255) / 256;
    uint4 zv[NZ][4], xv[NX][4];
    unsigned ok[NZ + NX];
    // item it: row q, pixels 4 k4 .., channels o8 ..  Two channel groups next to
    // each other, then the row's pixels: 32 lanes write 8 bytes each to two LDS
    // rows eight channels apart, every bank once (all of a pixel's channels
    // first would meet in the same banks four times over).
    auto item = [](int it, int n4, int nch8, int &q, int &k4, int &o8) {
        const int g = it / (2 * n4), rem = it - g * (2 * n4);
        q = g / (nch8 / 2);
        k4 = rem >> 1;
        o8 = 16 * (g - q * (nch8 / 2)) + 8 * (rem & 1);
    };
    // item it of rows r .. of a [N][H][W][C] tensor from column c and channel ch0
    auto item_load = [&](uint4 *v, const u16 *src, int C, int ch0, int r, int c, int it, int n4,
                         int nch8, int items) -> unsigned {
        int q, k4, o8;
        item(it, n4, nch8, q, k4, o8);
        // may point before the tensor: only pixels inside it are dereferenced
        const u16 *p = src + (img + (long long)r * W + c) * C + ch0 +
                       ((unsigned long long)(unsigned)q * (unsigned)W + (unsigned)(4 * k4)) * (unsigned)C + o8;
        const bool row = (it < items) & ((unsigned)(r + q) < (unsigned)H) & (ch0 + o8 < C);
        unsigned okb = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool in = row & ((unsigned)(c + 4 * k4 + u) < (unsigned)W);
            okb |= (unsigned)in << u;
            v[u] = *(const uint4 *)(in ? p + u * C : dZ);
        }
        return okb;
    };
    // its four pixels, channel by channel, to rows of kWgLD at dst (nch rows per image row)
    auto item_store = [&](const uint4 *s, unsigned okb, u16 *dst) {
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const unsigned keep = 0u - (okb >> u & 1u);
            v[u] = make_uint4(s[u].x & keep, s[u].y & keep, s[u].z & keep, s[u].w & keep);
        }
        const uint32_t *w0 = (const uint32_t *)&v[0], *w1 = (const uint32_t *)&v[1];
        const uint32_t *w2 = (const uint32_t *)&v[2], *w3 = (const uint32_t *)&v[3];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned sel = e & 1 ? 0x07060302u : 0x05040100u;  // the odd or even halves
            uint2 w;
            w.x = __builtin_amdgcn_perm(w1[e / 2], w0[e / 2], sel);
            w.y = __builtin_amdgcn_perm(w3[e / 2], w2[e / 2], sel);
            *(uint2 *)(dst + e * kWgLD) = w;
        }
    };
    auto x_store = [&](const uint4 *v, unsigned okb, int it, int slot0) {  // slot0: LDS row of its q = 0
        int q, k4, o8;
        item(it, K4X, XC / 8, q, k4, o8);
        int slot = slot0 + q;
        if (slot >= XR) slot -= XR;
        item_store(v, okb, sX + (slot * XC + o8) * kWgLD + 4 * k4);
    };
    // rows r .. r + 3 of dZ and the four X rows that a step adds: r + halo ..
    auto stage_load = [&](int r) {
        const int tid = opaque_tid();
#pragma unroll
        for (int k = 0; k < NZ; ++k)
            ok[k] = item_load(zv[k], dZ, Cout, co0, r, c0, tid + 256 * k, kWgPix / 4, ZC / 8, 4 * zrow);
#pragma unroll
        for (int k = 0; k < NX; ++k)
            ok[NZ + k] = item_load(xv[k], X, Cin, ci0, r + halo, c0 - halo, tid + 256 * k, K4X, XC / 8,
                                   4 * xrow);
    };
    auto stage_store = [&](int slot0) {
        const int tid = opaque_tid();
#pragma unroll
        for (int k = 0; k < NZ; ++k) {
            const int it = tid + 256 * k;
            if (256 * k + 256 > 4 * zrow && it >= 4 * zrow) break;
            int q, k4, o8;
            item(it, kWgPix / 4, ZC / 8, q, k4, o8);
            item_store(zv[k], ok[k], sZ + (q * ZC + o8) * kWgLD + 4 * k4);
        }
#pragma unroll
        for (int k = 0; k < NX; ++k) {
            const int it = tid + 256 * k;
            if (256 * k + 256 > 4 * xrow && it >= 4 * xrow) break;
            x_store(xv[k], ok[NZ + k], it, slot0);
        }
    };
    const int st0 = rc * kst, nst = min(kst, (H + 3) / 4 - st0);
    // X row r - halo + j of a step is in LDS row (base + j) % XR; a step keeps
    // the last 2 halo rows of the one before (the first step's come here)
    int base = 0;
    stage_load(st0 * 4);
    if constexpr (halo > 0) {
        constexpr int items = 2 * halo * xrow;
#pragma unroll 1
        for (int it = threadIdx.x; it < items; it += 256) {
            uint4 v[4];
            const unsigned okb = item_load(v, X, Cin, ci0, st0 * 4 - halo, c0 - halo, it, K4X, XC / 8, items);
            x_store(v, okb, it, 0);
        }
    }
    for (int st = 0; st < nst; ++st) {
        __syncthreads();  // the previous step is done with the LDS
        stage_store(base + 2 * halo < XR ? base + 2 * halo : base + 2 * halo - XR);
        __syncthreads();
        if (st + 1 < nst) stage_load((st0 + st + 1) * 4);
        if (bias && (int)threadIdx.x < 4 * ZC) {  // row t / ZC, channel t % ZC
            const u16 *zr = sZ + (size_t)threadIdx.x * kWgLD;
#pragma unroll
            for (int k = 0; k < kWgPix; k += 8) {
                const uint4 v = *(const uint4 *)(zr + k);
                const u16 *e = (const u16 *)&v;
#pragma unroll
                for (int q = 0; q < 8; ++q) bsum += bf2f(e[q]);
            }
        }
        // lane group grp takes pixels 16 grp .. + 15, eight per matrix-core step
        Frag a[WN][2][TMS];
#pragma unroll
        for (int r = 0; r < WN; ++r)
#pragma unroll
            for (int i = 0; i < TMS; ++i)
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    a[r][k][i].u = *(const uint4 *)(sZ + ((wr * WN + r) * ZC + i * 16 + m) * kWgLD +
                                                    16 * grp + 8 * k);
#pragma unroll
        for (int x = 0; x < WN + 2 * halo; ++x) {  // the X rows that this wave's rows reach
            const int s = base + wr * WN + x, slot = s < XR ? s : s - XR;
#pragma unroll
            for (int j = 0; j < TNS; ++j) {
                const u16 *xr = sX + (slot * XC + (wn * TNS + j) * 16 + m) * kWgLD + 16 * grp;
                Frag b[2][KS];
                b[0][0].u = *(const uint4 *)xr;
                b[1][0].u = *(const uint4 *)(xr + 8);
                if constexpr (KS == 3) {
                    const uint32_t nx[2] = {b[1][0].u.x, *(const uint32_t *)(xr + 16)};
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const uint4 v = b[k][0].u;
                        b[k][1].u = make_uint4(__builtin_amdgcn_alignbit(v.y, v.x, 16),
                                               __builtin_amdgcn_alignbit(v.z, v.y, 16),
                                               __builtin_amdgcn_alignbit(v.w, v.z, 16),
                                               __builtin_amdgcn_alignbit(nx[k], v.w, 16));
                        b[k][2].u = make_uint4(v.y, v.z, v.w, nx[k]);
                    }
                }
#pragma unroll
                for (int dr = 0; dr < KS; ++dr) {
                    if (x - dr < 0 || x - dr >= WN) continue;
#pragma unroll
                    for (int k = 0; k < 2; ++k)
#pragma unroll
                        for (int dc = 0; dc < KS; ++dc)
#pragma unroll
                            for (int i = 0; i < TMS; ++i)
                                acc[KS * dr + dc][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    a[x - dr][k][i].v, b[k][dc].v, acc[KS * dr + dc][i][j], 0, 0, 0);
                }
            }
        }
        base = base + 4 < XR ? base + 4 : base + 4 - XR;
    }
    // the row groups' sums, added in order, one tap at a time
    float *red = (float *)lds_raw;  // [WR - 1][WN][TMS][TNS][4][64]
    float *dst = part + (size_t)chunk * pstride;
    constexpr int RW = TMS * TNS * 4 * 64;  // floats of a wave
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if constexpr (WR > 1) {
            __syncthreads();
            if (wr > 0) {
#pragma unroll
                for (int i = 0; i < TMS; ++i)
#pragma unroll
                    for (int j = 0; j < TNS; ++j)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            red[(wid - WN) * RW + ((i * TNS + j) * 4 + q) * 64 + lane] = acc[t][i][j][q];
            }
            __syncthreads();
            if (wr > 0) continue;
        }
#pragma unroll
        for (int i = 0; i < TMS; ++i)
#pragma unroll
            for (int j = 0; j < TNS; ++j) {
                const int ci = ci0 + (wn * TNS + j) * 16 + m;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v = acc[t][i][j][q];
#pragma unroll
                    for (int w = 0; w < WR - 1; ++w)
                        v += red[(w * WN + wn) * RW + ((i * TNS + j) * 4 + q) * 64 + lane];
                    if (ci < Cin)
                        dst[((size_t)t * CoutP + co0 + i * 16 + 4 * grp + q) * Cin + ci] = v;
                }
            }
    }
    if (bias) {
        __syncthreads();
        if ((int)threadIdx.x < 4 * ZC) red[threadIdx.x] = bsum;
        __syncthreads();
        if ((int)threadIdx.x < ZC) {
            const int c = threadIdx.x;
            dst[len + co0 + c] = ((red[c] + red[ZC + c]) + red[2 * ZC + c]) + red[3 * ZC + c];
        }
    }
}

// seg[s][i] = sum over chunks q in [s L, min(nchunk, (s + 1) L)) of
// part[q][i]; four interleaved running sums, combined in a fixed order.
__global__ __launch_bounds__(256) void k_sum_seg(const float *__restrict__ part,
                                                 float *__restrict__ seg, int nchunk, size_t len,
                                                 int L)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= len) return;
    const int q0 = blockIdx.y * L, q1 = min(nchunk, q0 + L);
    float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
    int q = q0;
    for (; q + 4 <= q1; q += 4) {
        a0 += part[(size_t)q * len + i];
        a1 += part[(size_t)(q + 1) * len + i];
        a2 += part[(size_t)(q + 2) * len + i];
        a3 += part[(size_t)(q + 3) * len + i];
    }
    for (; q < q1; ++q) a0 += part[(size_t)q * len + i];
    seg[(size_t)blockIdx.y * len + i] = (a0 + a1) + (a2 + a3);
}

// The sum of the nseg segments in segment order: element i < len0 to out0[i],
// the rest to out1[i - len0].
__global__ __launch_bounds__(256) void k_sum_out(const float *__restrict__ seg,
                                                 float *__restrict__ out0, float *__restrict__ out1,
                                                 int nseg, size_t len0, size_t len)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= len) return;
    float s = 0.f;
    int q = 0;
    for (; q + 16 <= nseg; q += 16) {  // sixteen loads in flight, added in order
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = seg[(size_t)(q + k) * len + i];
#pragma unroll
        for (int k = 0; k < 16; ++k) s += v[k];
    }
    for (; q < nseg; ++q) s += seg[(size_t)q * len + i];
    if (i < len0) out0[i] = s;
    else out1[i - len0] = s;
}

// Segments for summing nchunk partials of len values: enough blocks to
// spread the reads over the GPU, at least 4 chunks per segment and at most
// 64 segments (the second pass adds them one after another).
inline int sum_segments(int nchunk, size_t len)
{
    const size_t bx = (len + 255) / 256;
    size_t S = (2048 + bx - 1) / bx;
    S = std::min<size_t>(S, (size_t)std::max(1, nchunk / 4));
    S = std::min<size_t>(S, 64);
    return (int)std::max<size_t>(1, S);
}

// --------------------------------------------------------- elementwise ---
// dgrad weights: Wd[tap'][ci][co] = Wk[taps-1-tap'][co][ci], CinP rows padded.
__global__ void k_wflip(const u16 *__restrict__ Wk, u16 *__restrict__ Wd, int taps, int Cin,
                        int Cout, int CoutP, int CinP)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t total = (size_t)taps * CinP * Cout;
    if (i >= total) return;
    int co = (int)(i % Cout);
    size_t rest = i / Cout;
    int ci = (int)(rest % CinP);
    int tp = (int)(rest / CinP);
    u16 v = 0;
    if (ci < Cin) v = Wk[((size_t)(taps - 1 - tp) * CoutP + co) * Cin + ci];
    Wd[i] = v;
}

__global__ void k_relu_bwd(const u16 *__restrict__ dy, const u16 *__restrict__ y,
                           u16 *__restrict__ dz, size_t n)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    dz[i] = bf2f(y[i]) > 0.f ? dy[i] : (u16)0;
}

// the same, 8 elements (16 bytes) per thread; n8 = n / 8
__global__ void k_relu_bwd8(const uint4 *__restrict__ dy, const uint4 *__restrict__ y,
                            uint4 *__restrict__ dz, size_t n8)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n8) return;
    uint4 a = dy[i], b = y[i], r;
    const u16 *ea = (const u16 *)&a, *eb = (const u16 *)&b;
    u16 *er = (u16 *)&r;
#pragma unroll
    for (int q = 0; q < 8; ++q) er[q] = bf2f(eb[q]) > 0.f ? ea[q] : (u16)0;
    dz[i] = r;
}

// 2x2 max pool, stride 2 (H, W even); idx records the winning sub-pixel.
__global__ void k_pool_fwd(const u16 *__restrict__ x, u16 *__restrict__ y,
                           uint8_t *__restrict__ idx, int N, int H, int W, int C)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int Ho = H / 2, Wo = W / 2;
    size_t total = (size_t)N * Ho * Wo * C;
    if (i >= total) return;
    int c = (int)(i % C);
    size_t p = i / C;
    int wo = (int)(p % Wo), ho = (int)((p / Wo) % Ho), n = (int)(p / ((size_t)Wo * Ho));
    float best = -INFINITY;
    int bi = 0;
    for (int q = 0; q < 4; ++q) {
        int hh = 2 * ho + q / 2, ww = 2 * wo + q % 2;
        float v = bf2f(x[(((size_t)n * H + hh) * W + ww) * C + c]);
        if (v > best) { best = v; bi = q; }
    }
    y[i] = f2bf(best);
    idx[i] = (uint8_t)bi;
}

__global__ void k_pool_bwd(const u16 *__restrict__ dy, const uint8_t *__restrict__ idx,
                           u16 *__restrict__ dx, int N, int H, int W, int C)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;  // over dx
    size_t total = (size_t)N * H * W * C;
    if (i >= total) return;
    int c = (int)(i % C);
    size_t p = i / C;
    int w = (int)(p % W), h = (int)((p / W) % H), n = (int)(p / ((size_t)W * H));
    const int Ho = H / 2, Wo = W / 2;
    size_t o = (((size_t)n * Ho + h / 2) * Wo + w / 2) * C + c;
    dx[i] = idx[o] == (uint8_t)((h % 2) * 2 + (w % 2)) ? dy[o] : (u16)0;
}

// depth-to-space: y[n][2i+a][2j+b][c] = t[n][i][j][(2a+b)*C + c]; mode 1 inverts.
__global__ void k_shuffle(const u16 *__restrict__ src, u16 *__restrict__ dst, int N, int Hin,
                          int Win, int C, int inverse)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;  // over the 2x image
    const int H = 2 * Hin, W = 2 * Win;
    size_t total = (size_t)N * H * W * C;
    if (i >= total) return;
    int c = (int)(i % C);
    size_t p = i / C;
    int w = (int)(p % W), h = (int)((p / W) % H), n = (int)(p / ((size_t)W * H));
    size_t t = (((size_t)n * Hin + h / 2) * Win + w / 2) * (4 * C) + ((h % 2) * 2 + (w % 2)) * C + c;
    if (!inverse) dst[i] = src[t];
    else dst[t] = src[i];
}

// channel concat: z[p][0:C1] = a[p], z[p][C1:C1+C2] = b[p]; inverse splits.
__global__ void k_concat(u16 *__restrict__ a, u16 *__restrict__ b, u16 *__restrict__ z, size_t P,
                         int C1, int C2, int inverse)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int C = C1 + C2;
    if (i >= P * C) return;
    size_t p = i / C;
    int c = (int)(i % C);
    u16 *s = c < C1 ? a + p * C1 + c : b + p * C2 + (c - C1);
    if (!inverse) z[i] = *s;
    else *s = z[i];
}

__global__ void k_add(const u16 *__restrict__ a, const u16 *__restrict__ b, u16 *__restrict__ z,
                      size_t n)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) z[i] = f2bf(bf2f(a[i]) + bf2f(b[i]));
}

// z = bf16(a + b) where y > 0, else 0 (a sum's gradient through a ReLU)
__global__ void k_add_relu_bwd(const u16 *__restrict__ a, const u16 *__restrict__ b,
                               const u16 *__restrict__ y, u16 *__restrict__ z, size_t n)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    z[i] = bf2f(y[i]) > 0.f ? f2bf(bf2f(a[i]) + bf2f(b[i])) : (u16)0;
}

__global__ void k_add_relu_bwd8(const uint4 *__restrict__ a, const uint4 *__restrict__ b,
                                const uint4 *__restrict__ y, uint4 *__restrict__ z, size_t n8)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n8) return;
    uint4 x = a[i], w = b[i], m = y[i], r;
    const u16 *ex = (const u16 *)&x, *ew = (const u16 *)&w, *em = (const u16 *)&m;
    u16 *er = (u16 *)&r;
#pragma unroll
    for (int q = 0; q < 8; ++q) er[q] = bf2f(em[q]) > 0.f ? f2bf(bf2f(ex[q]) + bf2f(ew[q])) : (u16)0;
    z[i] = r;
}

__global__ void k_add8(const uint4 *__restrict__ a, const uint4 *__restrict__ b,
                       uint4 *__restrict__ z, size_t n8)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n8) return;
    uint4 x = a[i], y = b[i], r;
    const u16 *ex = (const u16 *)&x, *ey = (const u16 *)&y;
    u16 *er = (u16 *)&r;
#pragma unroll
    for (int q = 0; q < 8; ++q) er[q] = f2bf(bf2f(ex[q]) + bf2f(ey[q]));
    z[i] = r;
}

// channel concat / split in 8-channel (16-byte) pieces (C1, C2 % 8 == 0)
__global__ void k_concat8(uint4 *__restrict__ a, uint4 *__restrict__ b, uint4 *__restrict__ z,
                          size_t P, int C1, int C2, int inverse)
{
    const int g1 = C1 / 8, g = (C1 + C2) / 8;
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= P * g) return;
    size_t p = i / g;
    int c = (int)(i - p * g);
    uint4 *s = c < g1 ? a + p * g1 + c : b + p * (g - g1) + (c - g1);
    if (!inverse) z[i] = *s;
    else *s = z[i];
}

// z = (depth-to-space of t: C1 channels, s: C2 channels) in 8-channel pieces,
// one thread per piece of z; inverse: t and s from z
__global__ void k_shuffle_concat8(uint4 *__restrict__ t, uint4 *__restrict__ s,
                                  uint4 *__restrict__ z, int N, int Hin, int Win, int C1, int C2,
                                  int inverse)
{
    const int g1 = C1 / 8, g = (C1 + C2) / 8;
    const int H = 2 * Hin, W = 2 * Win;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)N * H * W * g) return;
    const size_t p = i / g;
    const int c = (int)(i - p * g);
    uint4 *src;
    if (c < g1) {
        const int w = (int)(p % W), h = (int)((p / W) % H), n = (int)(p / ((size_t)W * H));
        src = t + (((size_t)n * Hin + h / 2) * Win + w / 2) * (4 * g1) +
              ((h % 2) * 2 + (w % 2)) * g1 + c;
    } else {
        src = s + p * (g - g1) + (c - g1);
    }
    if (!inverse) z[i] = *src;
    else *src = z[i];
}

// depth-to-space in 8-channel pieces (C % 8 == 0)
__global__ void k_shuffle8(const uint4 *__restrict__ src, uint4 *__restrict__ dst, int N, int Hin,
                           int Win, int C, int inverse)
{
    const int g = C / 8;
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;  // over the 2x image, 8 channels each
    const int H = 2 * Hin, W = 2 * Win;
    size_t total = (size_t)N * H * W * g;
    if (i >= total) return;
    int c = (int)(i % g);
    size_t p = i / g;
    int w = (int)(p % W), h = (int)((p / W) % H), n = (int)(p / ((size_t)W * H));
    size_t t = (((size_t)n * Hin + h / 2) * Win + w / 2) * (4 * g) + ((h % 2) * 2 + (w % 2)) * g + c;
    if (!inverse) dst[i] = src[t];
    else dst[t] = src[i];
}

// 2x2 max pool, 8 channels per thread (C % 8 == 0)
__global__ void k_pool_fwd8(const u16 *__restrict__ x, u16 *__restrict__ y,
                            uint8_t *__restrict__ idx, int N, int H, int W, int C)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int Ho = H / 2, Wo = W / 2, g = C / 8;
    size_t total = (size_t)N * Ho * Wo * g;
    if (i >= total) return;
    int c = (int)(i % g) * 8;
    size_t p = i / g;
    int wo = (int)(p % Wo), ho = (int)((p / Wo) % Ho), n = (int)(p / ((size_t)Wo * Ho));
    float best[8];
    uint8_t bi[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) { best[q] = -INFINITY; bi[q] = 0; }
    for (int s = 0; s < 4; ++s) {
        int hh = 2 * ho + s / 2, ww = 2 * wo + s % 2;
        uint4 v = *(const uint4 *)(x + (((size_t)n * H + hh) * W + ww) * C + c);
        const u16 *e = (const u16 *)&v;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float f = bf2f(e[q]);
            if (f > best[q]) { best[q] = f; bi[q] = (uint8_t)s; }
        }
    }
    uint4 r;
    u16 *er = (u16 *)&r;
    uint2 ri;
    uint8_t *eri = (uint8_t *)&ri;
#pragma unroll
    for (int q = 0; q < 8; ++q) { er[q] = f2bf(best[q]); eri[q] = bi[q]; }
    const size_t o = p * C + c;
    *(uint4 *)(y + o) = r;
    *(uint2 *)(idx + o) = ri;
}

__global__ void k_pool_bwd8(const u16 *__restrict__ dy, const uint8_t *__restrict__ idx,
                            u16 *__restrict__ dx, int N, int H, int W, int C)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;  // over dx, 8 channels each
    const int g = C / 8;
    size_t total = (size_t)N * H * W * g;
    if (i >= total) return;
    int c = (int)(i % g) * 8;
    size_t p = i / g;
    int w = (int)(p % W), h = (int)((p / W) % H), n = (int)(p / ((size_t)W * H));
    const int Ho = H / 2, Wo = W / 2;
    size_t o = (((size_t)n * Ho + h / 2) * Wo + w / 2) * C + c;
    const uint4 d = *(const uint4 *)(dy + o);
    const uint2 ix = *(const uint2 *)(idx + o);
    const u16 *ed = (const u16 *)&d;
    const uint8_t *ei = (const uint8_t *)&ix;
    const uint8_t me = (uint8_t)((h % 2) * 2 + (w % 2));
    uint4 r;
    u16 *er = (u16 *)&r;
#pragma unroll
    for (int q = 0; q < 8; ++q) er[q] = ei[q] == me ? ed[q] : (u16)0;
    *(uint4 *)(dx + p * C + c) = r;
}

__global__ void k_f32_to_bf16(const float *__restrict__ x, u16 *__restrict__ y, size_t n)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = f2bf(x[i]);
}

__global__ void k_bf16_to_f32(const u16 *__restrict__ x, float *__restrict__ y, size_t n)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = bf2f(x[i]);
}

// Adam on FP32 master weights; also refreshes the BF16 working copy.
__global__ void k_adam(float *__restrict__ w, float *__restrict__ mom, float *__restrict__ var,
                       const float *__restrict__ g, u16 *__restrict__ wb, size_t n, float lr,
                       float b1, float b2, float eps, float c1, float c2, float wd)
{
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float gi = g[i] + wd * w[i];
    float mi = b1 * mom[i] + (1.f - b1) * gi;
    float vi = b2 * var[i] + (1.f - b2) * gi * gi;
    mom[i] = mi;
    var[i] = vi;
    float upd = lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    float nw = w[i] - upd;
    w[i] = nw;
    if (wb) wb[i] = f2bf(nw);
}

// MSE over the first `used` of C channels of y (f32) against t (f32):
// per-block partial sums (f64) and the gradient dy = 2 (y - t) / count.
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ y,
                                             const float *__restrict__ t, float *__restrict__ dy,
                                             double *__restrict__ partial, size_t P, int C,
                                             int used, double inv_count)
{
    double acc = 0.0;
    for (int j = 0; j < 4; ++j) {
        size_t i = ((size_t)blockIdx.x * 4 + j) * 256 + threadIdx.x;
        if (i < P * C) {
            int c = (int)(i % C);
            float d = 0.f;
            if (c < used) {
                size_t p = i / C;
                d = y[i] - t[p * used + c];
                acc += (double)d * d;
            }
            if (dy) dy[i] = (float)(2.0 * inv_count) * d;
        }
    }
    __shared__ double sh[256];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}

inline unsigned blocks(size_t n) { return (unsigned)((n + 255) / 256); }

// Blocks of 256 threads of kernel k resident on the current device at once
// (its compute units times the blocks per unit that its registers and lds
// bytes of LDS allow), queried once per device, kernel and LDS size.
int resident_blocks(const void *k, size_t lds)
{
    static std::mutex mu;
    static std::map<std::tuple<int, const void *, size_t>, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = -1;
    const auto key = std::make_tuple(dev, k, lds);
    std::lock_guard<std::mutex> g(mu);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int per_cu = 0, cus = 0;
    if (!k || dev < 0 ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, 256, lds) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        per_cu <= 0 || cus <= 0) {
        (void)hipGetLastError();
        per_cu = 2;
        cus = 256;
    }
    return cache[key] = per_cu * cus;
}

// The weights of every chunk stay in LDS where two blocks per CU still fit.
// (From 80 output channels they never do.)
template <int NT>
void conv3_launch(const u16 *X, const u16 *Wk, const float *bias, void *y, int N, int H, int W,
                         int Cin, int Cout, int relu, int out_f32, const u16 *mask, hipStream_t s)
{
    const int nch = (Cin + kC3Chunk - 1) / kC3Chunk;
    const bool whole = !out_f32 && Cout == 16 * NT;
    const bool wall = NT <= 4 && whole && conv3_lds(NT, nch, true, 0) <= kC3LdsMax / 2;
    const size_t lds = conv3_lds(NT, nch, wall, out_f32);
    const int tx = (W + 31) / 32, ty = (H + kC3Rows - 1) / kC3Rows;
    const int ntile = N * tx * ty;
    const auto k = wall    ? k_conv3<NT, NT <= 4, true>
                   : whole ? k_conv3<NT, false, true>
                           : k_conv3<NT, false, false>;
    const int room = resident_blocks((const void *)k, lds) / 8;
    const unsigned grid = (unsigned)(8 * std::max(1, std::min(room, (ntile + 7) / 8)));
    hipLaunchKernelGGL(k, dim3(grid), dim3(256), (unsigned)lds, s, X, Wk, bias, y, H, W, Cin, Cout, relu,
                       out_f32, mask, tx, ty, ntile);
}

}  // namespace

// LDS bytes k_conv_fwd<NT> uses for a layer: the largest staged input window
// and, unless an FP32 tile goes straight from the registers, the output tile.
static size_t conv_fwd_lds(int nt, int Cin, int ks, int out_f32)
{
    const int mt = conv_mt(nt), tr = 2 * mt, halo = ks == 3 ? 1 : 0;
    const size_t cc = (size_t)std::min(kConvChunk, Cin);
    const size_t win = (size_t)(tr + 2 * halo) * (32 + 2 * halo) * (cc + 8) * 2;
    const size_t tile = (size_t)tr * 32 * nt * 16 * (out_f32 ? 4 : 2);
    const bool tile_in_lds = !(out_f32 && tile > (size_t)kConvLds);
    return std::max(win, tile_in_lds ? tile : (size_t)0);
}

extern "C" {

const char *dect_nn_last_error(void) { return g_nn_err; }

static dect_status conv_fwd_launch(const void *x, const void *w, const float *bias,
                                   const void *mask, void *y, int32_t N, int32_t H, int32_t W,
                                   int32_t Cin, int32_t Cout, int32_t ksize, int32_t relu,
                                   int32_t out_f32, void *stream)
{
    if (!x || !w || !y || N <= 0 || H <= 0 || W <= 0 || Cin <= 0 || Cout <= 0)
        return nn_fail(DECT_ERR_INVALID_ARG, "conv_fwd: bad arguments");
    if (Cin % 8 != 0 || Cout > 256 || (ksize != 1 && ksize != 3))
        return nn_fail(DECT_ERR_INVALID_ARG, "conv_fwd: Cin % 8, Cout <= 256, ksize in {1,3}");
    if (mask && (((uintptr_t)mask & 15) != 0))
        return nn_fail(DECT_ERR_INVALID_ARG, "conv_fwd: mask must be 16-byte aligned");
    const int NT = (Cout + 15) / 16;
    hipStream_t s = (hipStream_t)stream;
    const u16 *X = (const u16 *)x, *Wk = (const u16 *)w, *Mk = (const u16 *)mask;
    if (ksize == 3 && conv3_use(NT, Cin, W)) {
        switch (NT) {
#define CASE3(nt) \
    case nt: conv3_launch<nt>(X, Wk, bias, y, N, H, W, Cin, Cout, relu, out_f32, Mk, s); break;
            CASE3(1) CASE3(2) CASE3(3) CASE3(4) CASE3(5) CASE3(6) CASE3(7) CASE3(8)
#undef CASE3
            default: return nn_fail(DECT_ERR_INVALID_ARG, "conv_fwd: no 3x3 kernel for this width");
        }
        NN_HIP(hipGetLastError());
        return DECT_OK;
    }
    switch (NT) {
#define CASE(nt)                                                                         \
    case nt: {                                                                           \
        dim3 grid((W + 31) / 32, (H + 2 * conv_mt(nt) - 1) / (2 * conv_mt(nt)), N);      \
        hipLaunchKernelGGL(k_conv_fwd<nt>, grid, dim3(256),                                \
                           (unsigned)conv_fwd_lds(nt, Cin, ksize, out_f32), s, X, Wk, bias, y, \
                           H, W, Cin, Cout, ksize, relu, out_f32, Mk);                   \
    } break;
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
        CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14) CASE(15) CASE(16)
#undef CASE
    }
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_conv_fwd(const void *x, const void *w, const float *bias, void *y, int32_t N,
                             int32_t H, int32_t W, int32_t Cin, int32_t Cout, int32_t ksize,
                             int32_t relu, int32_t out_f32, void *stream)
{
    return conv_fwd_launch(x, w, bias, nullptr, y, N, H, W, Cin, Cout, ksize, relu, out_f32,
                           stream);
}

dect_status dect_nn_conv_fwd_masked(const void *x, const void *w, const float *bias,
                                    const void *mask, void *y, int32_t N, int32_t H, int32_t W,
                                    int32_t Cin, int32_t Cout, int32_t ksize, int32_t relu,
                                    int32_t out_f32, void *stream)
{
    if (!mask) return nn_fail(DECT_ERR_INVALID_ARG, "conv_fwd_masked: null mask");
    return conv_fwd_launch(x, w, bias, mask, y, N, H, W, Cin, Cout, ksize, relu, out_f32, stream);
}

// Tiles per weight-gradient block: TMS output-channel x TNS WN input-channel
// tiles (taps x TMS x TNS accumulators of four floats per lane: at most 108
// for 3x3; staged rows within 64 KB of LDS for 1x1, 80 KB for 3x3: two blocks
// per CU), the first entry of a fixed list that divides the layer's tile
// counts.  For 3x3 one input tile per wave, as many waves apart as divide the
// layer's: four (64 -> 32 at 8 x 512^2) read dZ once and take 112 us, one took
// 264.  (3, 1, 4) spills its registers.
//
// On small planes the partial sums' bytes allow few chunks, and the first entry
// may leave most of the chip idle: the first that gives enough blocks is taken,
// or the one that gives most.  Below kWgXcdChunks chunks the blocks go to the XCDs
// as they come (a chunk's splits on one XCD, fewer than eight chunks use as many
// XCDs), and narrower tiles pay longer.  Event times with the partial sums (us),
// with a wave per row and one input tile / the first entry, by XCD / this: 4 x 32^2
// 128 -> 128 24 / 36 / 21, 16^2 64 -> 64 16 / 21 / 14, 300 x 3 128 -> 64 97 / 224 / 96;
// both sides of the lines: 4 x 64^2 128 -> 128 (16 chunks) 128 blocks 27.9, 256
// 24.6, 512 27.2; 8 x 32^2 256 -> 128 (8 chunks) 128 blocks 38.5, 256 31.4, 512 29.7, 1024
// 33.6; 8 chunks by XCD 25.5, as they come 24.8, 16 chunks 20.6 and 21.2.
constexpr size_t kWgEnough = 200, kWgEnoughFew = 500;
constexpr int kWgXcdChunks = 16;

struct WgTiles {
    int tms, tns, wn;
};

#define WG_KERNELS(WG)                                                                          \
    WG(3, 2, 1, 4) WG(3, 1, 1, 4) WG(3, 2, 1, 2) WG(3, 3, 1, 2) WG(3, 1, 1, 2) WG(3, 2, 1, 1)   \
    WG(3, 3, 1, 1) WG(3, 1, 1, 1)                                                               \
    WG(1, 4, 2, 1) WG(1, 3, 3, 1) WG(1, 2, 3, 1) WG(1, 3, 2, 1) WG(1, 4, 1, 1) WG(1, 2, 2, 1)   \
    WG(1, 3, 1, 1) WG(1, 1, 3, 1) WG(1, 2, 1, 1) WG(1, 1, 2, 1) WG(1, 1, 1, 1)

using WgKernel = void (*)(const u16 *, const u16 *, float *, int, int, int, int, int, int, int, int,
                          int, int, int, size_t, size_t);

static WgKernel wgrad_kernel(int ks, const WgTiles &t)
{
#define WG(k, a, b, c) \
    if (ks == k && t.tms == a && t.tns == b && t.wn == c) return k_wgrad<k, a, b, c>;
    WG_KERNELS(WG)
#undef WG
    return nullptr;
}

struct WgradPlan {
    WgKernel kernel;
    int nsm, nsn, nstrip, nrc, kst, nchunk, nseg, by_xcd;
    size_t lds, len, pstride;
};

static WgradPlan wgrad_plan_of(const WgTiles &t, int N, int H, int W, int Cin, int Cout, int ksize)
{
    WgradPlan q;
    const int CoutP = (Cout + 15) / 16 * 16, CinP = (Cin + 15) / 16 * 16;
    q.kernel = wgrad_kernel(ksize, t);
    q.nsm = CoutP / 16 / t.tms;
    q.nsn = CinP / 16 / (t.tns * t.wn);
    const int nsplit = q.nsm * q.nsn;
    q.nstrip = (W + kWgPix - 1) / kWgPix;
    const size_t RG = (size_t)(H + 3) / 4;  // steps of four rows per strip
    const size_t strips = (size_t)N * q.nstrip;
    q.len = (size_t)ksize * ksize * CoutP * Cin;
    q.pstride = q.len + CoutP;
    const size_t stage =
        ((size_t)4 * 16 * t.tms + (size_t)wg_xrows(ksize) * 16 * t.tns * t.wn) * kWgLD * sizeof(u16);
    const size_t red = (size_t)(4 - t.wn) * t.tms * t.tns * 4 * 64 * sizeof(float);
    q.lds = std::max(stage, red);
    // one round of resident blocks, fewer while the partials would outweigh
    // twice the layer's own bytes
    const size_t units = strips * RG * nsplit;
    const size_t target =
        units <= kWgEnough ? kWgEnough : (size_t)resident_blocks((const void *)q.kernel, q.lds);
    size_t kst = std::max<size_t>(1, (units + target - 1) / target);
    const double in_bytes = (double)N * H * W * (Cin + Cout) * 2;
    while (kst < RG && (double)strips * ((RG + kst - 1) / kst) * q.pstride * 4 > 2.0 * in_bytes)
        kst *= 2;
    kst = std::min(kst, RG);
    q.kst = (int)kst;
    q.nrc = (int)((RG + kst - 1) / kst);
    q.nchunk = (int)(strips * q.nrc);
    q.nseg = sum_segments(q.nchunk, q.pstride);
    q.by_xcd = q.nchunk >= kWgXcdChunks;
    return q;
}

static WgradPlan wgrad_plan(int N, int H, int W, int Cin, int Cout, int ksize)
{
    static const WgTiles k3[] = {{2, 1, 4}, {2, 1, 2}, {3, 1, 2}, {1, 1, 4}, {1, 1, 2},
                                 {2, 1, 1}, {3, 1, 1}, {1, 1, 1}};
    static const WgTiles k1[] = {{4, 2, 1}, {3, 3, 1}, {2, 3, 1}, {3, 2, 1}, {4, 1, 1}, {2, 2, 1},
                                 {3, 1, 1}, {1, 3, 1}, {2, 1, 1}, {1, 2, 1}, {1, 1, 1}};
    const WgTiles *list = ksize == 3 ? k3 : k1;
    const int n = ksize == 3 ? 8 : 11, TM = (Cout + 15) / 16, TN = (Cin + 15) / 16;
    WgradPlan best{};
    size_t most = 0;
    for (int i = 0; i < n; ++i) {
        if (TM % list[i].tms != 0 || TN % (list[i].tns * list[i].wn) != 0) continue;
        const WgradPlan q = wgrad_plan_of(list[i], N, H, W, Cin, Cout, ksize);
        const size_t blocks = (size_t)q.nchunk * q.nsm * q.nsn;
        if (blocks > most) {
            most = blocks;
            best = q;
        }
        if (most >= (q.by_xcd ? kWgEnough : kWgEnoughFew) || ksize == 1) break;
    }
    return best;
}

static size_t wgrad_bytes(const WgradPlan &q)
{
    return ((size_t)q.nchunk + q.nseg) * q.pstride * sizeof(float);
}

size_t dect_nn_wgrad_workspace(int32_t N, int32_t H, int32_t W, int32_t Cin, int32_t Cout,
                               int32_t ksize)
{
    if (N <= 0 || H <= 0 || W <= 0 || Cin <= 0 || Cout <= 0 || (ksize != 1 && ksize != 3))
        return 0;
    return wgrad_bytes(wgrad_plan(N, H, W, Cin, Cout, ksize));
}

dect_status dect_nn_conv_wgrad(const void *dz, const void *x, float *dw, float *db, int32_t N,
                               int32_t H, int32_t W, int32_t Cin, int32_t Cout, int32_t ksize,
                               void *workspace, size_t ws_bytes, void *stream)
{
    if (!dz || !x || !dw || !db || !workspace || N <= 0 || H <= 0 || W <= 0)
        return nn_fail(DECT_ERR_INVALID_ARG, "conv_wgrad: bad arguments");
    if (Cin <= 0 || Cout <= 0 || Cin % 8 != 0 || Cout % 8 != 0 || Cin > 256 || Cout > 256 ||
        (ksize != 1 && ksize != 3))
        return nn_fail(DECT_ERR_INVALID_ARG, "conv_wgrad: Cin, Cout % 8 and <= 256");
    const WgradPlan q = wgrad_plan(N, H, W, Cin, Cout, ksize);
    if (ws_bytes < wgrad_bytes(q))
        return nn_fail(DECT_ERR_INVALID_ARG, "conv_wgrad: workspace too small");
    const size_t nblk = (q.by_xcd ? ((size_t)q.nchunk + 7) / 8 * 8 : q.nchunk) * q.nsm * q.nsn;
    if (nblk > 0x7fffffffu) return nn_fail(DECT_ERR_INVALID_ARG, "conv_wgrad: problem too large");
    float *part = (float *)workspace;
    float *seg = part + (size_t)q.nchunk * q.pstride;
    hipStream_t s = (hipStream_t)stream;
    if (!q.kernel) return nn_fail(DECT_ERR_INVALID_ARG, "conv_wgrad: no kernel for this tiling");
    hipLaunchKernelGGL(q.kernel, dim3((unsigned)nblk), dim3(256), (unsigned)q.lds, s, (const u16 *)dz,
                       (const u16 *)x, part, H, W, Cin, Cout, q.nstrip, N * q.nstrip, q.nrc, q.kst, q.nsn,
                       q.nsm * q.nsn, q.by_xcd, q.len, q.pstride);
    NN_HIP(hipGetLastError());
    const int L = (q.nchunk + q.nseg - 1) / q.nseg;
    hipLaunchKernelGGL(k_sum_seg, dim3(blocks(q.pstride), q.nseg), dim3(256), 0, s, part, seg,
                       q.nchunk, q.pstride, L);
    hipLaunchKernelGGL(k_sum_out, dim3(blocks(q.pstride)), dim3(256), 0, s, seg, dw, db, q.nseg,
                       q.len, q.pstride);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_weight_flip(const void *w, void *wd, int32_t Cin, int32_t Cout, int32_t ksize,
                                void *stream)
{
    if (!w || !wd || Cin <= 0 || Cout <= 0) return nn_fail(DECT_ERR_INVALID_ARG, "weight_flip");
    const int taps = ksize * ksize;
    const int CoutP = (Cout + 15) / 16 * 16, CinP = (Cin + 15) / 16 * 16;
    size_t total = (size_t)taps * CinP * Cout;
    hipLaunchKernelGGL(k_wflip, dim3(blocks(total)), dim3(256), 0, (hipStream_t)stream,
                       (const u16 *)w, (u16 *)wd, taps, Cin, Cout, CoutP, CinP);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

static bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

dect_status dect_nn_relu_bwd(const void *dy, const void *y, void *dz, size_t n, void *stream)
{
    if (n == 0) return DECT_OK;
    if (n % 8 == 0 && aligned16(dy) && aligned16(y) && aligned16(dz))
        hipLaunchKernelGGL(k_relu_bwd8, dim3(blocks(n / 8)), dim3(256), 0, (hipStream_t)stream,
                           (const uint4 *)dy, (const uint4 *)y, (uint4 *)dz, n / 8);
    else
        hipLaunchKernelGGL(k_relu_bwd, dim3(blocks(n)), dim3(256), 0, (hipStream_t)stream,
                           (const u16 *)dy, (const u16 *)y, (u16 *)dz, n);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_pool(const void *x, void *y, void *idx, int32_t N, int32_t H, int32_t W,
                         int32_t C, int32_t backward, void *stream)
{
    if (H % 2 || W % 2) return nn_fail(DECT_ERR_INVALID_ARG, "pool: H and W must be even");
    hipStream_t s = (hipStream_t)stream;
    const bool v8 = C % 8 == 0 && aligned16(x) && aligned16(y) && ((uintptr_t)idx & 7) == 0;
    if (!backward) {
        size_t total = (size_t)N * (H / 2) * (W / 2) * C;
        if (v8)
            hipLaunchKernelGGL(k_pool_fwd8, dim3(blocks(total / 8)), dim3(256), 0, s,
                               (const u16 *)x, (u16 *)y, (uint8_t *)idx, N, H, W, C);
        else
            hipLaunchKernelGGL(k_pool_fwd, dim3(blocks(total)), dim3(256), 0, s, (const u16 *)x,
                               (u16 *)y, (uint8_t *)idx, N, H, W, C);
    } else {  // x = dy (pooled), y = dx (full)
        size_t total = (size_t)N * H * W * C;
        if (v8)
            hipLaunchKernelGGL(k_pool_bwd8, dim3(blocks(total / 8)), dim3(256), 0, s,
                               (const u16 *)x, (const uint8_t *)idx, (u16 *)y, N, H, W, C);
        else
            hipLaunchKernelGGL(k_pool_bwd, dim3(blocks(total)), dim3(256), 0, s, (const u16 *)x,
                               (const uint8_t *)idx, (u16 *)y, N, H, W, C);
    }
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_shuffle(const void *src, void *dst, int32_t N, int32_t Hin, int32_t Win,
                            int32_t C, int32_t inverse, void *stream)
{
    size_t total = (size_t)N * 4 * Hin * Win * C;
    if (C % 8 == 0 && aligned16(src) && aligned16(dst))
        hipLaunchKernelGGL(k_shuffle8, dim3(blocks(total / 8)), dim3(256), 0, (hipStream_t)stream,
                           (const uint4 *)src, (uint4 *)dst, N, Hin, Win, C, inverse);
    else
        hipLaunchKernelGGL(k_shuffle, dim3(blocks(total)), dim3(256), 0, (hipStream_t)stream,
                           (const u16 *)src, (u16 *)dst, N, Hin, Win, C, inverse);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_concat(void *a, void *b, void *z, size_t P, int32_t C1, int32_t C2,
                           int32_t inverse, void *stream)
{
    size_t total = P * (size_t)(C1 + C2);
    if (C1 % 8 == 0 && C2 % 8 == 0 && aligned16(a) && aligned16(b) && aligned16(z))
        hipLaunchKernelGGL(k_concat8, dim3(blocks(total / 8)), dim3(256), 0, (hipStream_t)stream,
                           (uint4 *)a, (uint4 *)b, (uint4 *)z, P, C1, C2, inverse);
    else
        hipLaunchKernelGGL(k_concat, dim3(blocks(total)), dim3(256), 0, (hipStream_t)stream,
                           (u16 *)a, (u16 *)b, (u16 *)z, P, C1, C2, inverse);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_shuffle_concat(void *t, void *s, void *z, int32_t N, int32_t Hin, int32_t Win,
                                   int32_t C1, int32_t C2, int32_t inverse, void *stream)
{
    if (!t || !s || !z || N <= 0 || Hin <= 0 || Win <= 0 || C1 <= 0 || C2 <= 0 ||
        C1 % 8 != 0 || C2 % 8 != 0 || !aligned16(t) || !aligned16(s) || !aligned16(z))
        return nn_fail(DECT_ERR_INVALID_ARG,
                       "shuffle_concat: channels must be positive multiples of 8, pointers "
                       "16-byte aligned");
    const size_t pieces = (size_t)N * 4 * Hin * Win * ((C1 + C2) / 8);
    hipLaunchKernelGGL(k_shuffle_concat8, dim3(blocks(pieces)), dim3(256), 0,
                       (hipStream_t)stream, (uint4 *)t, (uint4 *)s, (uint4 *)z, N, Hin, Win, C1,
                       C2, inverse);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_add(const void *a, const void *b, void *z, size_t n, void *stream)
{
    if (n == 0) return DECT_OK;
    if (n % 8 == 0 && aligned16(a) && aligned16(b) && aligned16(z))
        hipLaunchKernelGGL(k_add8, dim3(blocks(n / 8)), dim3(256), 0, (hipStream_t)stream,
                           (const uint4 *)a, (const uint4 *)b, (uint4 *)z, n / 8);
    else
        hipLaunchKernelGGL(k_add, dim3(blocks(n)), dim3(256), 0, (hipStream_t)stream,
                           (const u16 *)a, (const u16 *)b, (u16 *)z, n);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_add_relu_bwd(const void *a, const void *b, const void *y, void *z, size_t n,
                                 void *stream)
{
    if (n == 0) return DECT_OK;
    if (!a || !b || !y || !z) return nn_fail(DECT_ERR_INVALID_ARG, "add_relu_bwd: null argument");
    if (n % 8 == 0 && aligned16(a) && aligned16(b) && aligned16(y) && aligned16(z))
        hipLaunchKernelGGL(k_add_relu_bwd8, dim3(blocks(n / 8)), dim3(256), 0, (hipStream_t)stream,
                           (const uint4 *)a, (const uint4 *)b, (const uint4 *)y, (uint4 *)z, n / 8);
    else
        hipLaunchKernelGGL(k_add_relu_bwd, dim3(blocks(n)), dim3(256), 0, (hipStream_t)stream,
                           (const u16 *)a, (const u16 *)b, (const u16 *)y, (u16 *)z, n);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_convert(const void *src, void *dst, size_t n, int32_t to_bf16, void *stream)
{
    if (n == 0) return DECT_OK;
    if (to_bf16)
        hipLaunchKernelGGL(k_f32_to_bf16, dim3(blocks(n)), dim3(256), 0, (hipStream_t)stream,
                           (const float *)src, (u16 *)dst, n);
    else
        hipLaunchKernelGGL(k_bf16_to_f32, dim3(blocks(n)), dim3(256), 0, (hipStream_t)stream,
                           (const u16 *)src, (float *)dst, n);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

dect_status dect_nn_adam(float *w, float *m, float *v, const float *g, void *w_bf16, size_t n,
                         double lr, double beta1, double beta2, double eps, int32_t step,
                         double weight_decay, void *stream)
{
    if (n == 0) return DECT_OK;
    if (step < 1) return nn_fail(DECT_ERR_INVALID_ARG, "adam: step counts from 1");
    float c1 = (float)(1.0 - std::pow(beta1, step)), c2 = (float)(1.0 - std::pow(beta2, step));
    hipLaunchKernelGGL(k_adam, dim3(blocks(n)), dim3(256), 0, (hipStream_t)stream, w, m, v, g,
                       (u16 *)w_bf16, n, (float)lr, (float)beta1, (float)beta2, (float)eps, c1,
                       c2, (float)weight_decay);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

size_t dect_nn_mse_partials(size_t P, int32_t C) { return (P * C + 1023) / 1024; }

dect_status dect_nn_mse(const float *y, const float *t, float *dy, double *partial, size_t P,
                        int32_t C, int32_t used, void *stream)
{
    size_t nb = dect_nn_mse_partials(P, C);
    double inv = 1.0 / ((double)P * used);
    hipLaunchKernelGGL(k_mse, dim3((unsigned)nb), dim3(256), 0, (hipStream_t)stream, y, t, dy,
                       partial, P, C, used, inv);
    NN_HIP(hipGetLastError());
    return DECT_OK;
}

}  // extern "C"
