// FP64 sums over a wavefront and a block in a fixed order, by VALU lane moves;
// the order of a wavefront's own LDS accesses.
#pragma once

#include <hip/hip_runtime.h>

namespace dect {

// Orders a wavefront's LDS accesses before and after it (the hardware takes
// them in order; no instruction).
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v of this lane moved along the wavefront by the DPP control CTRL (rows of 16
// lanes not in ROW_MASK, and lanes whose source lies outside their row, get
// 0); an FP64 value moves as its two 32-bit halves
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_f64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROW_MASK, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROW_MASK, 0xf, true);
    return __hiloint2double(hi, lo);
}

// Sum of v over the 64 lanes of a full wavefront, in a fixed order, returned
// to every lane: a prefix sum within each row of 16 lanes (shifts by 1, 2, 4
// and 8 lanes), then rows 1 and 3 add the total of the row before them (the
// row's last lane, broadcast), and rows 2 and 3 add lane 31; lane 63 then
// holds the total, which is read back as a wavefront-uniform value.  Every
// step is a VALU lane move, with no LDS round trip.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_f64<0x111>(v);       // row_shr:1
    v += dpp_f64<0x112>(v);       // row_shr:2
    v += dpp_f64<0x114>(v);       // row_shr:4
    v += dpp_f64<0x118>(v);       // row_shr:8
    v += dpp_f64<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_f64<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

// x + y where lanes 0-31 take x of lanes l and l + 32, lanes 32-63 y of lanes
// l - 32 and l (permlane32 swap of the upper half of x with the lower half of
// y); with ROWS16, rows of 16 lanes instead: even rows take x of rows r and
// r + 1, odd rows y of rows r - 1 and r
template <bool ROWS16>
__device__ __forceinline__ double swap_add(double x, double y)
{
    const unsigned xl = (unsigned)__double2loint(x), xh = (unsigned)__double2hiint(x);
    const unsigned yl = (unsigned)__double2loint(y), yh = (unsigned)__double2hiint(y);
    if constexpr (ROWS16) {
        const auto lo = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
        return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    } else {
        const auto lo = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
        return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    }
}

// Fixed-order sum over a 256-thread block of NV values; every thread gets
// the totals in `out` (LDS).  Ends with a barrier.  For 3 to 8 values the
// wavefront reduces them together: each exchange step halves the values a
// lane holds and doubles the lanes each partial covers (wave halves, then
// row pairs, then the two halves of each row: 8 values, 4, 2, 1), and a
// butterfly over the last 8 lanes completes each sum, so that lane 8 j holds
// value j's wavefront total.  The four wavefronts' totals are added in
// wavefront order.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double *out)
{
    __shared__ double sh[4][NV];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if constexpr (NV >= 3 && NV <= 8) {
        double a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = j < NV ? v[j] : 0.0;
        double b[4], c[2];
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = swap_add<false>(a[j], a[j + 4]);
#pragma unroll
        for (int j = 0; j < 2; ++j) c[j] = swap_add<true>(b[j], b[j + 2]);
        // lanes with bit 3 clear keep c[0] and send c[1] to lane l ^ 8
        // (row_ror:8), the others the reverse
        const bool up = (lane & 8) != 0;
        const double keep = up ? c[1] : c[0], send = up ? c[0] : c[1];
        double d = keep + dpp_f64<0x128>(send);
        d += dpp_f64<0xB1>(d);   // quad_perm [1, 0, 3, 2]
        d += dpp_f64<0x4E>(d);   // quad_perm [2, 3, 0, 1]
        d += dpp_f64<0x141>(d);  // row_half_mirror
        if ((lane & 7) == 0 && (lane >> 3) < NV) sh[wid][lane >> 3] = d;
    } else {
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = wave_sum(v[i]);
        if (lane == 0)
#pragma unroll
            for (int i = 0; i < NV; ++i) sh[wid][i] = v[i];
    }
    __syncthreads();
    if ((int)threadIdx.x < NV) {
        int t = threadIdx.x;
        out[t] = ((sh[0][t] + sh[1][t]) + sh[2][t]) + sh[3][t];
    }
    __syncthreads();
}

}  // namespace dect
