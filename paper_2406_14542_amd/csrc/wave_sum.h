// Sums over the lanes of a wave for the adjoint Legendre and Wigner-d steps.
//
// v_mfma_f64_4x4x4_4b with A_b[i][k] = [i = l mod 4] takes the lane values as they lie (B_b[k][j] in
// lane j + 4 b + 16 k) and adds those of the lanes x, x + 16, x + 32, x + 48 into lane x + 16 i of D,
// so the MFMAs of four consecutive l leave 16 partial sums of each in one register; wave_rows
// then sums four such registers within the rows of 16 lanes.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace nusht {
namespace {

// the double of the lane that DPP control CTRL names (within rows of 16 lanes)
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}

constexpr int kDppXor1 = 0xB1;  // quad_perm [1, 0, 3, 2]
constexpr int kDppXor2 = 0x4E;  // quad_perm [2, 3, 0, 1]
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128;

// the sum of q[x & 3] over the row's 16 lanes, in lane x of each row
__device__ inline double wave_rows(const double (&q)[4], int x)
{
    const bool o1 = x & 1, o2 = x & 2;
    const double a = (o1 ? q[1] : q[0]) + dpp_f64<kDppXor1>(o1 ? q[0] : q[1]);
    const double b = (o1 ? q[3] : q[2]) + dpp_f64<kDppXor1>(o1 ? q[2] : q[3]);
    double v = (o2 ? b : a) + dpp_f64<kDppXor2>(o2 ? a : b);
    v += dpp_f64<kDppRor4>(v);
    v += dpp_f64<kDppRor8>(v);
    return v;
}

}  // namespace
}  // namespace nusht
