// corr_wave.h -- sums of doubles over the 64 lanes of a wave, in a fixed order.
#ifndef CORR_WAVE_H
#define CORR_WAVE_H

#include <hip/hip_runtime.h>

namespace corr {

// v of the lane whose index differs in one bit (8, 4, 2 or 1).
template <int BIT> __device__ __forceinline__ double lane_xor(double v)
{
    union { double d; int w[2]; } u, o;
    u.d = v;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if constexpr (BIT == 8) o.w[i] = __builtin_amdgcn_update_dpp(0, u.w[i], 0x128, 0xf, 0xf, true); // row_ror:8
        else if constexpr (BIT == 4) o.w[i] = __builtin_amdgcn_ds_swizzle(u.w[i], 0x101f);            // xor 4
        else if constexpr (BIT == 2) o.w[i] = __builtin_amdgcn_update_dpp(0, u.w[i], 0x4e, 0xf, 0xf, true);
        else o.w[i] = __builtin_amdgcn_update_dpp(0, u.w[i], 0xb1, 0xf, 0xf, true);
    }
    return o.d;
}

// a of the lanes with the bit (32 or 16) clear and b of those with it set,
// each added to the same value of the lane that differs in that bit.
template <int BIT> __device__ __forceinline__ double pair_fold(double a, double b)
{
    union { double d; unsigned w[2]; } x, y;
    x.d = a;
    y.d = b;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if constexpr (BIT == 32) {
            const auto r = __builtin_amdgcn_permlane32_swap(x.w[i], y.w[i], false, false);
            x.w[i] = r[0];
            y.w[i] = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane16_swap(x.w[i], y.w[i], false, false);
            x.w[i] = r[0];
            y.w[i] = r[1];
        }
    }
    return x.d + y.d;
}

// Sums of N = 8 or 16 values over the wave's 64 lanes: lane l returns the sum
// of v[l / (64 / N)].  Every sum is the binary tree over lane distances 32,
// 16, .., 1, but after each exchange a lane carries on only half of the
// values: 7 (or 15) exchanges and 3 (2) more instead of 6 for each value.
template <int N> __device__ __forceinline__ double wave_sums(const double (&v)[N])
{
    static_assert(N == 8 || N == 16, "8 or 16 values");
    const int lane = (int)(threadIdx.x & 63);
    double a[N / 2], b[N / 4];
#pragma unroll
    for (int j = 0; j < N / 2; ++j) a[j] = pair_fold<32>(v[j], v[j + N / 2]);
#pragma unroll
    for (int j = 0; j < N / 4; ++j) b[j] = pair_fold<16>(a[j], a[j + N / 4]);
    double c[N / 8];
    const bool up8 = lane & 8;
#pragma unroll
    for (int j = 0; j < N / 8; ++j)
        c[j] = (up8 ? b[j + N / 8] : b[j]) + lane_xor<8>(up8 ? b[j] : b[j + N / 8]);
    double s;
    if constexpr (N == 16) {
        const bool up4 = lane & 4;
        s = (up4 ? c[1] : c[0]) + lane_xor<4>(up4 ? c[0] : c[1]);
    } else {
        s = c[0] + lane_xor<4>(c[0]);
    }
    s += lane_xor<2>(s);
    s += lane_xor<1>(s);
    return s;
}

} // namespace corr

#endif
