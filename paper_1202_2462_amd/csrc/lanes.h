// Sums over the 64 lanes of a wave without LDS: lane permutations on the vector
// units (DPP within a row of 16 lanes, the gfx950 row swaps across rows).
#pragma once

#include <hip/hip_runtime.h>

namespace mgdd {

// v moved by a DPP control (0xB1: lane ^ 1, 0x4E: lane ^ 2 within a quad;
// 0x141: mirrored within 8 lanes; 0x128: rotated by 8 within 16 lanes)
template <int CTRL> __device__ inline float dpp_mov(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
template <int CTRL> __device__ inline double dpp_mov(double v) {
    const int2 i = __builtin_bit_cast(int2, v);
    int2 r;
    r.x = __builtin_amdgcn_update_dpp(0, i.x, CTRL, 0xF, 0xF, false);
    r.y = __builtin_amdgcn_update_dpp(0, i.y, CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, r);
}

// a + b with the rows exchanged: in the lanes of even rows (rows of R = 32 or
// 16 lanes) a summed over the row and the next one, in those of odd rows b
template <int R> __device__ inline float swap_add(float a, float b) {
    const unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    const auto r = R == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                           : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
template <int R> __device__ inline double swap_add(double a, double b) {
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    const auto r = R == 32 ? __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false)
                           : __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
    const auto s = R == 32 ? __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false)
                           : __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    const uint2 p = make_uint2(r[0], s[0]), q = make_uint2(r[1], s[1]);
    return __builtin_bit_cast(double, p) + __builtin_bit_cast(double, q);
}

// the sum of v over 8 lanes (lane / 8 equal), in each of them
template <typename T> __device__ inline T sum_of_8(T v) {
    v += dpp_mov<0x141>(v);
    v += dpp_mov<0x4E>(v);
    return v + dpp_mov<0xB1>(v);
}

// eight sums over the wave at once: lane l returns the sum of v[l / 8] over
// the 64 lanes. Each step adds two halves of the lanes and keeps half of the
// values in each, so 8 sums take 10 additions, not 48.
template <typename T> __device__ inline T wave_sum8(const T *v) {
    T a[4], b[2];
#pragma unroll
    for (int i = 0; i < 4; i++) a[i] = swap_add<32>(v[i], v[4 + i]);
#pragma unroll
    for (int i = 0; i < 2; i++) b[i] = swap_add<16>(a[i], a[2 + i]);
    const bool odd = threadIdx.x & 8;
    return sum_of_8((odd ? b[1] : b[0]) + dpp_mov<0x128>(odd ? b[0] : b[1]));
}

// the sum of v over the wave, in every lane
template <typename T> __device__ inline T wave_sum1(T v) {
    v = swap_add<32>(v, v);
    v = swap_add<16>(v, v);
    v += dpp_mov<0x128>(v);
    return sum_of_8(v);
}

// LDS written by lanes of this wave is read by others of it after this
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace mgdd
