// wave_many.hpp -- sums of many values over a wavefront at once.
//
// The includer declares lane_id() and exchange<Stride>() (wave.hpp does; a
// host emulation may supply its own), so this file needs nothing of HIP.
#pragma once

namespace spx {

// Index of a lane that holds the sum of none of the K values.
constexpr int kWaveSumNone = 64;

// Wavefront sums of K <= 64 values at once: at each stride a lane keeps half
// of the values it still holds and adds its partner's copies of them, so K
// sums take about K exchanges instead of 6 K. Returns the sum of value *k,
// *k starting at 0. An odd half is padded with a zero; `real` counts the
// values a lane holds that are not padding, and a lane left with padding
// alone gets *k = kWaveSumNone: every index below K belongs to lanes that
// hold that value's sum.
template <int K, int Stride = 32, typename T>
__device__ __forceinline__ T wave_sum_many(const T (&v)[K], int *k, int real = K)
{
    if constexpr (K == 1) {
        T t = v[0] + exchange<Stride>(v[0]);
        if constexpr (Stride > 1) {
            const T one[1] = {t};
            return wave_sum_many<1, Stride / 2>(one, k, real);
        }
        if (real == 0) *k = kWaveSumNone;
        return t;
    } else {
        constexpr int kHalf = (K + 1) / 2;
        const bool hi = (lane_id() & Stride) != 0;
        T t[kHalf];
#pragma unroll
        for (int i = 0; i < kHalf; ++i) {
            const T b = i + kHalf < K ? v[i + kHalf < K ? i + kHalf : 0] : T(0);
            const T keep = hi ? b : v[i], send = hi ? v[i] : b;
            t[i] = keep + exchange<Stride>(send);
        }
        if (hi) *k += kHalf;
        if (hi) real = real > kHalf ? real - kHalf : 0;
        else real = real < kHalf ? real : kHalf;
        if constexpr (Stride > 1) return wave_sum_many<kHalf, Stride / 2>(t, k, real);
        if (real == 0) *k = kWaveSumNone;
        return t[0];
    }
}

}  // namespace spx
