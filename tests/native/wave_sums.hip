// wave_sums.hip -- wave_sum_many on the GPU, for the tests: one wavefront
// sums K values per lane (in[k * 64 + lane]) and every lane stores the sum and
// the index it ends with.
#include <hip/hip_runtime.h>

#include <utility>

#include "wave.hpp"

template <int K>
__global__ __launch_bounds__(64) void wave_sums_kernel(const double *__restrict__ in, double *__restrict__ sum,
                                                       int *__restrict__ index)
{
    double v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = in[k * 64 + threadIdx.x];
    int own = 0;
    sum[threadIdx.x] = spx::wave_sum_many<K>(v, &own);
    index[threadIdx.x] = own;
}

template <int... I>
static bool launch(int count, const double *in, double *sum, int *index, std::integer_sequence<int, I...>)
{
    return ((count == I + 1 && (wave_sums_kernel<I + 1><<<1, 64>>>(in, sum, index), true)) || ...);
}

// 0, or -1 for a count outside 1..64 or a failed launch.
extern "C" int wave_sums(int count, const double *in, double *sum, int *index)
{
    if (!launch(count, in, sum, index, std::make_integer_sequence<int, 64>())) return -1;
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
