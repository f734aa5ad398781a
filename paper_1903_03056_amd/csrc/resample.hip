// Moving fields between species-specific velocity grids.
//
// With an independent grid per species (the remedy named in the remark after
// eq. (domain), Sec. 4) the pair (i, j) is evaluated on the wider of the two boxes.  A
// field is carried from one grid to another by its real trigonometric interpolant,
// which is a product of three one-dimensional maps T (N x N, host-built): one pass per
// axis, each output point a length-N dot product of a row of T with an input pencil.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "plan.hpp"

namespace dgfs {
namespace {

// out[b][..a..] (+)= sum_m T[a][m] in[b][..m..] along AXIS (0 = x, 1 = y, 2 = z fastest).
// One thread per pencil: it holds the pencil's N values, and the rows of T are the same for
// every thread (scalar loads), four output points at a time so that four sums are in flight.
// With one thread per output point every thread read its own row of T beside the pencil, along
// z a row per lane: 100 FP32 fields at N = 48 took 929 / 317 / 277 us along z / y / x, now 66 / 30 /
// 43 us (the heavy/light call of 100 nodes 122.4 -> 119.8 ms).
template <typename T, int N, int AXIS>
__global__ __launch_bounds__(256) void resample_pass(const T* __restrict__ in, int64_t in_stride,
                                                     T* __restrict__ out, int64_t out_stride,
                                                     const T* __restrict__ Tm, int64_t nb, int accumulate) {
    const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (t >= nb * (N * N)) return;
    const int64_t b = t / (N * N);
    const int r = int(t - b * (N * N));
    constexpr int step = AXIS == 0 ? N * N : (AXIS == 1 ? N : 1);
    const int base = AXIS == 0 ? r : (AXIS == 1 ? (r / N) * (N * N) + r % N : r * N);
    const T* src = in + b * in_stride + base;
    T* dst = out + b * out_stride + base;
    T v[N];
#pragma unroll
    for (int m = 0; m < N; ++m) v[m] = src[m * step];
#pragma unroll 1
    for (int a = 4 * int(blockIdx.y); a < N; a += 4 * int(gridDim.y)) {
        T acc[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int m = 0; m < N; ++m)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = fma(Tm[(a + j) * N + m], v[m], acc[j]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            T* o = dst + (a + j) * step;
            *o = accumulate ? *o + acc[j] : acc[j];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(256) void copy_fields(const T* __restrict__ in, int64_t in_stride, T* __restrict__ out,
                                                   int64_t out_stride, int64_t n3, int64_t nb, int accumulate) {
    const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
    if (t >= nb * n3) return;
    const int64_t b = t / n3, e = t - b * n3;
    const T v = in[b * in_stride + e];
    T* dst = out + b * out_stride + e;
    *dst = accumulate ? *dst + v : v;
}

template <typename T, int N>
hipError_t resample(const T* in, int64_t in_stride, T* out, int64_t out_stride, const T* Tm, int64_t nb,
                    bool accumulate, T* tmp, hipStream_t st) {
    constexpr int64_t n3 = int64_t(N) * N * N;
    // few pencils: their output points over several threads, to about two wavefronts per SIMD
    const int64_t pencils = nb * N * N;
    const unsigned parts = unsigned(std::max<int64_t>(1, std::min<int64_t>(N / 4, 131072 / pencils)));
    const dim3 grid(unsigned((pencils + 255) / 256), parts), block(256);
    T* t1 = tmp;
    T* t2 = tmp + nb * n3;
    resample_pass<T, N, 2><<<grid, block, 0, st>>>(in, in_stride, t1, n3, Tm, nb, 0);
    resample_pass<T, N, 1><<<grid, block, 0, st>>>(t1, n3, t2, n3, Tm, nb, 0);
    resample_pass<T, N, 0><<<grid, block, 0, st>>>(t2, n3, out, out_stride, Tm, nb, accumulate ? 1 : 0);
    return hipGetLastError();
}

template <typename T>
hipError_t move_impl(const T* in, int64_t in_stride, T* out, int64_t out_stride, const T* Tm, int N, int64_t nb,
                     bool accumulate, T* tmp, hipStream_t st) {
    if (!Tm) {
        const int64_t n3 = int64_t(N) * N * N;
        const dim3 grid(unsigned((nb * n3 + 255) / 256)), block(256);
        copy_fields<T><<<grid, block, 0, st>>>(in, in_stride, out, out_stride, n3, nb, accumulate ? 1 : 0);
        return hipGetLastError();
    }
    switch (N) {
        case 16: return resample<T, 16>(in, in_stride, out, out_stride, Tm, nb, accumulate, tmp, st);
        case 24: return resample<T, 24>(in, in_stride, out, out_stride, Tm, nb, accumulate, tmp, st);
        case 32: return resample<T, 32>(in, in_stride, out, out_stride, Tm, nb, accumulate, tmp, st);
        case 48: return resample<T, 48>(in, in_stride, out, out_stride, Tm, nb, accumulate, tmp, st);
        case 64: return resample<T, 64>(in, in_stride, out, out_stride, Tm, nb, accumulate, tmp, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_move(const dgfs_plan& p, const void* in, int64_t in_stride, void* out, int64_t out_stride,
                       const void* Tm, int64_t nb, bool accumulate, void* tmp, hipStream_t st) {
    if (nb <= 0) return hipSuccess;
    if (p.precision == DGFS_FP64)
        return move_impl<double>(static_cast<const double*>(in), in_stride, static_cast<double*>(out), out_stride,
                                 static_cast<const double*>(Tm), p.N, nb, accumulate, static_cast<double*>(tmp), st);
    return move_impl<float>(static_cast<const float*>(in), in_stride, static_cast<float*>(out), out_stride,
                            static_cast<const float*>(Tm), p.N, nb, accumulate, static_cast<float*>(tmp), st);
}

}  // namespace dgfs
