// First-order dual numbers: a value and its derivatives along K directions.
// The collision's device functions are templates on their real type and use
// only + - * / and constants, so evaluating them on Dual gives directional
// derivatives of the post-collision populations (forward-mode
// differentiation) without a second, hand-differentiated copy of the scheme.
#pragma once

#include <hip/hip_runtime.h>

namespace lbm {

template <int K> struct Dual {
    float v, d[K];
    Dual() = default;
    __host__ __device__ constexpr Dual(double c) : v((float)c), d{} {}
};

template <int K> __host__ __device__ inline Dual<K> operator+(Dual<K> a, Dual<K> b)
{
    Dual<K> r;
    r.v = a.v + b.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] + b.d[k];
    return r;
}
template <int K> __host__ __device__ inline Dual<K> operator-(Dual<K> a, Dual<K> b)
{
    Dual<K> r;
    r.v = a.v - b.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] - b.d[k];
    return r;
}
template <int K> __host__ __device__ inline Dual<K> operator-(Dual<K> a)
{
    Dual<K> r;
    r.v = -a.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = -a.d[k];
    return r;
}
template <int K> __host__ __device__ inline Dual<K> operator*(Dual<K> a, Dual<K> b)
{
    Dual<K> r;
    r.v = a.v * b.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = a.d[k] * b.v + a.v * b.d[k];
    return r;
}
template <int K> __host__ __device__ inline Dual<K> operator/(Dual<K> a, Dual<K> b)
{
    Dual<K> r;
    r.v = a.v / b.v;
#pragma unroll
    for (int k = 0; k < K; ++k) r.d[k] = (a.d[k] - r.v * b.d[k]) / b.v;
    return r;
}
template <int K> __host__ __device__ inline Dual<K>& operator+=(Dual<K>& a, Dual<K> b) { return a = a + b; }
template <int K> __host__ __device__ inline Dual<K>& operator-=(Dual<K>& a, Dual<K> b) { return a = a - b; }

} // namespace lbm
