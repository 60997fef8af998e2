// Pieces shared by the kernels that hold whole levels or tiles of them in LDS
// in the accumulator format (mg_tail.hip, mg_tile2d.hip): rounding to and
// memory access in a storage format given at run time, so that one kernel
// serves FP32, FP16 and BF16 levels.
#pragma once
#include "mg_device.h"
#include "mg_launch.h"

namespace mg {

// Round an accumulator value to format p (as a value of the accumulator type).
__device__ __forceinline__ float rnd(float v, int p) {
    if (p == P_F16) return widen(Store<f16>::from_acc(v));
    if (p == P_BF16) return widen(Store<bf16>::from_acc(v));
    return v;
}
__device__ __forceinline__ double rnd(double v, int) { return v; }
// Round an FP64 value once into format p, as a value of A.
template <class A> __device__ __forceinline__ A rnd64(double v, int p) {
    if constexpr (std::is_same<A, double>::value) {
        return v;
    } else {
        if (p == P_F16) return widen(Store<f16>::from_f64(v));
        if (p == P_BF16) return widen(Store<bf16>::from_f64(v));
        return (float)v;
    }
}
template <class A> __device__ __forceinline__ A rnd_w(float v, int p) { return rnd(v, p); }
template <class A> __device__ __forceinline__ A rnd_w(double v, int p) { return rnd64<A>(v, p); }

// The same for a run of values (one test of the format).
template <int V> __device__ __forceinline__ void rnd_run(float (&v)[V], int p) {
    if (p == P_F16) {
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] = widen(Store<f16>::from_acc(v[i]));
    } else if (p == P_BF16) {
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] = widen(Store<bf16>::from_acc(v[i]));
    }
}
template <int V> __device__ __forceinline__ void rnd_run(double (&)[V], int) {}

// V values of a level vector in memory, in format p (o: element offset).
template <class A, int V> __device__ __forceinline__ void mem_load(const void *m, size_t o, int p, A (&v)[V]) {
    if constexpr (std::is_same<A, double>::value) {
        if (p == P_F64) {
            load_row<double, V>(static_cast<const double *>(m) + o, v);
            return;
        }
    }
    if (p == P_F16) load_row<f16, V>(static_cast<const f16 *>(m) + o, v);
    else if (p == P_BF16) load_row<bf16, V>(static_cast<const bf16 *>(m) + o, v);
    else load_row<float, V>(static_cast<const float *>(m) + o, v);
}
template <class T, int V, class A> __device__ __forceinline__ void mem_store_t(void *m, size_t o, const A (&v)[V]) {
    T t[V];
#pragma unroll
    for (int i = 0; i < V; ++i) t[i] = store_as<T>(v[i]);
    store_row<T, V>(static_cast<T *>(m) + o, t);
}
// (values are rounded to p on the way: a no-op for values of the format)
template <class A, int V> __device__ __forceinline__ void mem_store(void *m, size_t o, int p, const A (&v)[V]) {
    if (p == P_F64) mem_store_t<double, V>(m, o, v);
    else if (p == P_F16) mem_store_t<f16, V>(m, o, v);
    else if (p == P_BF16) mem_store_t<bf16, V>(m, o, v);
    else mem_store_t<float, V>(m, o, v);
}

}  // namespace mg
