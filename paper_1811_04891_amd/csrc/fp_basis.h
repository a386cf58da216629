// Device-side Lagrange basis on GLL nodes for one lane, and the address spaces that
// element data is read through: wave-uniform pointers to data that is not written
// while a kernel runs compile to scalar loads (a multiply-add then takes the node
// value as a scalar operand), staged elements to LDS reads.
#pragma once

#include "fp_internal.h"

namespace fp {

// h_i(r) = wb_i prod_{m != i} (r - z_m) and h_i'(r), by prefix and suffix
// products (O(n1) per evaluation, no division, exact zeros at other nodes).
// The basis table (z[16] then wb[16]) is read from device memory through the
// scalar cache each time instead of being held in scalar registers.
template <class T>
struct BasisPtr {
    const __attribute__((address_space(4))) T *p;
    __device__ __forceinline__ T z(int i) const { return p[i]; }
    __device__ __forceinline__ T wb(int i) const { return p[kMaxN1 + i]; }
};

template <int N1, class T>
__device__ __forceinline__ void lagrange_d(BasisPtr<T> B, T r, T (&h)[N1], T (&d)[N1])
{
    asm volatile("" : "+s"(B.p));
    T t[N1], pl[N1], dpl[N1];
#pragma unroll
    for (int i = 0; i < N1; ++i) t[i] = r - B.z(i);
    pl[0] = T(1);
    dpl[0] = T(0);
#pragma unroll
    for (int i = 1; i < N1; ++i) {
        dpl[i] = dpl[i - 1] * t[i - 1] + pl[i - 1];
        pl[i] = pl[i - 1] * t[i - 1];
    }
    T pr = T(1), dpr = T(0);
#pragma unroll
    for (int i = N1 - 1; i >= 0; --i) {
        h[i] = B.wb(i) * (pl[i] * pr);
        d[i] = B.wb(i) * (dpl[i] * pr + pl[i] * dpr);
        dpr = dpr * t[i] + pr;
        pr = pr * t[i];
    }
}

template <int N1, class T>
__device__ __forceinline__ void lagrange(BasisPtr<T> B, T r, T (&h)[N1])
{
    asm volatile("" : "+s"(B.p));
    T t[N1], pl[N1];
#pragma unroll
    for (int i = 0; i < N1; ++i) t[i] = r - B.z(i);
    pl[0] = T(1);
#pragma unroll
    for (int i = 1; i < N1; ++i) pl[i] = pl[i - 1] * t[i - 1];
    T pr = T(1);
#pragma unroll
    for (int i = N1 - 1; i >= 0; --i) {
        h[i] = B.wb(i) * (pl[i] * pr);
        pr = pr * t[i];
    }
}

// Keep a wave-uniform pointer in scalar registers and opaque to loop-
// invariant code motion: without this the compiler hoists all 3V element
// loads out of the Newton loop into vector registers and spills them.
#define FP_PIN_SGPR(p) asm volatile("" : "+s"(p))
#define FP_KEEP(v) asm volatile("" ::"v"(v))

// Element data is read through the constant address space: it is not written
// while a kernel runs, and uniform loads from it are always scalar loads.
template <class T>
using cptr = const __attribute__((address_space(4))) T *;

template <class T>
__device__ __forceinline__ cptr<T> as_const(const T *p)
{
    return (cptr<T>)p;
}

// Element data staged in LDS, read through the LDS address space.
template <class T>
using lptr = const __attribute__((address_space(3))) T *;

}  // namespace fp
