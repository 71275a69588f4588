// Global memory through a uniform base pointer and a 32-bit element index.
//
// A pointer that a kernel loads from memory (the plan's argument structure, the
// control block) is a generic pointer to the compiler: its accesses become flat
// instructions, which take a 64-bit address per lane and whose waits also wait
// for every LDS operation in flight.  GP states that the memory is global and
// the base uniform, so that accesses are global instructions with a scalar base
// and a 32-bit offset (arrays up to 4 GB; the largest grid and intermediate hold
// 134 MB).  KRef reads the plan's arguments and its control block through the
// scalar cache, as one set of loads in flight.  Together (every kernel of a march
// used to follow six to nine dependent flat loads before its first work): 512^2
// march 41.9 -> 38.1 ms, 2048^2 656 -> 572, 24 plans 195 -> 170.
//
// What KRef reads is constant to the compiler, and the scalar cache does not see
// the vector stores of the kernel that reads it.  So a word read through KRef must
// not be written by the same kernel until every use of the value is complete, or
// the value is pinned in registers (an asm volatile with it as an operand).  The
// control block's readers that also write it keep to that: the line-row kernel reads
// the stopping values of the iteration before the one whose it raises, the kernels
// that end a step have consumed or pinned what they read before they rewrite it.
#pragma once

#include <hip/hip_runtime.h>

namespace lpide {

#define LPIDE_GLOBAL __attribute__((address_space(1)))
#define LPIDE_CONST __attribute__((address_space(4)))

template <typename T>
struct GWord { using type = T; };
template <>
struct GWord<double2> { typedef double type __attribute__((ext_vector_type(2))); };
template <>
struct GWord<float2> { typedef float type __attribute__((ext_vector_type(2))); };

template <typename T>
struct GP {
    using W = typename GWord<T>::type;
    const LPIDE_GLOBAL char* p;

    __device__ __forceinline__ explicit GP(const T* q) : p((const LPIDE_GLOBAL char*)(const char*)q) {}
    // the array from element `first` on (first uniform)
    __device__ __forceinline__ GP(GP a, size_t first) : p(a.p + first * sizeof(T)) {}

    __device__ __forceinline__ T operator[](unsigned i) const {
        const W v = *(const LPIDE_GLOBAL W*)(p + (unsigned)(i * (unsigned)sizeof(T)));
        if constexpr (sizeof(W) == sizeof(T) && !__is_same(W, T)) {
            T t;
            t.x = v.x;
            t.y = v.y;
            return t;
        } else {
            return v;
        }
    }
    __device__ __forceinline__ void put(unsigned i, T t) const {
        LPIDE_GLOBAL W* q = (LPIDE_GLOBAL W*)(p + (unsigned)(i * (unsigned)sizeof(T)));
        if constexpr (!__is_same(W, T)) {
            W v;
            v.x = t.x;
            v.y = t.y;
            *q = v;
        } else {
            *q = t;
        }
    }
};

template <typename T>
using KRef = const LPIDE_CONST T&;

template <typename T>
__device__ __forceinline__ KRef<T> kref(const T* p) { return *(const LPIDE_CONST T*)p; }

}  // namespace lpide
