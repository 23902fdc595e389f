// Accesses of the streaming kernels to rows of a population plane: a uniform
// row address and a 32-bit offset per lane.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sllbm {

// x modulo n, in 0 .. n - 1
__device__ __forceinline__ int wrapi(int x, int n)
{
    const int r = x % n;
    return r < 0 ? r + n : r;
}

// Byte offset of a node in an x-y plane: 32 bits suffice (two states, of 90 planes or
// in two dimensions 38, whose x-y plane had 4 GB would not fit the card), so that an
// access is a uniform row address plus one register per lane.
template <typename S>
__device__ __forceinline__ uint32_t plane_offset(int node)
{
    return static_cast<uint32_t>(node) * static_cast<uint32_t>(sizeof(S));
}
// A row of a plane as the compiler must see it, a uniform address that it does
// not know: otherwise it keeps plane address + offset, 64 bits per lane and
// access, across the loop.
template <typename S>
using GlobalRow = __attribute__((address_space(1))) S *;
template <typename S>
__device__ __forceinline__ GlobalRow<S> plane_row(S *base, int64_t node)
{
    GlobalRow<S> r = (GlobalRow<S>)(base + node);
    asm volatile("" : "+s"(r));
    return r;
}
template <typename S>
__device__ __forceinline__ S load_at(GlobalRow<S> row, uint32_t off)
{
    return *(GlobalRow<S>)((__attribute__((address_space(1))) char *)row + off);
}
template <bool NTH, typename S>
__device__ __forceinline__ void store_at(GlobalRow<S> row, uint32_t off, S v)
{
    GlobalRow<S> p = (GlobalRow<S>)((__attribute__((address_space(1))) char *)row + off);
    if constexpr (NTH) __builtin_nontemporal_store(v, p);
    else *p = v;
}

}  // namespace sllbm
