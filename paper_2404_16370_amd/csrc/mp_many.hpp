// mp_many.hpp -- one launch over several filters: a table of the arguments that
// each would be launched with, and the first workgroup of each.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "mp_internal.hpp"

template <class A>
struct Many {
    const A* tab;
    const int32_t* first;   // ascending, one per filter
    int32_t n;
};

// The arguments of this workgroup's filter, and its place in that filter's
// launch.  The table is read-only while the kernel runs: its words are read
// through the constant address space, so that they land in scalar registers.
template <class A>
__device__ __forceinline__ A many_args(const Many<A>& M, int& block) {
    int lo = 0, hi = M.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (M.first[mid] <= (int)blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    block = (int)blockIdx.x - M.first[lo];
    typedef const __attribute__((address_space(4))) uint32_t ConstWord;
    static_assert(sizeof(A) % 4 == 0, "word copy");
    A a;
    ConstWord* src = (ConstWord*)(M.tab + lo);
    uint32_t* dst = reinterpret_cast<uint32_t*>(&a);
#pragma unroll
    for (int w = 0; w < (int)(sizeof(A) / 4); ++w) dst[w] = src[w];
    return a;
}

// the launch's table in T; `blocks` workgroups of each filter, `grid` in all
template <class A>
Many<A> many_table(ManyTab& T, const std::vector<A>& a, const std::vector<int32_t>& blocks, unsigned& grid) {
    std::vector<int32_t> first;
    int32_t at = 0;
    for (int32_t b : blocks) {
        first.push_back(at);
        at += b;
    }
    grid = (unsigned)at;
    Many<A> M;
    M.tab = static_cast<const A*>(T.put(a.data(), sizeof(A) * a.size()));
    M.first = static_cast<const int32_t*>(T.put(first.data(), sizeof(int32_t) * first.size()));
    M.n = (int32_t)a.size();
    return M;
}
