// The positions and the walk back through the lists of k_sym_list, also built for the host (its
// indices are checked there against the arrays they go into).
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define MSP_LIST_FN __host__ __device__ __forceinline__
#else
#define MSP_LIST_FN inline
#endif

namespace msp {

constexpr int kListEnd = 0xffff;      // 16-bit predecessor of a list's first member

// Position in B of a row's product q from the 48 bits kept of its A entry's
// (the entry's first position less its first product's number, which may be
// below 0).
MSP_LIST_FN long long list_position(uint32_t lo, uint16_t hi, int q) {
    return (long long)(((uint64_t)hi << 32 | lo) + (uint64_t)q & 0xffffffffffffull);
}

// One step back for N products of a lane.  prev[i] is the member of the list
// that product i meets next (below 0: none left; bit i of `live` is then
// clear), col(m) and before(m) a member's column and predecessor.  Bit i of
// `own` is cleared when product i meets its own column.  Every index passed to
// col and before is a member: a product whose walk is over reads member 0.
template <int N, typename Col, typename Before>
MSP_LIST_FN void list_step(const int* c, int* prev, int& live, uint32_t& own, Col col, Before before) {
    int x[N], y[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int m = prev[i] > 0 ? prev[i] : 0;
        x[i] = col(m);
        y[i] = before(m);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const bool on = (live >> i) & 1, same = x[i] == c[i];
        if (on && same) own &= ~(1u << i);
        const bool over = same || y[i] == kListEnd;
        if (on && over) live &= ~(1 << i);
        if (on) prev[i] = over ? -1 : y[i];
    }
}

}  // namespace msp
