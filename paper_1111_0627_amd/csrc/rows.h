// Walks over a row's edges.  Positions go up to 2^31 - 1 (m's limit), so a step
// past the end of the last rows leaves int: strided walks count in unsigned.
#pragma once

#ifdef __HIPCC__
#define OCM_HD __host__ __device__ __forceinline__
#else
#define OCM_HD inline
#endif

namespace ocm {

// Edges [first, last) of a row, U at a time with their loads in flight together:
// u = head(position), y = value(u), then f(position, u, y) in order until it
// returns true.  A head is never negative.
template <int U, typename H, typename V, typename F>
OCM_HD void for_row(int first, int last, H&& head, V&& value, F&& f)
{
    const unsigned end = (unsigned)last;
    for (unsigned e = (unsigned)first; e < end; e += U) {
        int u[U], y[U];
#pragma unroll
        for (int j = 0; j < U; ++j) u[j] = e + j < end ? head(e + j) : -1;
#pragma unroll
        for (int j = 0; j < U; ++j) y[j] = u[j] >= 0 ? value(u[j]) : 0;
#pragma unroll
        for (int j = 0; j < U; ++j)
            if (u[j] >= 0 && f(e + j, u[j], y[j])) return;
    }
}

}  // namespace ocm
