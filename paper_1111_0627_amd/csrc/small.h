// Small graphs solved whole by one workgroup (small.hip).
#pragma once

#include "kernels.h"
#include "ocm.h"

namespace ocm {

constexpr int kSmallMaxN = 4096;
constexpr int kSmallMaxM = 65535;      // edge positions take 16 bits
constexpr int kSmallFallback = 1;      // status: sums too large, the general path decides
constexpr int kSmallClasses = 4;

struct SmallOpts {
    int validate;          // check the CSR (and its column range)
    int bound;             // apply the weight bound (the batch has done so)
    int fast_path;
    int tie_check;
    int iter_cap;
    long long cycle_cap;   // room for C's edges (single solves)
};

struct SmallOut {
    long long W, L;
    int status;            // ocm_status or kSmallFallback
    int s, iterations, fast, general, connect_rounds, jump_rounds, value_rounds;
    unsigned clen, tight, tie;
};

struct SmallPtrs {
    const int* init;       // warm start's policy, or null
    int* policy;           // outputs of a converged solve, or null
    long long* potential;
    int* cycle;
    SmallOut* out;         // device or mapped host memory
    unsigned* seq;         // set to want once out is written (mapped host memory), or null
    unsigned want;
};

struct SmallBatch {        // the batch's arrays, by graph and by union vertex
    const long long* vptr;
    const long long* eptr;
    long long* W;
    long long* L;
    int* s;
    int* iter;
    int* status;
    int* mode;
    int* pi;
    int* succ;
    long long* V;
    int* hop;
    unsigned char* onC;
};

// Class 0 .. kSmallClasses - 1 of a graph (LDS size), or -1.
int small_class(int64_t n, int64_t m, bool ratio);
void launch_small_one(int n, int m, const int* row_ptr, const int* col, const void* w, int wtype,
                      const int* t, int neg, const SmallOpts& o, const SmallPtrs& p, hipStream_t st);
// wide: some graph's sums may not fit the entries; those are solved again with
// 64-bit values, and left to the loop only where a value leaves +-2^62.
void launch_small_batch(int cls, const int* list, int nlist, const SmallBatch& b, const int* row_ptr,
                        const int* col, const void* w, int wtype, int neg, const SmallOpts& o,
                        bool wide, hipStream_t st);
// A sum over a path of a graph of n vertices with weights up to max|w| is at most
// 2 n^2 max|w|; the entries hold less than 2^51.
inline bool small_sums_may_not_fit(int64_t n, unsigned long long maxw)
{
    return (unsigned __int128)2 * (unsigned)n * (unsigned)n * maxw >= (unsigned __int128)1 << 51;
}

// ocm_min / ocm_max (neg) without the int128 fallback: a value that leaves int64
// gives OCM_E_OVERFLOW, as in the batch.
ocm_status solve_int64(const ocm_graph* g, const ocm_options* o, void* ws, size_t ws_bytes,
                       int32_t* cycle_edges, int64_t cap, ocm_result* out, void* stream, int neg);

}  // namespace ocm
