// Cycles of a functional graph by records (kernels.hip: one policy, batch.hip:
// the policies of a batch).
#pragma once

#include "device_util.h"

namespace ocm {

// Jump rounds touch every vertex some log2(depth) + 3 times, each time a gather
// of 8 bytes and the barrier of a launch (2^22 vertices: 12 to 15 rounds, 560 to
// 1390 us; 20,000: 13 launches).  Here vertices are ordered by a multiplicative
// hash of their index, and each finds
//   N: the first vertex on its path that is lower than itself, by jumping along
//      the entries of the vertices in between, in place (a vertex below its
//      whole path, hence on no cycle, ends at the cycle's lowest);
//   T: the lowest vertex its path reaches, along the N's;
// a vertex with N = itself is the lowest of its cycle.  Expected 2 to 4 gathers
// of 4 bytes per vertex and step whatever the numbering, in two or three
// launches: as in the value chase an entry seen late is still a vertex of the
// path with nothing lower before it, so every order of the updates ends in the
// same N and T.  2^22 vertices: 290 to 600 us with the marks, bound by the
// gathers; 20,000: 42 us.
// The jump rounds take over if a path takes more than kLowSteps steps or a cycle
// has more than kLowQueue vertices.
constexpr int kLowSteps = 256;
constexpr int kLowFirst = 8;   // steps of a large graph's first pass
constexpr int kLowQueue = 8192;

__device__ __forceinline__ unsigned low_key(unsigned v) { return v * 0x9E3779B1u; }

// N[v], up to `steps` steps; *open: not reached yet.
template <int LD, int ST>
__device__ __forceinline__ unsigned low_next(unsigned* N, unsigned v, int steps, bool* open)
{
    const unsigned own = low_key(v);
    unsigned j = __hip_atomic_load(&N[v], __ATOMIC_RELAXED, LD);
    unsigned low = j;   // the lowest vertex passed since the last restart
    bool on = low_key(j) > own;
    for (int k = 1; k <= steps && on; ++k) {
        const unsigned r = __hip_atomic_load(&N[j], __ATOMIC_RELAXED, LD);
        // at the cycle's lowest, or back at the lowest passed, which is that
        // (unless it is off the cycle: hence the restarts): a vertex off the
        // cycle, below its whole path
        on = r != j && r != low && low_key(r) > own;
        if (low_key(r) < low_key(low) || (k & 31) == 0) low = r;
        j = r;
        __hip_atomic_store(&N[v], j, __ATOMIC_RELAXED, ST);
    }
    *open = on;
    return j;
}

// T[v] from the N's in T, in place; true if v is the lowest of a cycle.
template <int LD, int ST>
__device__ __forceinline__ bool low_root(unsigned* T, unsigned v, bool* open)
{
    unsigned j = __hip_atomic_load(&T[v], __ATOMIC_RELAXED, LD);
    const bool root = j == v;
    bool on = !root;
    for (int k = 0; k < kLowSteps && on; ++k) {
        const unsigned r = __hip_atomic_load(&T[j], __ATOMIC_RELAXED, LD);
        on = r != j;
        if (on) {
            j = r;
            __hip_atomic_store(&T[v], j, __ATOMIC_RELAXED, ST);
        }
    }
    *open = on;
    return root;
}

// Marks the cycles from their lowest vertices and adds up their edges: dependent
// reads, so the loads of a step are issued together and the sums a step behind.
// A thread walks a cycle of up to kLowWalk vertices; longer ones are left to the
// workgroup: the vertices between v and N[v] are the chain succ(v), N(succ(v)),
// ... up to N[v], each with those between itself and its own N, which spreads a
// cycle of l random vertices over the threads in some 2 ln l levels (1000
// vertices of 2^20: 46 us, not 600).  With a workgroup per cycle the walk is given up
// after kLowWalkFew steps.
constexpr int kLowWalk = 48, kLowWalkFew = 8;
constexpr int kLowLevel = 2048;   // vertices of two consecutive levels

// All threads of every workgroup call it.  root(i) is the lowest vertex of cycle
// i < nroots; close(i, r, smallest index, W, T, length) is called once per cycle,
// or fail(i) (by every thread of a workgroup) if it is too long.
template <typename WT, typename Root, typename Close, typename Fail>
__device__ __forceinline__ void low_mark(unsigned nroots, const int* __restrict__ succ,
                                         const unsigned* __restrict__ N, const int* __restrict__ pi,
                                         const WT* __restrict__ w, int neg,
                                         const int* __restrict__ tm, unsigned char* __restrict__ onc,
                                         Root&& root, Close&& close, Fail&& fail)
{
    __shared__ int all[kLowQueue];                            // the cycle's vertices
    __shared__ int qn[kLowLevel], qs[kLowLevel];   // their N and succ, by slot mod kLowLevel
    __shared__ int longs[kWG];
    __shared__ unsigned nlong, tail, over;
    __shared__ int low;
    const int t = threadIdx.x;
    const unsigned walk = nroots <= gridDim.x ? kLowWalkFew : kLowWalk;
    for (unsigned b = 0; b * gridDim.x + blockIdx.x < nroots; b += kWG) {
        if (t == 0) nlong = 0;
        __syncthreads();
        const unsigned i = (b + t) * gridDim.x + blockIdx.x;   // neighbours go to different workgroups
        if (i < nroots) {
            const int r = root(i);
            int u = r, mn = r, e = -1;
            unsigned len = 0;
            long long W = 0, T = 0;
            do {
                const int next = succ[u], e1 = pi[u];
                const long long we = e >= 0 ? wval(w, e, neg) : 0, te = tm && e >= 0 ? tm[e] : 0;
                onc[u] = 1;
                mn = u < mn ? u : mn;
                W += we;
                T += te;
                e = e1;
                u = next;
                ++len;
            } while (u != r && len < walk);
            if (u == r) close(i, r, mn, W + wval(w, e, neg), tm ? T + tm[e] : 0, len);
            else longs[atomicAdd(&nlong, 1u)] = (int)i;
        }
        __syncthreads();
        const unsigned nl = nlong;
        for (unsigned x = 0; x < nl; ++x) {
            const unsigned li = (unsigned)longs[x];
            const int r = root(li);
            __syncthreads();   // every thread has read what close() may overwrite
            if (t == 0) {
                all[0] = qn[0] = low = r;
                qs[0] = succ[r];
                onc[r] = 1;
                tail = 1;
                over = 0;
            }
            __syncthreads();
            unsigned lo = 0, hi = 1;
            bool stop = false;
            while (lo < hi && !stop) {
                for (unsigned y = lo + t; y < hi; y += kWG) {
                    const int end = qn[y % kLowLevel];
                    int u = qs[y % kLowLevel];
                    while (u != end) {
                        const int n = (int)N[u], s = succ[u];
                        onc[u] = 1;
                        const unsigned slot = atomicAdd(&tail, 1u);
                        if (slot >= (unsigned)kLowQueue || slot - lo >= (unsigned)kLowLevel) {
                            over = 1;
                            break;
                        }
                        all[slot] = u;
                        qn[slot % kLowLevel] = n;
                        qs[slot % kLowLevel] = s;
                        u = n;
                    }
                }
                __syncthreads();
                lo = hi;
                hi = tail;
                stop = over != 0;
                __syncthreads();
            }
            if (stop) {   // uniform
                fail(li);
                continue;
            }
            int mn = r;
            long long W = 0, T = 0;
            for (unsigned y = t; y < hi; y += kWG) {
                const int u = all[y], e = pi[u];
                mn = u < mn ? u : mn;
                W += wval(w, e, neg);
                if (tm) T += tm[e];
            }
            atomicMin(&low, mn);
            unsigned long long sums[2] = {(unsigned long long)W, (unsigned long long)T};
            block_sums_u64(sums);   // two's complement sums
            if (t == 0) close(li, r, low, (long long)sums[0], (long long)sums[1], hi);
        }
        __syncthreads();
    }
}

}  // namespace ocm
