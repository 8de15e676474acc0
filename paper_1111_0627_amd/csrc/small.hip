// Small graphs solved whole by one workgroup, state and edges in LDS: single
// solves (one launch, validation and tie test included) and the small class
// of the batched form.
#include "small.h"

#include "device_util.h"

namespace ocm {
namespace sm {

// ---------------------------------------------------------------------------
// One workgroup per graph.  Rules and phases are the solver's (R1-R10, fast
// path included): R1's first sweep; cycles by pointer jumping; per-cycle sums
// and the (W/L, rep) minimum; breadth-first rebuild rounds; values by the
// in-place chase; the improvement sweep, a thread per vertex over its row.
//   * Bound: barriers and LDS latency, 8 to 10 us an iteration at n = 1000.
//     A launch per phase costs about 5 us each on such graphs, and reading the
//     CSR from L2 in every sweep 6 us, so everything stays on the CU: vertex
//     numbers and edge positions in 16 bits, weights (and times) in 32.
//     Weights beyond 32 bits, and edges beyond the class, are read from memory.
//   * One array serves as chase entries and as values: a finished entry is
//     (value << kBits) | s.  A sweep reads the values, and after a barrier its
//     threads write the next entries.
//   * Classes (vertices, edges, threads in a batch; LDS): 512, 4096, 256 (36
//     KB, 4 per CU); 1024, 8192, 512 (72 KB, 2 per CU); 2048, 16384, 1024 (143
//     KB); 4096, edges in memory, 1024 (94 KB).  A single solve, alone on its
//     CU, takes 128 to 512 threads up to 512 vertices and 1024 beyond.
//   * A thread walks its vertex's row, a wave the rows of more than kLongEdges
//     edges, the whole workgroup those of more than kWideEdges: see below.
// Sums that do not fit an entry (kBits for the vertex, 51 and a sign for the
// sum) end the solve with kSmallFallback: the general path takes the graph, in a
// batch first a second launch with wider entries.
// ---------------------------------------------------------------------------
constexpr int kBits = 12;
constexpr unsigned long long kMask = (1ull << kBits) - 1;
static_assert(kSmallMaxN <= (1 << kBits), "vertex numbers fit the entry");

// Rows that one thread would keep the others waiting for, four edges at a time:
// long ones take a wave each, wide ones all waves.  Whole solves, by a thread / so
// (launches per phase: the general path), us: 4000 vertices with a hub to all of
// them 13500 / 765 (3016), 700 with a row of 30,000 edges 42200 / 209 (1728), 4000
// with a row of 50,000 99300 / 630 (2651).  The lines: 500 rows of 100 to 129
// edges 945 with long rows from 65 on, 1450 from 129 on; 1000 rows of 50 to 65
// 1136 so, 1440 from 33 on.  The hub of 4000 by all waves 769, by one 931, the row
// of 50,000 630 and 2349; ten rows of 1000 by a wave each 350, by all 615.
constexpr int kLongEdges = 64, kWideEdges = 2048;
constexpr int kRowSteps = 4;   // edges a lane has in flight on them
constexpr int kWideRows = kSmallMaxM / (kWideEdges + 1);

// a before b in the order (W / L, rep); r < 0: none.
__device__ __forceinline__ bool cand_less(long long aw, long long al, int ar, long long bw,
                                          long long bl, int br)
{
    if (br < 0) return ar >= 0;
    if (ar < 0) return false;
    const __int128 x = (__int128)aw * bl, y = (__int128)bw * al;
    if (x != y) return x < y;
    return ar < br;
}

template <int N, int M, bool RATIO>
struct Lds {
    unsigned long long E[N];             // chase entries / values; rebuild: per-cycle weights
    long long T[RATIO ? N : 1];          // per-cycle times
    unsigned JM[N];                      // cycles: vertex reached | smallest on the way << 16;
                                         //   then per-cycle lengths
    int w[M > 0 ? M : 1];
    int t[RATIO && M > 0 ? M : 1];
    unsigned short c[M > 0 ? M : 1];
    unsigned short rb[N + 1];            // first edge of each row, from the graph's first edge
    unsigned short pi[N];                // policy edge, likewise
    unsigned short succ[N];
    unsigned short rep[N];               // smallest vertex of the reached cycle
    unsigned short layer[N];             // rebuild round (0xffff unattached); heads; alive
    unsigned char onc[N];                // 1 on a policy cycle, 3 on C
    unsigned short longs[(M > 0 ? M : kSmallMaxM) / (kLongEdges + 1) + 1];   // long rows' vertices
    unsigned short wides[kWideRows + 1];                                     // wide rows' vertices
    unsigned nlong, nwide;
    long long wk[1024 / 64];             // a wide row's best by wave: key, edge, head
    int wp[1024 / 64], wh[1024 / 64];
    unsigned acc[2][4];                  // sweep: changed, broken, tight, certain (by parity)
    unsigned got[3];                     // rebuild rounds: vertices attached
    unsigned stall, over, cnt, flag;
    unsigned long long maxw;
    unsigned maxt, err, cap;
    long long selW, selL;
    int selS;
};

// The graph as the kernel reads it: edges [e0, e0 + m), vertices from v0.
template <typename WT, int N, int M, bool RATIO, bool WIDE>
struct View {
    Lds<N, M, RATIO>& S;
    const int* col;
    const WT* w;
    const int* t;
    int v0, e0;
    bool neg, lds;
    __device__ __forceinline__ long long weight(int e) const
    {
        if (M > 0 && lds) return neg ? -(long long)S.w[e] : (long long)S.w[e];
        return wval(w, e0 + e, neg);
    }
    __device__ __forceinline__ long long time(int e) const
    {
        if (!RATIO) return 1;
        return M > 0 && lds ? S.t[e] : t[e0 + e];
    }
    __device__ __forceinline__ int head(int e) const
    {
        return M > 0 && lds ? (int)S.c[e] : col[e0 + e] - v0;
    }
    // the value of a finished entry
    __device__ __forceinline__ long long value(int v) const
    {
        return WIDE ? (long long)S.E[v] : (long long)S.E[v] >> kBits;
    }
    // v's entry for the edge e to h; false if its sum does not fit
    __device__ __forceinline__ bool entry(int v, int s, long long L, long long W, int e, int h) const
    {
        if (WIDE) S.JM[v] = v == s ? (unsigned)s : (unsigned)h;
        unsigned long long x = WIDE ? 0ull : (unsigned long long)(unsigned)s;
        bool fits = true;
        if (v != s) {
            const long long d = L * weight(e) - (RATIO ? W * time(e) : W);
            if (WIDE) x = (unsigned long long)d;
            else fits = chase_pack(d, (unsigned)h, kBits, &x);
        }
        S.E[v] = x;
        return fits;
    }
};

// The best edge of a row over a wave's lanes, ties to the lowest position (every
// lane gets it; no edge: arg = INT32_MAX), from edge first on in steps of `step`
// runs of 64 lanes with U edges each.  FIRST: by weight alone.  Else by the head's value too,
// and the tight edges other than cur are counted as in the sweep.
template <bool FIRST, typename WT, int N, int M, bool RATIO, bool WIDE>
__device__ __forceinline__ void wave_row(const View<WT, N, M, RATIO, WIDE>& g, long long L, long long W,
                                         int v, int first, int end, int step, int cur, long long own,
                                         bool onC, long long& best, int& arg, int& bh,
                                         unsigned& tight, unsigned& certain)
{
    constexpr int U = kRowSteps;
    best = INT64_MAX;
    arg = INT32_MAX;
    bh = 0;
    for (int eb = first + (threadIdx.x & 63); eb < end; eb += 64 * U * step) {
        int x[U];
        long long key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = eb + 64 * u < end ? eb + 64 * u : end - 1;
            x[u] = g.head(e);
            key[u] = FIRST ? g.weight(e) : L * g.weight(e) - (RATIO ? W * g.time(e) : W);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (!FIRST) key[u] += g.value(x[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = eb + 64 * u;
            if (e >= end) break;
            if (key[u] < best) {
                best = key[u];
                arg = e;
                bh = x[u];
            }
            if (!FIRST && key[u] == own && e != cur) {
                ++tight;
                certain += x[u] == v || onC;
            }
        }
    }
    wave_argmin<long long, true>(best, arg, bh);
}

// done(v, best, arg, head) for every listed row, by every lane of the wave that
// scanned it (of the first one for the wide rows).  All threads call it.
template <bool FIRST, typename WT, int N, int M, bool RATIO, bool WIDE, typename F>
__device__ __forceinline__ void listed_rows(const View<WT, N, M, RATIO, WIDE>& g, int nl, int nw,
                                            long long L, long long W, unsigned& tight,
                                            unsigned& certain, F&& done)
{
    Lds<N, M, RATIO>& S = g.S;
    const int wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    for (int i = wave; i < nl; i += waves) {
        const int v = S.longs[i];
        long long best;
        int arg, bh;
        wave_row<FIRST>(g, L, W, v, S.rb[v], S.rb[v + 1], 1, S.pi[v], g.value(v),
                        S.onc[v] == 3, best, arg, bh, tight, certain);
        done(v, best, arg, bh);
    }
    for (int i = 0; i < nw; ++i) {
        const int v = S.wides[i];
        long long best;
        int arg, bh;
        wave_row<FIRST>(g, L, W, v, S.rb[v] + 64 * kRowSteps * wave, S.rb[v + 1], waves, S.pi[v],
                        g.value(v), S.onc[v] == 3, best, arg, bh, tight, certain);
        if ((threadIdx.x & 63) == 0) {
            S.wk[wave] = best;
            S.wp[wave] = arg;
            S.wh[wave] = bh;
        }
        __syncthreads();
        if (wave == 0) {
            const int l = threadIdx.x < (unsigned)waves ? threadIdx.x : 0;
            best = S.wk[l];
            arg = S.wp[l];
            bh = S.wh[l];
            wave_argmin<long long, true>(best, arg, bh);
            done(v, best, arg, bh);
        }
        __syncthreads();   // the next row reuses wk
    }
}

// In-place chase of every vertex to s (see k_chase): at most n steps, each at
// least one policy edge, so a vertex that has not arrived by then never does.
// A thread's vertices step together, so that their reads overlap.
template <int N>
constexpr int kVpt = N == 4096 ? 4 : 2;   // vertices per thread at most

// Values of 64 bits with the vertex reached beside them (JM): a pair cannot be
// read whole while its owner writes it, so the vertices jump in rounds.
template <int N, int M, bool RATIO>
__device__ __forceinline__ void jump(Lds<N, M, RATIO>& S, int n, unsigned s)
{
    constexpr int VPT = kVpt<N>;
    const int t = threadIdx.x, B = blockDim.x;
    bool bad = false;
    for (int span = 1;; span <<= 1) {
        long long d[VPT];
        unsigned j[VPT];
        bool open = false;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            const int v = t + i * B;
            j[i] = v < n ? S.JM[v] : s;
            if (j[i] == s) continue;
            open = true;
            bad |= __builtin_add_overflow((long long)S.E[v], (long long)S.E[j[i]], &d[i]);
            j[i] = S.JM[j[i]] | 0x10000u;
        }
        if (!__syncthreads_or(open)) break;
        if (span >= 2 * n) {   // uniform: a path of n edges has met s or never does
            S.stall = 1;
            break;
        }
#pragma unroll
        for (int i = 0; i < VPT; ++i)
            if (j[i] & 0x10000u) {
                S.E[t + i * B] = (unsigned long long)d[i];
                S.JM[t + i * B] = j[i] & 0xffffu;
            }
        __syncthreads();
    }
    for (int v = t; v < n; v += B) bad |= (long long)S.E[v] > kValLimit || (long long)S.E[v] < -kValLimit;
    if (bad) S.over = 1;
}

template <bool WIDE, int N, int M, bool RATIO>
__device__ __forceinline__ void chase(Lds<N, M, RATIO>& S, int n, unsigned s)
{
    if (WIDE) {
        jump(S, n, s);
        return;
    }
    constexpr int WGS = __HIP_MEMORY_SCOPE_WORKGROUP, VPT = kVpt<N>;
    const int t = threadIdx.x, B = blockDim.x;
    unsigned long long e[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) e[i] = t + i * B < n ? S.E[t + i * B] : (unsigned long long)s;
    bool fits = true;
    for (int k = 1;; ++k) {
        unsigned long long r[VPT];
        bool open = false;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            r[i] = chase_load<WGS>(&S.E[e[i] & kMask]);   // a finished vertex rereads s
            open |= (e[i] & kMask) != s;
        }
        if (!open) break;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            if ((e[i] & kMask) == s) continue;
            const unsigned h = (unsigned)(r[i] & kMask);
            fits &= chase_pack(((long long)e[i] >> kBits) + ((long long)r[i] >> kBits), h, kBits,
                               &e[i]);
            chase_store<WGS>(&S.E[t + i * B], e[i]);
            if (h == (unsigned)(t + i * B)) S.stall = 1;
        }
        if (k > n) S.stall = 1;
        if ((k & 3) == 0 && __hip_atomic_load(&S.stall, __ATOMIC_RELAXED, WGS)) break;
    }
    if (!fits) S.over = 1;
}

struct Run {
    int status, iter, fast, general, connect, jumps, values;
    int s;
    long long W, L;
    unsigned clen, tight, certain;
    bool tie;
};

// From the first sweep, or the warm start's policy, to the end.  LISTED: there
// are nl long and nw wide rows.  (Without, their tests alone cost 2 to 8 %.)
template <bool LISTED, typename WT, int N, int M, bool RATIO, bool WIDE>
__device__ __forceinline__ void iterate(const View<WT, N, M, RATIO, WIDE>& g, int nl, int nw, int n, int e0,
                                        const SmallOpts& o, const int* __restrict__ init, Run& R)
{
    Lds<N, M, RATIO>& S = g.S;
    const int t = threadIdx.x, B = blockDim.x;
    constexpr int VPT = kVpt<N>;
    if (init) {
        bool bad = false;
        for (int v = t; v < n; v += B) {
            const int p = init[v] - e0;
            const bool in = p >= (int)S.rb[v] && p < (int)S.rb[v + 1];
            bad |= !in;
            S.pi[v] = (unsigned short)(in ? p : S.rb[v]);
            S.succ[v] = (unsigned short)g.head(S.pi[v]);
        }
        if (__syncthreads_or(bad)) {
            R.status = OCM_E_INVALID_ARG;
            return;
        }
    } else {
        // R1: the lowest-position minimum-weight out-edge
        unsigned none = 0;
        if (LISTED) listed_rows<true>(g, nl, nw, 1, 0, none, none, [&](int v, long long, int arg, int bh) {
            if ((t & 63) != 0) return;
            S.pi[v] = (unsigned short)arg;
            S.succ[v] = (unsigned short)bh;
        });
        for (int v = t; v < n; v += B) {
            int arg = S.rb[v];
            if (LISTED && (int)S.rb[v + 1] - arg > kLongEdges) continue;
            long long best = g.weight(arg);
            for (int e = arg + 1; e < (int)S.rb[v + 1]; ++e) {
                const long long x = g.weight(e);
                if (x < best) {
                    best = x;
                    arg = e;
                }
            }
            S.pi[v] = (unsigned short)arg;
            S.succ[v] = (unsigned short)g.head(arg);
        }
        R.iter = 1;
        if (R.iter >= o.iter_cap) {
            R.status = OCM_E_NOT_CONVERGED;
            return;
        }
    }
    int s = 0, par = 0;
    long long W = 0, L = 1;
    bool general = true;
    __syncthreads();
    for (;;) {
        if (general) {
            ++R.general;
            // cycles: after K rounds (2^K >= n) the vertex reached lies on
            // v's cycle and its own way holds that cycle's smallest vertex;
            // the image is the set of cycle vertices
            unsigned* Pa = S.JM;
            unsigned* Pb = (unsigned*)S.E;
            for (int v = t; v < n; v += B) {
                Pa[v] = (unsigned)S.succ[v] | ((unsigned)v << 16);
                S.onc[v] = 0;
            }
            __syncthreads();
            for (int span = 1; span < n; span <<= 1) {
                for (int v = t; v < n; v += B) {
                    const unsigned a = Pa[v], b = Pa[a & 0xffffu];
                    const unsigned ma = a >> 16, mb = b >> 16;
                    Pb[v] = (b & 0xffffu) | ((ma < mb ? ma : mb) << 16);
                }
                __syncthreads();
                unsigned* x = Pa;
                Pa = Pb;
                Pb = x;
                ++R.jumps;
            }
            for (int v = t; v < n; v += B) {
                const unsigned x = Pa[v] & 0xffffu;
                S.onc[x] = 1;
                S.rep[v] = (unsigned short)(Pa[x] >> 16);
            }
            if (t == 0) S.cnt = 0;
            __syncthreads();
            // per-cycle sums keyed by the smallest vertex, cycle heads listed
            for (int v = t; v < n; v += B)
                if (S.rep[v] == v) {   // only a cycle's smallest vertex
                    S.E[v] = 0;
                    S.JM[v] = 0;
                    if (RATIO) S.T[v] = 0;
                    S.layer[atomicAdd(&S.cnt, 1u)] = (unsigned short)v;
                }
            __syncthreads();
            for (int v = t; v < n; v += B)
                if (S.onc[v]) {
                    const int r = S.rep[v];
                    atomicAdd(&S.E[r], (unsigned long long)g.weight(S.pi[v]));
                    atomicAdd(&S.JM[r], 1u);
                    if (RATIO)
                        atomicAdd((unsigned long long*)&S.T[r], (unsigned long long)g.time(S.pi[v]));
                }
            __syncthreads();
            if (t < 64) {
                long long bw = 0, bl = 1;
                int br = -1;
                for (unsigned i = t; i < S.cnt; i += 64) {
                    const int r = S.layer[i];
                    const long long cw = (long long)S.E[r];
                    const long long cl = RATIO ? S.T[r] : (long long)S.JM[r];
                    if (cand_less(cw, cl, r, bw, bl, br)) {
                        bw = cw;
                        bl = cl;
                        br = r;
                    }
                }
                for (int off = 32; off > 0; off >>= 1) {
                    const long long ow = __shfl_xor(bw, off, 64), ol = __shfl_xor(bl, off, 64);
                    const int orr = __shfl_xor(br, off, 64);
                    if (cand_less(ow, ol, orr, bw, bl, br)) {
                        bw = ow;
                        bl = ol;
                        br = orr;
                    }
                }
                if (t == 0) {
                    S.selW = bw;
                    S.selL = bl;
                    S.selS = br;
                    S.cap = S.JM[br];   // C's edges
                    S.cnt = 0;
                }
            }
            __syncthreads();
            s = S.selS;
            W = S.selW;
            L = S.selL;
            R.clen = S.cap;
            // rebuild (R5, R6): C's component keeps its edges; round k
            // attaches every other vertex with an out-edge into the vertices
            // attached before round k, by its lowest such edge.  A vertex
            // attached in round k is written at once: the others' test
            // (layer < k) ignores it either way.
            unsigned mine = 0;
            for (int v = t; v < n; v += B) {
                const bool keep = S.rep[v] == s;
                S.layer[v] = keep ? 0 : 0xffffu;
                mine += !keep;
                if (keep && S.onc[v]) S.onc[v] = 3;
            }
            unsigned left = __popcll(__ballot(mine & 1)) + 2 * __popcll(__ballot(mine & 2)) +
                            4 * __popcll(__ballot(mine & 4));
            if ((t & 63) == 0 && left) atomicAdd(&S.cnt, left);
            if (t < 2) S.got[t + 1] = 0;
            __syncthreads();
            left = S.cnt;
            for (int k = 1; left > 0; ++k) {
                // counters take turns: round k adds to got[k % 3], which all
                // read after its barrier, and clears the next round's
                if (t == 0 && k > 1) S.got[(k + 1) % 3] = 0;
                unsigned got = 0;
                for (int i = t >> 6; LISTED && i < nl + nw; i += B >> 6) {
                    const int v = i < nl ? S.longs[i] : S.wides[i - nl];
                    if (S.layer[v] != 0xffffu) continue;   // this wave's to write
                    const int end = S.rb[v + 1];
                    int at = -1, x = 0;
                    for (int eb = S.rb[v]; eb < end && at < 0; eb += 64 * kRowSteps) {
                        int h[kRowSteps];
                        unsigned short ly[kRowSteps];
#pragma unroll
                        for (int u = 0; u < kRowSteps; ++u) {
                            const int e = eb + 64 * u + (t & 63);
                            h[u] = g.head(e < end ? e : end - 1);
                        }
#pragma unroll
                        for (int u = 0; u < kRowSteps; ++u) ly[u] = S.layer[h[u]];
#pragma unroll
                        for (int u = kRowSteps - 1; u >= 0; --u) {
                            const unsigned long long hit =
                                __ballot((int)ly[u] < k && eb + 64 * u + (t & 63) < end);
                            if (!hit) continue;
                            const int l = __ffsll((long long)hit) - 1;
                            at = eb + 64 * u + l;
                            x = __shfl(h[u], l, 64);
                        }
                    }
                    if (at >= 0 && (t & 63) == 0) {
                        S.pi[v] = (unsigned short)at;
                        S.succ[v] = (unsigned short)x;
                        S.layer[v] = (unsigned short)k;
                        ++got;
                    }
                }
                for (int v = t; v < n; v += B) {
                    if (S.layer[v] != 0xffffu) continue;
                    if (LISTED && (int)S.rb[v + 1] - (int)S.rb[v] > kLongEdges) continue;
                    for (int e = S.rb[v]; e < (int)S.rb[v + 1]; ++e) {
                        const int x = g.head(e);
                        if ((int)S.layer[x] < k) {
                            S.pi[v] = (unsigned short)e;
                            S.succ[v] = (unsigned short)x;
                            S.layer[v] = (unsigned short)k;
                            ++got;
                            break;
                        }
                    }
                }
                if (got) atomicAdd(&S.got[k % 3], got);
                __syncthreads();
                got = S.got[k % 3];
                ++R.connect;
                if (got == 0) {
                    R.status = OCM_E_NOT_STRONGLY_CONNECTED;
                    break;
                }
                left -= got;
            }
            if (R.status != OCM_OK) break;
            for (int v = t; v < n; v += B) {
                if (!g.entry(v, s, L, W, S.pi[v], S.succ[v])) S.over = 1;
            }
            __syncthreads();
        }
        ++R.values;
        ++R.jumps;
        chase<WIDE>(S, n, (unsigned)s);
        __syncthreads();
        if (S.stall) {
            if (general) {
                R.status = kSmallFallback;   // cannot be: every vertex is attached
                break;
            }
            general = true;
            __syncthreads();
            if (t == 0) S.stall = S.over = 0;
            __syncthreads();
            continue;
        }
        if (S.over) {
            R.status = kSmallFallback;
            break;
        }
        if (!general) ++R.fast;
        // improvement sweep (R2): strict improvement, lowest position; counts
        // the tight edges other than the policy edge as the tie scan does
        int np[VPT], nh[VPT];
        unsigned tight = 0, certain = 0, changed = 0;
        bool broke = false;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            const int v = t + i * B;
            bool ch = false;
            np[i] = nh[i] = 0;
            if (v < n) {
                const long long own = g.value(v);
                const int cur = S.pi[v];
                const bool onC = S.onc[v] == 3;
                long long best = INT64_MAX;
                int arg = 0, bh = 0;
                const int end = S.rb[v + 1];
                const bool listed = LISTED && end - (int)S.rb[v] > kLongEdges;
                for (int eb = listed ? end : S.rb[v]; eb < end; eb += 4) {
                    // four edges in flight (past the row: its last edge again)
                    int x[4];
                    long long key[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int e = eb + u < end ? eb + u : end - 1;
                        x[u] = g.head(e);
                        key[u] = L * g.weight(e) - (RATIO ? W * g.time(e) : W);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) key[u] += g.value(x[u]);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (eb + u >= end) break;
                        if (key[u] < best) {
                            best = key[u];
                            arg = eb + u;
                            bh = x[u];
                        }
                        if (key[u] == own && eb + u != cur) {
                            ++tight;
                            certain += x[u] == v || onC;
                        }
                    }
                }
                ch = best < own;
                np[i] = listed ? -1 : ch ? arg : cur;
                nh[i] = ch ? bh : (int)S.succ[v];
                broke |= ch && onC;
            }
            changed += __popcll(__ballot(ch));
        }
        // their policy is written at once: only the row's own scan reads it
        if (LISTED) listed_rows<false>(g, nl, nw, L, W, tight, certain, [&](int v, long long best, int arg, int bh) {
            if (best >= g.value(v)) return;
            ++changed;
            broke |= S.onc[v] == 3;
            if ((t & 63) == 0) {
                S.pi[v] = (unsigned short)arg;
                S.succ[v] = (unsigned short)bh;
            }
        });
        const bool any_t = __ballot(tight != 0) != 0, any_b = __ballot(broke) != 0;
        if (any_t) {
            tight = (unsigned)wave_sum_u64(tight);
            certain = (unsigned)wave_sum_u64(certain);
        }
        if ((t & 63) == 0) {
            if (changed) atomicAdd(&S.acc[par][0], changed);
            if (any_b) atomicOr(&S.acc[par][1], 1u);
            if (any_t) {
                atomicAdd(&S.acc[par][2], tight);
                atomicAdd(&S.acc[par][3], certain);
            }
        }
        __syncthreads();
        changed = S.acc[par][0];
        R.tight = S.acc[par][2];
        R.certain = S.acc[par][3];
        general = S.acc[par][1] != 0 || !o.fast_path;
        ++R.iter;
        if (changed == 0) break;
        if (R.iter >= o.iter_cap) {
            R.status = OCM_E_NOT_CONVERGED;
            break;
        }
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            const int v = t + i * B;
            if (v < n) {
                if (LISTED && np[i] < 0) {   // a listed row
                    np[i] = S.pi[v];
                    nh[i] = S.succ[v];
                }
                S.pi[v] = (unsigned short)np[i];
                S.succ[v] = (unsigned short)nh[i];
                if (!general && !g.entry(v, s, L, W, np[i], nh[i])) S.over = 1;
            }
        }
        par ^= 1;
        if (t < 4) S.acc[par][t] = 0;
        __syncthreads();
    }
    __syncthreads();
    R.s = s;
    R.W = W;
    R.L = L;
    if (R.status != OCM_OK || !o.tie_check || R.tight == 0) return;
    if (R.certain) {
        R.tie = true;
        return;
    }
    // Exact uniqueness of C: no tight edge leaves C, so a second critical
    // cycle lies outside it.  Vertices are taken out, C first, once no tight
    // edge leads to one that is left; a cycle is all that can stay.
    for (int v = t; v < n; v += B) S.layer[v] = S.onc[v] != 3;
    for (;;) {
        __syncthreads();
        if (t == 0) S.flag = S.cnt = 0;
        __syncthreads();
        bool out = false, stay = false;
        for (int i = t >> 6; LISTED && i < nl + nw; i += B >> 6) {
            const int v = i < nl ? S.longs[i] : S.wides[i - nl];
            if (!S.layer[v]) continue;   // this wave's to write
            const long long own = g.value(v);
            const int end = S.rb[v + 1];
            bool alive = false;
            for (int eb = S.rb[v]; eb < end && !alive; eb += 64) {
                const int e = eb + (t & 63);
                bool a = false;
                if (e < end) {
                    const int x = g.head(e);
                    a = S.layer[x] &&
                        g.value(x) + L * g.weight(e) - (RATIO ? W * g.time(e) : W) == own;
                }
                alive = __ballot(a) != 0;
            }
            if (!alive && (t & 63) == 0) S.layer[v] = 0;
            out |= !alive;
            stay |= alive;
        }
        for (int v = t; v < n; v += B) {
            if (!S.layer[v] || (LISTED && (int)S.rb[v + 1] - (int)S.rb[v] > kLongEdges)) continue;
            const long long own = g.value(v);
            bool alive = false;
            for (int e = S.rb[v]; e < (int)S.rb[v + 1] && !alive; ++e) {
                const int x = g.head(e);
                if (!S.layer[x]) continue;
                alive = g.value(x) + L * g.weight(e) - (RATIO ? W * g.time(e) : W) == own;
            }
            if (!alive) S.layer[v] = 0;
            out |= !alive;
            stay |= alive;
        }
        if (out) S.flag = 1;
        if (stay) S.cnt = 1;
        __syncthreads();
        if (S.cnt == 0) return;
        if (S.flag == 0) break;
    }
    R.tie = true;
}

// The whole solve; every thread returns the same Run.  row_ptr[0..n] holds the
// rows' edge positions (e0 = row_ptr[0] when the CSR is known to be sound).
template <bool WIDE, typename WT, int N, int M, bool RATIO>
__device__ void solve_one(Lds<N, M, RATIO>& S, int n, int m, int v0, int e0,
                          const int* __restrict__ row_ptr, const int* __restrict__ col,
                          const WT* __restrict__ w, const int* __restrict__ tm, bool neg,
                          const SmallOpts& o, const int* __restrict__ init, Run& R)
{
    const int t = threadIdx.x, B = blockDim.x;
    R = Run{};
    R.status = OCM_OK;
    R.s = 0;
    R.L = 1;
    // rows, edges, validation (as k_validate), the weight bound
    if (t == 0) {
        S.err = 0;
        S.maxw = 0;
        S.maxt = 1;
        S.cap = 0;
        S.nlong = S.nwide = 0;
        S.stall = S.over = 0;
        for (int p = 0; p < 2; ++p)
            for (int i = 0; i < 4; ++i) S.acc[p][i] = 0;
    }
    __syncthreads();
    {
        unsigned err = 0;
        for (int v = t; v < n; v += B) {
            const int b = row_ptr[v], x = row_ptr[v + 1];
            if (o.validate) {
                if ((v == 0 && b != e0) || (v == n - 1 && x != e0 + m) || b < e0 || x > e0 + m || b > x)
                    err |= kErrBadCsr;
                else if (b == x) err |= kErrNoOut;
            }
            S.rb[v] = (unsigned short)(b - e0);
            if (v == n - 1) S.rb[n] = (unsigned short)(x - e0);
        }
        unsigned long long mw = 0;
        int mt = 1;
        bool bad_t = false;
        for (int e = t; e < m; e += B) {
            const int h = col[e0 + e] - v0;
            if (o.validate && (h < 0 || h >= n)) err |= kErrBadCsr;
            const long long x = (long long)w[e0 + e];
            const unsigned long long ax = uabs64(x);
            mw = ax > mw ? ax : mw;
            if (M > 0) {
                S.c[e] = (unsigned short)h;
                S.w[e] = (int)x;
            }
            if (RATIO) {
                const int y = tm[e0 + e];
                bad_t |= y < 1;
                mt = y > mt ? y : mt;
                if (M > 0) S.t[e] = y;
            }
        }
        if (err) atomicOr(&S.err, err);
        if (bad_t) atomicOr(&S.cap, 1u);
        mw = wave_max_u64(mw);
        if ((t & 63) == 0) atomicMax(&S.maxw, mw);
        if (RATIO) atomicMax(&S.maxt, (unsigned)mt);
    }
    __syncthreads();
    const unsigned long long maxw = S.maxw;
    if (S.err & kErrBadCsr) R.status = OCM_E_BAD_CSR;
    else if (S.err & kErrNoOut) R.status = OCM_E_NO_OUT_EDGE;
    else if (S.cap) R.status = OCM_E_INVALID_ARG;
    else if ((unsigned __int128)2 * (unsigned)n * maxw * S.maxt >= ((unsigned __int128)1 << 62) &&
             o.bound)
        R.status = OCM_E_OVERFLOW;
    if (R.status != OCM_OK) {
        R.tight = R.status == OCM_E_INVALID_ARG ? 1u : 0u;   // which argument: times
        return;
    }
    const View<WT, N, M, RATIO, WIDE> g{S, col, w, tm, v0, e0, neg, maxw <= (unsigned long long)INT32_MAX};

    for (int v = t; v < n; v += B) {
        const int len = (int)S.rb[v + 1] - (int)S.rb[v];
        if (len <= kLongEdges) continue;
        // (rows of an unchecked, unsound CSR may be more than there is room for)
        const bool wide = len > kWideEdges;
        const unsigned at = atomicAdd(wide ? &S.nwide : &S.nlong, 1u);
        if (at < (wide ? sizeof S.wides : sizeof S.longs) / 2) (wide ? S.wides : S.longs)[at] = (unsigned short)v;
        else atomicSub(wide ? &S.nwide : &S.nlong, 1u);
    }
    __syncthreads();
    const int nl = __builtin_amdgcn_readfirstlane((int)S.nlong);
    const int nw = __builtin_amdgcn_readfirstlane((int)S.nwide);

    if (nl + nw > 0) iterate<true>(g, nl, nw, n, e0, o, init, R);
    else iterate<false>(g, 0, 0, n, e0, o, init, R);
}

// Policy hops to s into out (the values are gone afterwards).
template <bool WIDE, int N, int M, bool RATIO>
__device__ __forceinline__ void hops(Lds<N, M, RATIO>& S, int n, int s)
{
    __syncthreads();
    for (int v = threadIdx.x; v < n; v += blockDim.x) {
        const unsigned to = v == s ? (unsigned)s : S.succ[v];
        if (WIDE) S.JM[v] = to;
        S.E[v] = WIDE ? (unsigned long long)(v != s) : ((unsigned long long)(v != s) << kBits) | to;
    }
    __syncthreads();
    chase<WIDE>(S, n, (unsigned)s);
    __syncthreads();
}

template <typename WT, int N, int M, bool RATIO>
__global__ __launch_bounds__(1024) void k_small_one(int n, int m, const int* __restrict__ row_ptr,
                                                    const int* __restrict__ col,
                                                    const WT* __restrict__ w,
                                                    const int* __restrict__ tm, int neg, SmallOpts o,
                                                    SmallPtrs p)
{
    __shared__ Lds<N, M, RATIO> S;
    Run R;
    solve_one<false, WT, N, M, RATIO>(S, n, m, 0, 0, row_ptr, col, w, tm, neg != 0, o, p.init, R);
    if (R.status == OCM_OK && (long long)R.clen <= o.cycle_cap) {
        for (int v = threadIdx.x; v < n; v += blockDim.x) {
            if (p.policy) p.policy[v] = S.pi[v];
            if (p.potential) p.potential[v] = (long long)S.E[v] >> kBits;
        }
        hops<false>(S, n, R.s);
        for (int v = threadIdx.x; v < n; v += blockDim.x)
            if (S.onc[v] == 3)
                p.cycle[v == R.s ? 0 : (int)R.clen - (int)(S.E[v] >> kBits)] = S.pi[v];
    }
    if (threadIdx.x == 0) {
        SmallOut x;
        x.W = R.W;
        x.L = R.L;
        x.status = R.status;
        x.s = R.s;
        x.iterations = R.iter;
        x.fast = R.fast;
        x.general = R.general;
        x.connect_rounds = R.connect;
        x.jump_rounds = R.jumps;
        x.value_rounds = R.values;
        x.clen = R.clen;
        x.tight = R.tight;
        x.tie = R.tie ? 1u : 0u;
        *p.out = x;
        if (p.seq) {
            __threadfence_system();
            __hip_atomic_store(p.seq, p.want, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// The batched small class: graphs list[0..nlist) of the union, a workgroup
// each (grid-stride).  A graph whose sums do not fit the entries is left to a
// second launch with 64-bit values (WIDE; the graphs that are done pass), then to
// the loop.  300 graphs of 1000 vertices, ms in the loop / so: weights to 2^44 4.08 /
// 1.01, to 2^50 8.99 / 0.79.
template <typename WT, int N, int M, bool WIDE>
__global__ __launch_bounds__(1024) void k_small_batch(const int* __restrict__ list, int nlist,
                                                      SmallBatch b, const int* __restrict__ row_ptr,
                                                      const int* __restrict__ col,
                                                      const WT* __restrict__ w, int neg, SmallOpts o)
{
    __shared__ Lds<N, M, false> S;
    for (int li = blockIdx.x; li < nlist; li += gridDim.x) {
        const int g = list[li];
        if (WIDE && b.mode[g] == 0) continue;
        const int v0 = (int)b.vptr[g], e0 = (int)b.eptr[g];
        const int n = (int)(b.vptr[g + 1] - v0), m = (int)(b.eptr[g + 1] - e0);
        Run R;
        solve_one<WIDE, WT, N, M, false>(S, n, m, v0, e0, row_ptr + v0, col, w, nullptr, neg != 0, o,
                                         nullptr, R);
        if (R.status == OCM_OK) {
            for (int v = threadIdx.x; v < n; v += blockDim.x) {
                b.pi[v0 + v] = e0 + S.pi[v];
                b.succ[v0 + v] = v0 + S.succ[v];
                b.V[v0 + v] = WIDE ? (long long)S.E[v] : (long long)S.E[v] >> kBits;
                b.onC[v0 + v] = S.onc[v] == 3;
            }
            hops<WIDE>(S, n, R.s);
            for (int v = threadIdx.x; v < n; v += blockDim.x)
                b.hop[v0 + v] = (int)(WIDE ? S.E[v] : S.E[v] >> kBits);
        }
        if (threadIdx.x == 0 && R.status != kSmallFallback) {
            b.W[g] = R.W;
            b.L[g] = R.L;
            b.s[g] = v0 + R.s;
            b.iter[g] = R.iter;
            b.status[g] = R.status;
            b.mode[g] = 0;   // done; a graph left to the loop keeps its initial state
        }
        __syncthreads();   // S is reused by the next graph
    }
}

}  // namespace sm

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Class of a graph: the smallest that holds it, -1 if none does.
int small_class(int64_t n, int64_t m, bool ratio)
{
    if (m > kSmallMaxM) return -1;
    if (n <= 512 && m <= 4096) return 0;
    if (n <= 1024 && m <= 8192) return 1;
    if (n <= 2048 && m <= (ratio ? 8192 : 16384)) return 2;
    return n <= kSmallMaxN ? 3 : -1;
}

template <typename WT, bool RATIO>
static void launch_one(int cls, int n, int m, const int* row_ptr, const int* col, const WT* w,
                       const int* t, int neg, const SmallOpts& o, const SmallPtrs& p, hipStream_t st)
{
    switch (cls) {
        case 0:
            sm::k_small_one<WT, 512, 4096, RATIO><<<1, n <= 128 ? 128 : n <= 256 ? 256 : 512, 0, st>>>(n, m, row_ptr, col, w, t, neg, o, p);
            break;
        case 1:
            sm::k_small_one<WT, 1024, 8192, RATIO><<<1, 1024, 0, st>>>(n, m, row_ptr, col, w, t, neg, o, p);
            break;
        case 2:
            sm::k_small_one<WT, 2048, RATIO ? 8192 : 16384, RATIO>
                <<<1, 1024, 0, st>>>(n, m, row_ptr, col, w, t, neg, o, p);
            break;
        default:
            sm::k_small_one<WT, 4096, 0, RATIO><<<1, 1024, 0, st>>>(n, m, row_ptr, col, w, t, neg, o, p);
    }
}

void launch_small_one(int n, int m, const int* row_ptr, const int* col, const void* w, int wtype,
                      const int* t, int neg, const SmallOpts& o, const SmallPtrs& p, hipStream_t st)
{
    const int cls = small_class(n, m, t != nullptr);
    if (wtype == kWI64) {
        if (t) launch_one<long long, true>(cls, n, m, row_ptr, col, (const long long*)w, t, neg, o, p, st);
        else launch_one<long long, false>(cls, n, m, row_ptr, col, (const long long*)w, t, neg, o, p, st);
    } else {
        if (t) launch_one<int, true>(cls, n, m, row_ptr, col, (const int*)w, t, neg, o, p, st);
        else launch_one<int, false>(cls, n, m, row_ptr, col, (const int*)w, t, neg, o, p, st);
    }
}

template <typename WT, bool WIDE>
static void launch_batch(int cls, const int* list, int nlist, const SmallBatch& b, const int* row_ptr,
                         const int* col, const WT* w, int neg, const SmallOpts& o, hipStream_t st)
{
    // one graph per workgroup, dispatched as earlier ones end
    switch (cls) {
        case 0:
            sm::k_small_batch<WT, 512, 4096, WIDE><<<nlist, 256, 0, st>>>(list, nlist, b, row_ptr, col, w, neg, o);
            break;
        case 1:
            sm::k_small_batch<WT, 1024, 8192, WIDE><<<nlist, 512, 0, st>>>(list, nlist, b, row_ptr, col, w, neg, o);
            break;
        case 2:
            sm::k_small_batch<WT, 2048, 16384, WIDE><<<nlist, 1024, 0, st>>>(list, nlist, b, row_ptr, col, w, neg, o);
            break;
        default:
            sm::k_small_batch<WT, 4096, 0, WIDE><<<nlist, 1024, 0, st>>>(list, nlist, b, row_ptr, col, w, neg, o);
    }
}

void launch_small_batch(int cls, const int* list, int nlist, const SmallBatch& b, const int* row_ptr,
                        const int* col, const void* w, int wtype, int neg, const SmallOpts& o,
                        bool wide, hipStream_t st)
{
    if (nlist <= 0) return;
    const auto* w64 = (const long long*)w;
    const auto* w32 = (const int*)w;
    if (wtype == kWI64) {
        launch_batch<long long, false>(cls, list, nlist, b, row_ptr, col, w64, neg, o, st);
        if (wide) launch_batch<long long, true>(cls, list, nlist, b, row_ptr, col, w64, neg, o, st);
    } else {
        launch_batch<int, false>(cls, list, nlist, b, row_ptr, col, w32, neg, o, st);
        if (wide) launch_batch<int, true>(cls, list, nlist, b, row_ptr, col, w32, neg, o, st);
    }
}

}  // namespace ocm
