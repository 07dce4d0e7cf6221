// Device code shared by the single-query kernels (query.hip) and the batched
// engine (batch.hip): triangle enumeration, the exact run filter, the temporal
// tests.  See query.hip for what each step computes and where the paper says so.
#pragma once

#include <cstdlib>

#include "folty_internal.h"

namespace folty {
namespace {

constexpr int BLK = 256;
constexpr int WPB = BLK / 64;         // wavefronts per block
constexpr int CAP = 512;              // N+(u) staged in LDS up to this length
constexpr int PERSIST_BLOCKS = 4096;
constexpr int ENUM_BLOCKS = 32768; // many more than are resident: a few items per wavefront, balanced by the dispatcher
constexpr int32_t CHUNK = 3072;       // closing probes per enumeration item (about; whole segments)

__device__ inline int lane_id() { return __lane_id(); }

// A pointer field of a table in device memory (a plan's per-job records), read
// as a pointer to global memory.  The compiler cannot tell where such a pointer
// points and would use flat instructions, whose completion shares one wait
// counter with LDS and scalar loads (so every LDS wait would also wait for the
// global loads in flight).
template <class T> __device__ inline T *global_ptr(T *const &field) {
    __attribute__((address_space(1))) T *g;
    __builtin_memcpy(&g, &field, sizeof g);
    return (T *)g;
}

// this wavefront's index in its block, as a value the compiler knows is uniform
// (so what is indexed by it is loaded into scalar registers)
__device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

__device__ inline unsigned long long lanes_below() { return (1ull << lane_id()) - 1ull; }

// make this wavefront's LDS writes visible to all of its lanes
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline int32_t wave_append(int32_t *counter, bool pred) {
    unsigned long long mask = __ballot(pred);
    if (!mask) return -1;
    int lane = lane_id();
    int leader = __ffsll((long long)mask) - 1;
    int32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, (int32_t)__popcll(mask));
    base = __shfl(base, leader);
    return pred ? base + (int32_t)__popcll(mask & lanes_below()) : -1;
}

template <class T> __device__ inline T wave_inclusive_sum(T x) {
    const int lane = lane_id();
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    return x;
}

// adds to this block's region's counter `what`
__device__ inline void region_add(unsigned long long *scal, int what, unsigned long long x) {
    atomicAdd(&scal[SCAL_REGIONS + (blockIdx.x % MAX_REGIONS) * REGION_WORDS + what], x);
}

// the predicate code as a compile-time constant for kernel templates
template <class F> void dispatch_variant(int v, F &&f) {
    switch (v) {
    case 0: f(std::integral_constant<int, 0>{}); break;
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    default: f(std::integral_constant<int, 7>{}); break;
    }
}

template <class T> __global__ void k_fill(T *p, T v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// directed lists of a triangle
// ---------------------------------------------------------------------------
struct Span {
    int32_t s, n;     // start in ts, length
    uint32_t lo, hi;  // first and last timestamp >> tshift
};

// D[i][j] = E_{x_i, x_j} for the triangle's vertices x0 < x1 < x2 (by rank)
struct TriLists {
    Span d01, d10, d02, d20, d12, d21;
    template <int I, int J> __device__ inline const Span &get() const {
        static_assert(I != J, "");
        if constexpr (I == 0 && J == 1) return d01;
        else if constexpr (I == 1 && J == 0) return d10;
        else if constexpr (I == 0 && J == 2) return d02;
        else if constexpr (I == 2 && J == 0) return d20;
        else if constexpr (I == 1 && J == 2) return d12;
        else return d21;
    }
};

// STARTS: also the lists' starts in ts (the filter needs only lengths and ranges)
template <bool STARTS>
__device__ inline void rec_spans(const EdgeRec *__restrict__ rec, int32_t p, Span &fwd, Span &bwd) {
    const uint4 *q = reinterpret_cast<const uint4 *>(rec + p);
    if constexpr (STARTS) {
        const uint4 a = q[0];
        fwd.n = (int32_t)a.x;
        bwd.n = (int32_t)a.y;
        fwd.s = (int32_t)a.z;
        bwd.s = (int32_t)a.w;
    } else {
        const uint2 a = *reinterpret_cast<const uint2 *>(q);
        fwd.n = (int32_t)a.x;
        bwd.n = (int32_t)a.y;
        fwd.s = bwd.s = 0;
    }
    const uint4 b = q[1];
    fwd.lo = b.x;
    fwd.hi = b.y;
    bwd.lo = b.z;
    bwd.hi = b.w;
}

// the three oriented edges (x0,x1), (x0,x2), (x1,x2) of a triangle
template <bool STARTS = true>
__device__ inline TriLists load_lists(const EdgeRec *__restrict__ rec, int32_t p01, int32_t p02, int32_t p12) {
    TriLists L;
    rec_spans<STARTS>(rec, p01, L.d01, L.d10);
    rec_spans<STARTS>(rec, p02, L.d02, L.d20);
    rec_spans<STARTS>(rec, p12, L.d12, L.d21);
    return L;
}

// Slack of the run test below in timestamps >> tshift: the range slack of the
// window bound, saturated to 32 bits (no difference of two such values exceeds it).
__host__ __device__ inline uint32_t run_slack(int64_t dq) {
    return dq >= (int64_t)0xffffffffu ? 0xffffffffu : (uint32_t)dq;
}

// The predicate code picks, for L1 = E_{a,b} (a = x_I, b = x_J, third w = x_C),
// L2 between X and w and L3 between Y and w (see folty.h for the bits).
template <int VAR, int I, int J> struct Pick {
    static constexpr int C = 3 - I - J;
    static constexpr int X = (VAR & 4) ? J : I;
    static constexpr int Y = (VAR & 4) ? I : J;
    static constexpr int L2a = (VAR & 1) ? C : X, L2b = (VAR & 1) ? X : C;
    static constexpr int L3a = (VAR & 2) ? C : Y, L3b = (VAR & 2) ? Y : C;
};

// A run can only count if all three lists are non-empty and some t <= t2 <= t3
// <= t + dmax is possible given each list's first and last timestamp.  The test
// reads the timestamps shifted right by tshift with slack dq = run_slack(
// range_slack(dmax, tshift)): a run it drops has no such t, t2, t3 (floors keep
// order, and floors of two values differ by at most one more unit than the
// values do); with tshift = 0 it is exact.  A run it keeps without such a
// window only adds tests that find nothing.
template <int VAR, int I, int J>
__device__ inline bool run_lists(const TriLists &T, uint32_t dq, Span &l1, Span &l2, Span &l3) {
    using P = Pick<VAR, I, J>;
    l1 = T.template get<I, J>();
    l2 = T.template get<P::L2a, P::L2b>();
    l3 = T.template get<P::L3a, P::L3b>();
    if (l1.n == 0 || l2.n == 0 || l3.n == 0) return false;
    if (l2.hi < l1.lo || l3.hi < l2.lo) return false;
    if ((l2.lo > l1.hi && l2.lo - l1.hi > dq) || (l3.lo > l1.hi && l3.lo - l1.hi > dq)) return false;
    return true;
}

// Tests of a run: |L1|, or with SS the shorter of |L1| and |L2| (the side the
// run is evaluated from; see chunk_run).
template <bool SS> __device__ inline int32_t run_tests(const Span &l1, const Span &l2) {
    return SS && l2.n < l1.n ? l2.n : l1.n;
}

template <int VAR, int I, int J, bool SS = false> __device__ inline int64_t run_work(const TriLists &T, uint32_t dq) {
    Span a, b, c;
    return run_lists<VAR, I, J>(T, dq, a, b, c) ? run_tests<SS>(a, b) : 0;
}

template <int VAR, bool SS = false> __device__ inline int64_t tri_work(const TriLists &T, uint32_t dq) {
    return run_work<VAR, 0, 1, SS>(T, dq) + run_work<VAR, 1, 0, SS>(T, dq) + run_work<VAR, 0, 2, SS>(T, dq) +
           run_work<VAR, 2, 0, SS>(T, dq) + run_work<VAR, 1, 2, SS>(T, dq) + run_work<VAR, 2, 1, SS>(T, dq);
}

// the runs that can count, as bits in the order of tri_work's sum
template <int VAR> __device__ inline uint32_t tri_live(const TriLists &T, uint32_t dq) {
    Span a, b, c;
    return (uint32_t)run_lists<VAR, 0, 1>(T, dq, a, b, c) | (uint32_t)run_lists<VAR, 1, 0>(T, dq, a, b, c) << 1 |
           (uint32_t)run_lists<VAR, 0, 2>(T, dq, a, b, c) << 2 | (uint32_t)run_lists<VAR, 2, 0>(T, dq, a, b, c) << 3 |
           (uint32_t)run_lists<VAR, 1, 2>(T, dq, a, b, c) << 4 | (uint32_t)run_lists<VAR, 2, 1>(T, dq, a, b, c) << 5;
}
// a predicate code read at run time (one per job in a batch)
__device__ inline uint32_t tri_live_rt(int variant, const TriLists &T, uint32_t dq) {
    switch (variant) {
    case 0: return tri_live<0>(T, dq);
    case 1: return tri_live<1>(T, dq);
    case 2: return tri_live<2>(T, dq);
    case 3: return tri_live<3>(T, dq);
    case 4: return tri_live<4>(T, dq);
    case 5: return tri_live<5>(T, dq);
    case 6: return tri_live<6>(T, dq);
    default: return tri_live<7>(T, dq);
    }
}

// Searches probe four entries at a time: a search is a chain of dependent reads,
// and four reads take as long as one (a list of up to four entries is decided by
// one step, one of 5,000 by six instead of thirteen).
struct Probe {
    int64_t x[4];
};
__device__ inline int32_t probe_step(int32_t len) { return len > 4 ? len >> 2 : 1; }
// entries a, a + step, a + 2 step, a + 3 step of L[a, b) (its last one past the end); b >= 1
__device__ inline Probe probe(const int64_t *__restrict__ L, int32_t a, int32_t b) {
    const int32_t q = probe_step(b - a);
    Probe P;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const int32_t i = a + k * q;
        P.x[k] = L[i < b ? i : b - 1];
    }
    return P;
}
// first position in [a, n) with L[position] >= key (n if none), whose entry is
// left in val; P = probe(L, a, n)
__device__ inline int32_t lower_bound(const int64_t *__restrict__ L, int32_t a, int32_t n, int64_t key, Probe P,
                                      int64_t &val) {
    int32_t b = n;
    while (a < b) {
        const int32_t q = probe_step(b - a);
        const int c = (P.x[0] < key) + (a + q < b && P.x[1] < key) + (a + 2 * q < b && P.x[2] < key) +
                      (a + 3 * q < b && P.x[3] < key); // probes below key: the first c
        const int32_t hi = a + c * q;
        if (c == 0) {
            val = P.x[0];
            return a;
        }
        if (c < 4 && hi < b) {
            val = c == 1 ? P.x[1] : c == 2 ? P.x[2] : P.x[3];
            b = hi;
        }
        a += (c - 1) * q + 1;
        if (a < b) P = probe(L, a, b);
    }
    return b;
}
// first position p in [from, n) with L[p] >= key (n if none)
__device__ inline int32_t lower_bound_from(const int64_t *__restrict__ L, int32_t from, int32_t n, int64_t key) {
    if (from >= n || L[from] >= key) return from; // a cursor often stays where it is
    int64_t val;
    return from + 1 < n ? lower_bound(L, from + 1, n, key, probe(L, from + 1, n), val) : n;
}

// A run's list L2 or L3.  ends: null, or the record's first and last timestamp
// (32 bits each), from which a list of one or two entries is read: most lists are
// that short, their entries are scattered reads that no neighbouring test shares,
// and the record has just been read.
struct List {
    const int64_t *p;
    int32_t n;
    const int64_t *ends;
    template <bool SHORT> __device__ inline Probe at(int32_t a) const {
        if constexpr (SHORT) {
            const int32_t q = probe_step(n - a);
            Probe P;
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const int32_t i = a + k * q;
                const int64_t *r = ends ? ends : p + (i < n ? i : n - 1);
                P.x[k] = *r;
            }
            if (ends) {
                const int64_t lo = (int64_t)(uint32_t)P.x[0], hi = (int64_t)((uint64_t)P.x[0] >> 32);
                P.x[0] = a == 0 ? lo : hi;
                P.x[1] = P.x[2] = P.x[3] = hi;
            }
            return P;
        } else {
            return probe(p, a, n);
        }
    }
};

// The test of an edge at time t (paper, Theorems 3.1 and 3.2): with t2 the first
// entry of L2 at or after t and t3 the first of L3 at or after t2, the edge's
// smallest window is t3 - t.  c2, c3: positions before which no entry can matter
// (below the lists' lengths), moved forward; p2, p3: the probes there.
enum TestEnd { TEST_MISS, TEST_HIT, TEST_END }; // TEST_END: nothing for any later edge either
__device__ inline TestEnd window_test(const List &l2, const List &l3, int32_t &c2, int32_t &c3, const Probe &p2,
                                      const Probe &p3, int64_t t, int64_t dmax, int64_t &win) {
    int64_t t2 = 0, t3 = 0;
    c2 = lower_bound(l2.p, c2, l2.n, t, p2, t2);
    if (c2 == l2.n) return TEST_END;
    if (t2 - t > dmax) return TEST_MISS;
    c3 = lower_bound(l3.p, c3, l3.n, t2, p3, t3);
    if (c3 == l3.n) return TEST_END;
    win = t3 - t;
    return win <= dmax ? TEST_HIT : TEST_MISS;
}

// counts the edges whose window is at most delta
struct DirectOp {
    int64_t delta;
    uint32_t *count;
    int32_t *diff; // per sorted edge + 1: +1 / -1 at the ends of edge ranges (interval evaluation)
    __device__ inline int64_t most() const { return delta; }
    __device__ inline void hit(int32_t e, int64_t) const { atomicAdd(&count[e], 1u); }

    // The same run evaluated from L2 (paper, the in-neighbour theorem: e forms
    // a triangle with w iff some entry t2 of L2, with t3 the first entry of L3
    // at or after t2 and t3 - t2 <= delta, has t3 - delta <= t(e) <= t2).
    // Those intervals have non-decreasing ends, so entry j adds exactly the
    // times in [max(t3 - delta, t2' + 1), t2] (t2' the entry before it) to the
    // union of the earlier ones; each such piece is a range of L1 marked +1 / -1
    // in diff, whose prefix sum over the sorted edges adds one per third vertex.
    // Entries [j0, j0 + cnt) of L2; l1s: L1's start among the sorted edges.
    __device__ inline void iv(const List &l1, int32_t l1s, int32_t j0, int32_t cnt, const List &l2,
                              const List &l3) const {
        int32_t c3 = 0, a = 0, b = 0;
        for (int32_t j = j0; j < j0 + cnt; j++) {
            const Probe p3 = probe(l3.p, c3, l3.n);
            const Probe p1 = probe(l1.p, b, l1.n); // b < |L1| (see below)
            const int64_t t2 = l2.p[j], before = l2.p[j > 0 ? j - 1 : 0];
            int64_t t3 = 0, x = 0;
            c3 = lower_bound(l3.p, c3, l3.n, t2, p3, t3);
            if (c3 == l3.n) break; // no t3 for this or any later entry
            if (t3 - t2 > delta) continue; // an empty interval
            int64_t lo = t3 - delta;
            if (j > 0 && before + 1 > lo) lo = before + 1;
            if (lo > t2) continue;
            // ends are past the earlier ones: lo > t2' >= the times before b
            a = lower_bound(l1.p, b, l1.n, lo, p1, x);
            if (a == l1.n) break; // later intervals start no earlier
            b = lower_bound(l1.p, a, l1.n, t2 + 1, probe(l1.p, a, l1.n), x);
            if (a < b) {
                atomicAdd(&diff[l1s + a], 1);
                atomicAdd(&diff[l1s + b], -1);
                if (b == l1.n) break;
            }
        }
    }
};

// the smallest window per (e, w) into a histogram over sorted window levels:
// level j counts w whose smallest window lies in (lv[j-1], lv[j]]
struct PoolOp {
    const int64_t *lv;
    int nl, nls;
    int64_t dmax; // the last level
    uint32_t *hist;
    unsigned long long *tmask; // per tile of 64 edges: bit e & 63 set once a counter of edge e is non-zero
    __device__ inline int64_t most() const { return dmax; }
    __device__ inline void hit(int32_t e, int64_t win) const {
        const int32_t a = lower_bound_from(lv, 0, nl, win); // win <= dmax, the last level
        // two atomics that nothing waits for, rather than one that returns whether
        // the other is needed
        atomicAdd(&hist[hist_at(e, a, nls)], 1u);
        atomicOr(&tmask[e >> 6], 1ull << (e & 63));
    }
};

// ---------------------------------------------------------------------------
// a.5: triangle enumeration, one wavefront per item
// ---------------------------------------------------------------------------
// inclusive sum over the wavefront (every lane active): row shifts, then the
// rows' totals broadcast onward
__device__ inline int32_t wave_scan(int32_t x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false); // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false); // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false); // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false); // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false); // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false); // row_bcast:31
    return x;
}

constexpr uint32_t MODE_B = 0x80000000u;

// Hands the triangle of segment edge (u, v) = pm, probe position p and owner-row
// position pw to a sink as (edge (x0,x1), edge (x0,x2), edge (x1,x2)):
// mode A: p is in v's row, pw in u's;  mode B: p is in u's row, pw in v's.
__device__ inline void tri_edges(int32_t pm, int32_t p, int32_t pw, int32_t &e01, int32_t &e02, int32_t &e12) {
    e01 = (int32_t)((uint32_t)pm & ~MODE_B);
    if ((uint32_t)pm & MODE_B) {
        e02 = p;
        e12 = pw;
    } else {
        e02 = pw;
        e12 = p;
    }
}

// Sinks.  kRanges: the sink tests the edges' time ranges (see FilterSink); the
// others see every triangle.
// hit(h, e01, e02, e12) is called by all lanes of the wave together.
struct CountSink { // triangles per item
    static constexpr bool kRanges = false, kAll = true, kFirst = false, kHits = false;
    int32_t *tri_u;
    int32_t c;
    __device__ void begin(int64_t) { c = 0; }
    __device__ void hit(bool h, int32_t, int32_t, int32_t) { c += (int32_t)__popcll(__ballot(h)); }
    __device__ void end(int64_t u) {
        if (lane_id() == 0) tri_u[u] = c;
    }
    __device__ void finish() {}
};

struct CacheSink { // the triangles themselves, from their item's offset
    static constexpr bool kRanges = false, kAll = true, kFirst = false, kHits = false;
    const int64_t *base;
    int32_t *tri;
    int64_t slot;
    __device__ void begin(int64_t u) { slot = base[u]; }
    __device__ void hit(bool h, int32_t a, int32_t b, int32_t c) {
        unsigned long long mask = __ballot(h);
        if (h) {
            int64_t pos = slot + __popcll(mask & lanes_below());
            tri[3 * pos] = a;
            tri[3 * pos + 1] = b;
            tri[3 * pos + 2] = c;
        }
        slot += __popcll(mask);
    }
    __device__ void end(int64_t) {}
    __device__ void finish() {}
};

struct TcntSink { // triangles per static edge
    static constexpr bool kRanges = false, kAll = true, kFirst = false, kHits = false;
    const uint32_t *oeid;
    int32_t *tcnt;
    __device__ void begin(int64_t) {}
    __device__ void hit(bool h, int32_t a, int32_t b, int32_t c) {
        if (h) {
            atomicAdd(&tcnt[oeid[a] & 0x7fffffffu], 1);
            atomicAdd(&tcnt[oeid[b] & 0x7fffffffu], 1);
            atomicAdd(&tcnt[oeid[c] & 0x7fffffffu], 1);
        }
    }
    __device__ void end(int64_t) {}
    __device__ void finish() {}
};

// Slack of a range test on timestamps shifted right by `shift`: floors of two
// values differ by at most one unit more than their difference does.
__host__ __device__ inline int64_t range_slack(int64_t dmax, int32_t shift) {
    return shift ? (dmax >> shift) + 1 : dmax;
}

// The ranges of an oriented edge's two lists (Index::erng), tail to head in x and
// head to tail in y: per list one pair of 16-bit numbers (-first, last) in the
// low and high half, timestamps in units of 2^rshift from a base (RNG_BITS bits); an
// empty list is (-32768, -32768).  In this form the tests below are packed additions
// whose signs decide, and an empty list fails every one of them.
constexpr int RNG_BITS = 14;
constexpr uint32_t RNG_EMPTY = 0x80008000u;
// A record's timestamp x in those units.  Timestamps before the base or past the
// last unit count as the first or last one: that keeps their order and makes no two
// lie further apart, so what the tests drop has no window, wherever the base lies.
// Base and unit follow the span of most timestamps (10M edges in one day, times from
// 0 and from 1.3e9, a window of 60 s: 0.21 and 0.78 ms when the unit followed the
// largest timestamp, now 0.21 and 0.21).
__host__ __device__ inline uint32_t rng_code(uint32_t x, uint32_t base, int32_t shift) {
    const uint32_t c = (x > base ? x - base : 0u) >> shift, most = (1u << RNG_BITS) - 1;
    return c < most ? c : most;
}
typedef short rng_t __attribute__((ext_vector_type(2)));
__host__ __device__ inline uint32_t rng_pack(uint32_t first, uint32_t last) {
    return (uint32_t)(uint16_t)(-(int32_t)first) | last << 16;
}
// the window bound in units of the ranges (no difference of two exceeds it)
__host__ __device__ inline int32_t rng_slack(int64_t dmax, int32_t rshift) {
    const int64_t d = range_slack(dmax, rshift), most = (1 << RNG_BITS) - 1;
    return (int32_t)(d > most ? most : d);
}
__device__ inline rng_t rng_of(uint32_t w) { return __builtin_bit_cast(rng_t, w); }
__device__ inline uint32_t rng_word(rng_t r) { return __builtin_bit_cast(uint32_t, r); }
__device__ inline rng_t rng_sum(rng_t a, rng_t b) { return __builtin_elementwise_add_sat(a, b); }
__device__ inline uint32_t rng_swap(uint32_t w) { return __builtin_amdgcn_alignbit(w, w, 16); }
// top bit set unless both halves are >= 0
__device__ inline uint32_t rng_bad(rng_t d) {
    const uint32_t w = rng_word(d);
    return w | w << 16;
}
// (last + dq, dq - first) of a list: summed with another list's (-first, last)
// both halves are >= 0 iff the lists come within dq of each other
__device__ inline uint32_t rng_near(uint32_t w, int32_t dq) {
    return rng_word(rng_sum(rng_of(rng_swap(w)), rng_of((uint32_t)dq | (uint32_t)dq << 16)));
}

// An edge's lists for the run test: p = (-first, last), q = (last + dq, -first).
// q of one list plus p of another: both halves >= 0 iff an entry of the other can
// follow one of the first by at most dq.
struct RngEdge {
    rng_t p[2], q[2];
    __device__ RngEdge(uint32_t x, uint32_t y, int32_t dq) {
        p[0] = rng_of(x);
        p[1] = rng_of(y);
        const rng_t d = rng_of((uint32_t)dq); // the low half
        q[0] = rng_sum(rng_of(rng_swap(x)), d);
        q[1] = rng_sum(rng_of(rng_swap(y)), d);
    }
};
// list E_{xI,xJ} of a triangle with edges (x0,x1), (x0,x2), (x1,x2)
template <int I, int J> struct RngList {
    static constexpr int edge = I + J - 1, dir = I < J ? 0 : 1;
};
// top bit clear iff run (I, J) can have t <= t2 <= t3 <= t + dmax by its lists' ranges
template <int VAR, int I, int J> __device__ inline uint32_t rng_run_bad(const RngEdge (&E)[3]) {
    using P = Pick<VAR, I, J>;
    using A = RngList<I, J>;
    using B = RngList<P::L2a, P::L2b>;
    using C = RngList<P::L3a, P::L3b>;
    const rng_t q1 = E[A::edge].q[A::dir];
    return rng_bad(rng_of(rng_word(rng_sum(q1, E[B::edge].p[B::dir])) | rng_word(rng_sum(q1, E[C::edge].p[C::dir])) |
                          rng_word(rng_sum(E[B::edge].q[B::dir], E[C::edge].p[C::dir]))));
}
template <int VAR> __device__ inline uint32_t rng_tri_bad(const RngEdge (&E)[3]) {
    return rng_run_bad<VAR, 0, 1>(E) & rng_run_bad<VAR, 1, 0>(E) & rng_run_bad<VAR, 0, 2>(E) &
           rng_run_bad<VAR, 2, 0>(E) & rng_run_bad<VAR, 1, 2>(E) & rng_run_bad<VAR, 2, 1>(E);
}
// a run of any of the predicates (bits, the same in every lane)
__device__ inline bool rng_can_run(uint32_t predicates, const RngEdge (&E)[3]) {
    uint32_t bad = ~0u;
    while (predicates) {
        const int v = __builtin_ctz(predicates);
        predicates &= predicates - 1;
        switch (v) {
        case 0: bad &= rng_tri_bad<0>(E); break;
        case 1: bad &= rng_tri_bad<1>(E); break;
        case 2: bad &= rng_tri_bad<2>(E); break;
        case 3: bad &= rng_tri_bad<3>(E); break;
        case 4: bad &= rng_tri_bad<4>(E); break;
        case 5: bad &= rng_tri_bad<5>(E); break;
        case 6: bad &= rng_tri_bad<6>(E); break;
        default: bad &= rng_tri_bad<7>(E); break;
        }
    }
    return (int32_t)bad >= 0;
}

// The triangles a filter keeps, in chunks of 64 slots (three oriented edges
// each): a wavefront fills one chunk after another, taking chunk numbers from
// its block's region (regions have counters on cache lines of their own, so
// the atomics of thousands of wavefronts do not queue at one address) or, once
// that is full, from the next one, and leaves the number of slots it filled in
// cnt.  A wavefront that finds every region full drops what it keeps and counts
// the chunks it would have needed, so the host learns what a repeat needs.

struct CandAppend {
    int32_t cur = -1;     // this wavefront's chunk (-1: none)
    int32_t n = 64;       // slots filled in it
    int32_t region = -1;  // where its next chunk comes from
    uint32_t lost = 0;    // chunks dropped
    int32_t group = 0;    // tag of the chunks taken
    __device__ int32_t take(const CandBuf &B) {
        if (lost) {
            lost++;
            return -1;
        }
        if (region < 0) region = (int32_t)(blockIdx.x % (unsigned)B.regions);
        for (int32_t tries = 0; tries < B.regions; tries++) {
            uint32_t k = 0;
            if (lane_id() == 0) k = atomicAdd(&B.ctr[region * CAND_STRIDE], 1u);
            k = __builtin_amdgcn_readfirstlane(k);
            if (k < (uint32_t)B.per_region) {
                const int32_t chunk = region * B.per_region + (int32_t)k;
                if (B.tag && lane_id() == 0) B.tag[chunk] = group;
                return chunk;
            }
            region = region + 1 == B.regions ? 0 : region + 1;
        }
        lost = 1;
        return -1;
    }
    __device__ void close(const CandBuf &B) { // the chunk takes no more
        if (cur >= 0 && lane_id() == 0) B.cnt[cur] = n;
        cur = -1;
        n = 64;
    }
    __device__ void push(const CandBuf &B, bool keep, int32_t a, int32_t b, int32_t c) {
        const unsigned long long mask = __ballot(keep);
        if (!mask) return;
        const int32_t add = (int32_t)__popcll(mask);
        const int32_t pos = n + (int32_t)__popcll(mask & lanes_below());
        int32_t next = cur;
        if (n + add > 64) {
            if (cur >= 0 && lane_id() == 0) B.cnt[cur] = 64;
            next = take(B);
        }
        const int32_t chunk = pos < 64 ? cur : next;
        if (keep && chunk >= 0) {
            int32_t *s = B.sv + 3 * ((int64_t)chunk * 64 + (pos & 63));
            s[0] = a;
            s[1] = b;
            s[2] = c;
        }
        n = n + add > 64 ? n + add - 64 : n + add;
        cur = next;
    }
    __device__ void finish(const CandBuf &B) {
        close(B);
        if (lost && lane_id() == 0) atomicAdd(B.dropped, lost);
    }
};

// Keeps the triangles with a run of one of the predicates that can count by its
// lists' ranges (a run needs t <= t2 <= t3 <= t + dmax; the temporal step decides
// from the records, whose ranges are exact).
// A probe's two known edges can be tested first (do any of their lists come
// within dmax of each other?) and the whole triangle after, or the triangle once:
//   FILTER_NARROW  known edges, then the membership of those that pass, then the triangle;
//   FILTER_WIDE    membership of every probe, then the triangle;
//   FILTER_COUNT   membership of every probe, counting the triangles, then both tests.
// VAR >= 0: one predicate, fixed at compile time; VAR < 0: the bits of `predicates`
// (a plan's jobs), all eight tests inlined.
enum FilterMode { FILTER_NARROW, FILTER_WIDE, FILTER_COUNT };
template <int VAR, FilterMode MODE> struct FilterSink {
    static constexpr bool kRanges = true;
    static constexpr bool kAll = MODE != FILTER_NARROW; // every probe's membership is decided
    static constexpr bool kFirst = MODE != FILTER_WIDE; // the known edges are tested first
    static constexpr bool kHits = MODE == FILTER_COUNT;
    const uint2 *rng;
    int32_t dq;               // rng_slack(dmax, rshift)
    uint32_t predicates;      // VAR < 0: bits
    CandBuf out;
    unsigned long long *scal; // FILTER_COUNT: the query's scalars (triangles seen, added once per wavefront)
    CandAppend app;
    unsigned long long nhit;
    __device__ void begin(int64_t) {}
    __device__ void end(int64_t) {}
    // do some list of the probed edge and some list of edge (u, v), given as
    // rng_near words, come within dq of each other?
    __device__ bool first(uint32_t n0, uint32_t n1, uint2 rp) const {
        const rng_t px = rng_of(rp.x), py = rng_of(rp.y);
        return (int32_t)(rng_bad(rng_sum(rng_of(n0), px)) & rng_bad(rng_sum(rng_of(n0), py)) &
                         rng_bad(rng_sum(rng_of(n1), px)) & rng_bad(rng_sum(rng_of(n1), py))) >= 0;
    }
    // a triangle (h) whose known edges meet; pw: the owner-row edge
    __device__ void found(bool h, uint32_t n0, uint32_t n1, uint2 rp, int32_t pm, int32_t p, int32_t pw) {
        bool keep = false;
        int32_t a = 0, b = 0, c = 0;
        if (h) {
            const uint2 rw = rng[(uint32_t)pw];
            const bool mode_b = ((uint32_t)pm & MODE_B) != 0;
            const uint2 r1 = mode_b ? rp : rw, r2 = mode_b ? rw : rp;
            // (last + dq, dq - first) back to (-first, last); an empty list stays empty
            const rng_t d = rng_of((uint32_t)dq | (uint32_t)dq << 16);
            const uint32_t x = rng_swap(rng_word(__builtin_elementwise_sub_sat(rng_of(n0), d)));
            const uint32_t y = rng_swap(rng_word(__builtin_elementwise_sub_sat(rng_of(n1), d)));
            const RngEdge E[3] = {RngEdge(x, y, dq), RngEdge(r1.x, r1.y, dq), RngEdge(r2.x, r2.y, dq)};
            if constexpr (VAR >= 0) keep = (int32_t)rng_tri_bad<VAR>(E) >= 0;
            else keep = rng_can_run(predicates, E);
            tri_edges(pm, p, pw, a, b, c);
        }
        app.push(out, keep, a, b, c);
    }
    __device__ void finish() {
        app.finish(out);
        if constexpr (kHits) {
            if (lane_id() == 0 && nhit) region_add(scal, REGION_HITS, nhit);
        }
    }
};

// LDS of one wavefront's item.  Probe q in [0, nq) belongs to segment
// popcount(marks below q): marks has a bit at q - 1 for the first probe q of
// every segment but the first, so a step of 64 probes finds its segments with
// one uniform 64-bit read and a bit count per lane.
// The owner's out-row is a hash table of buckets of four entries (id << 10 |
// position, ids by their low 22 bits): one 16-byte read and the smallest of
// four differences decide a probe and give its position, unless the bucket is
// full (3 % of them at the highest load, two entries per bucket).
constexpr int ITEM_SEGS = 64;     // probe segments per item
constexpr int TAB_BUCKETS = 256;
constexpr int POS_BITS = 10;
constexpr int ENUM_UNROLL = 4;    // probe steps whose loads overlap
struct EnumLds {
    uint4 tab[TAB_BUCKETS];        // loose items: int2 (start, length) of each segment's owner row
    // per segment: x: row start minus the segment's first probe (probe q reads
    // oadj[x + q]); y: oriented edge (u, v) | mode B << 31; z, w: its ranges (rng_near)
    uint4 sg[ITEM_SEGS];
    unsigned long long marks[64];
    uint2 queue[128]; // probes for the next dense step: (q | segment << 16, owner-row edge or unused)
};
static_assert(CHUNK + CAP + 64 * ENUM_UNROLL <= 64 * 64, "marks cover an item's probes and the steps past them");
static_assert(CAP <= 2 * TAB_BUCKETS && CAP < (1 << POS_BITS), "table load and positions");

__device__ inline uint32_t tab_key(int32_t x) { return (uint32_t)x << POS_BITS; }
__device__ inline uint32_t tab_hash(int32_t x, int tlog) { return ((uint32_t)x * 0x9E3779B1u) >> (32 - tlog); }

// buckets for a row of d entries, as a power of two: at most two entries each on average
__device__ inline int tab_log(int32_t d) {
    const int l = 32 - __builtin_clz((uint32_t)(d > 4 ? d - 1 : 4)) - 1;
    return l < 4 ? 4 : l;
}

// the owner row [b, b + d) into the table; v0: this lane's entry of the first 64
__device__ inline void tab_build(EnumLds &L, const int32_t *__restrict__ oadj, int32_t b, int32_t d, int32_t v0,
                                 int tlog) {
    const int lane = lane_id();
    const uint4 none = make_uint4(~0u, ~0u, ~0u, ~0u);
    for (int i = lane; i < (1 << tlog); i += 64) L.tab[i] = none;
    wave_sync();
    uint32_t *slot = reinterpret_cast<uint32_t *>(L.tab);
    const uint32_t nslots = 4u << tlog;
    for (int32_t i = lane; i < d; i += 64) {
        const int32_t x = i < 64 ? v0 : oadj[b + i];
        const uint32_t val = tab_key(x) | (uint32_t)i;
        uint32_t at = tab_hash(x, tlog) * 4;
        // buckets fill from their first slot on; a full one passes to the next
        while (atomicCAS(&slot[at], ~0u, val) != ~0u) at = at + 1 == nslots ? 0 : at + 1;
    }
    wave_sync();
}

// position of x in the owner row, or -1.  exact: ids are below 2^22, so equal
// low bits are equal ids; otherwise the row's entry decides.
__device__ inline int32_t tab_find(const EnumLds &L, const int32_t *__restrict__ oadj, int32_t b, int32_t x, int tlog,
                                   bool exact) {
    const uint32_t key = tab_key(x);
    uint32_t h = tab_hash(x, tlog);
    for (;;) {
        const uint4 s = L.tab[h];
        const uint32_t d0 = s.x ^ key, d1 = s.y ^ key, d2 = s.z ^ key, d3 = s.w ^ key;
        if (exact) {
            const uint32_t m0 = d0 < d1 ? d0 : d1, m1 = d2 < d3 ? d2 : d3;
            const uint32_t m = m0 < m1 ? m0 : m1;
            if (m < (uint32_t)CAP) return (int32_t)m;
        } else {
            const uint32_t dd[4] = {d0, d1, d2, d3};
#pragma unroll
            for (int j = 0; j < 4; j++)
                if (dd[j] < (uint32_t)CAP && oadj[b + (int32_t)dd[j]] == x) return (int32_t)dd[j];
        }
        if (s.w == ~0u) return -1;
        h = (h + 1) & ((1u << tlog) - 1u);
    }
}

// position of x in the ascending row [b, b + d) of global memory, or -1
__device__ inline int32_t row_find(const int32_t *__restrict__ oadj, int32_t b, int32_t d, int32_t x) {
    int32_t a = 0, c = d;
    while (a < c) {
        const int32_t mid = (a + c) >> 1;
        if (oadj[b + mid] < x) a = mid + 1;
        else c = mid;
    }
    return a < d && oadj[b + a] == x ? a : -1;
}

struct EnumGraph {
    const EnumItem *item;
    const int32_t *oadj;
    const int4 *seg;
    const uint2 *srng;    // the ranges of each segment's edge
    const int32_t *owner; // of each segment (read for loose items)
    const int32_t *ooff;
    int32_t exact; // ids below 2^22 (tab_find)
};

// An item's first owner-row entries and its segments (this lane's), loaded one
// item ahead.
struct StageAhead {
    int32_t v;
    int4 sg;
    uint2 r;
};

template <bool RANGES>
__device__ inline StageAhead stage_ahead(const EnumItem &item, const EnumGraph &G) {
    StageAhead a{0, make_int4(0, 0, 0, 0), make_uint2(0, 0)};
    const int lane = lane_id();
    if (lane < item.ng) {
        a.sg = G.seg[item.g0 + lane];
        if constexpr (RANGES) a.r = G.srng[item.g0 + lane];
    }
    if (lane < item.d && item.d <= CAP) a.v = G.oadj[item.b + lane];
    return a;
}

// One wavefront per item, whose segments' rows are probed as one flat range q in
// [0, nq).  LOOSE: the segments belong to owners with few probes each, whose
// rows are searched in global memory instead of a table.
template <bool LOOSE, class Sink>
__device__ inline void enum_flat(const EnumItem &item, const StageAhead &ahead, const EnumGraph &G, Sink &sink,
                                 EnumLds &L) {
    const int lane = lane_id();
    const int32_t *__restrict__ oadj = G.oadj;
    const int32_t nq = item.nq, b = item.b, d = item.d;
    const int4 sg = ahead.sg; // zero length past the item's segments
    const int32_t start = wave_scan(sg.y) - sg.y;
    const bool have = lane < item.ng;
    L.marks[lane] = 0;
    if (have) {
        uint4 e = make_uint4((uint32_t)(sg.x - start), (uint32_t)sg.z, 0, 0);
        if constexpr (Sink::kRanges) {
            e.z = rng_near(ahead.r.x, sink.dq);
            e.w = rng_near(ahead.r.y, sink.dq);
        }
        L.sg[lane] = e;
        if constexpr (LOOSE) {
            const int32_t w = G.owner[item.g0 + lane], ob = G.ooff[w];
            reinterpret_cast<int2 *>(L.tab)[lane] = make_int2(ob, G.ooff[w + 1] - ob);
        }
    }
    const int tlog = LOOSE ? 0 : tab_log(d);
    bool built = LOOSE;
    if constexpr (!LOOSE && Sink::kAll) {
        tab_build(L, oadj, b, d, ahead.v, tlog);
        built = true;
    } else {
        wave_sync();
    }
    if (have && lane > 0) atomicOr(&L.marks[(start - 1) >> 6], 1ull << ((start - 1) & 63));
    wave_sync();
    auto find = [&](uint32_t i, int32_t x, int32_t &pw) {
        int32_t at;
        if constexpr (LOOSE) {
            const int2 o = reinterpret_cast<const int2 *>(L.tab)[i];
            at = row_find(oadj, o.x, o.y, x);
            pw = o.x + at;
        } else {
            at = tab_find(L, oadj, b, x, tlog, G.exact != 0);
            pw = b + at;
        }
        return at >= 0;
    };
    // Probes that pass a step's test are a part of its lanes, often a small one, and
    // what follows costs as much for one lane as for 64: they queue in LDS until 64
    // have come together (or the item ends).  FILTER_NARROW queues the probes whose
    // known edges meet, the others the triangles that are left to test.  70M edges,
    // without and with the queue: 1 hour 1.28 and 1.31 ms, 1 day 1.51 and 1.39, 1 week
    // 2.26 and 1.52, 4 weeks 3.26 and 1.78; 1 year in one pass 4.32 and 3.95.
    int32_t qhead = 0, qlen = 0;
    auto drain = [&](int32_t n) {
        wave_sync();
        const bool on = lane < n;
        const uint2 c = L.queue[(qhead + lane) & 127];
        qhead += n;
        qlen -= n;
        const uint32_t i = on ? c.x >> 16 : 0u;
        const uint4 e = L.sg[i];
        const uint32_t p = e.x + (c.x & 0xffffu);
        if constexpr (Sink::kRanges) {
            const uint2 rp = on ? sink.rng[p] : make_uint2(RNG_EMPTY, RNG_EMPTY);
            bool h = on;
            int32_t pw = (int32_t)c.y;
            if constexpr (!Sink::kAll) {
                const int32_t x = on ? oadj[p] : -1;
                if (!built) {
                    tab_build(L, oadj, b, d, ahead.v, tlog);
                    built = true;
                }
                if (on) h = find(i, x, pw);
            }
            if (__ballot(h)) sink.found(h, e.z, e.w, rp, (int32_t)e.y, (int32_t)p, pw);
        }
        wave_sync(); // the entries' places are written again
    };
    auto enqueue = [&](bool on, uint32_t i, int32_t q, int32_t pw) {
        const unsigned long long mask = __ballot(on);
        if (!mask) return;
        if (on) L.queue[(qhead + qlen + (int32_t)__popcll(mask & lanes_below())) & 127] =
                    make_uint2((uint32_t)q | i << 16, (uint32_t)pw);
        qlen += (int32_t)__popcll(mask);
        if (qlen >= 64) drain(64);
    };
    int32_t seg0 = 0; // segment of the next step's first probe
    for (int32_t q0 = 0; q0 < nq; q0 += 64 * ENUM_UNROLL) {
        uint4 ek[ENUM_UNROLL];
        uint32_t ik[ENUM_UNROLL], pk[ENUM_UNROLL];
        int32_t xk[ENUM_UNROLL];
        uint2 rk[ENUM_UNROLL];
        bool vk[ENUM_UNROLL];
#pragma unroll
        for (int k = 0; k < ENUM_UNROLL; k++) {
            const int32_t q = q0 + 64 * k + lane;
            const unsigned long long w = L.marks[(q0 >> 6) + k];
            const uint32_t w0 = __builtin_amdgcn_readfirstlane((uint32_t)w);
            const uint32_t w1 = __builtin_amdgcn_readfirstlane((uint32_t)(w >> 32));
            ik[k] = __builtin_amdgcn_mbcnt_hi(w1, __builtin_amdgcn_mbcnt_lo(w0, (uint32_t)seg0));
            ek[k] = L.sg[ik[k]];
            seg0 += __builtin_popcount(w0) + __builtin_popcount(w1);
            vk[k] = q < nq;
            pk[k] = ek[k].x + (uint32_t)q;
        }
        if constexpr (Sink::kAll) {
#pragma unroll
            for (int k = 0; k < ENUM_UNROLL; k++) xk[k] = vk[k] ? oadj[pk[k]] : -1;
        }
        if constexpr (Sink::kFirst) {
#pragma unroll
            for (int k = 0; k < ENUM_UNROLL; k++) rk[k] = vk[k] ? sink.rng[pk[k]] : make_uint2(RNG_EMPTY, RNG_EMPTY);
        }
#pragma unroll
        for (int k = 0; k < ENUM_UNROLL; k++) {
            const int32_t q = q0 + 64 * k + lane;
            if constexpr (!Sink::kAll) {
                // false past the item's probes
                enqueue(sink.first(ek[k].z, ek[k].w, rk[k]), ik[k], q, 0);
            } else {
                if (q0 + 64 * k >= nq) continue;
                bool h = false;
                int32_t pw = 0;
                if (vk[k]) h = find(ik[k], xk[k], pw);
                if constexpr (!Sink::kRanges) {
                    int32_t e01 = 0, e02 = 0, e12 = 0;
                    if (h) tri_edges((int32_t)ek[k].y, (int32_t)pk[k], pw, e01, e02, e12);
                    sink.hit(h, e01, e02, e12);
                } else {
                    if constexpr (Sink::kHits) sink.nhit += (unsigned long long)__popcll(__ballot(h));
                    if constexpr (Sink::kFirst) h = h && sink.first(ek[k].z, ek[k].w, rk[k]);
                    enqueue(h, ik[k], q, pw);
                }
            }
        }
    }
    if (qlen > 0) drain(qlen);
    wave_sync(); // the next item overwrites this wave's LDS
}

// long owner rows (only in orientations without the degeneracy bound): each
// segment in turn, searched in the owner's row in global memory
template <class Sink>
__device__ inline void enum_long(const EnumItem &item, const EnumGraph &G, Sink &sink) {
    const int lane = lane_id();
    for (int32_t g = item.g0; g < item.g0 + item.ng; g++) {
        const int4 sg = G.seg[g];
        uint32_t n0 = 0, n1 = 0;
        if constexpr (Sink::kRanges) {
            const uint2 r = G.srng[g];
            n0 = rng_near(r.x, sink.dq);
            n1 = rng_near(r.y, sink.dq);
        }
        for (int32_t p0 = sg.x; p0 < sg.x + sg.y; p0 += 64) {
            const int32_t p = p0 + lane;
            bool h = p < sg.x + sg.y;
            uint2 rp = make_uint2(RNG_EMPTY, RNG_EMPTY);
            if constexpr (Sink::kRanges) {
                if (h) rp = sink.rng[p];
                if constexpr (!Sink::kAll) h = h && sink.first(n0, n1, rp);
            }
            int32_t at = -1;
            if (h) at = row_find(G.oadj, item.b, item.d, G.oadj[p]);
            h = at >= 0;
            if constexpr (!Sink::kRanges) {
                int32_t e01 = 0, e02 = 0, e12 = 0;
                if (h) tri_edges(sg.z, p, item.b + at, e01, e02, e12);
                sink.hit(h, e01, e02, e12);
            } else {
                if constexpr (Sink::kHits) sink.nhit += (unsigned long long)__popcll(__ballot(h));
                if constexpr (Sink::kAll && Sink::kFirst) h = h && sink.first(n0, n1, rp);
                if (__ballot(h)) sink.found(h, n0, n1, rp, sg.z, p, item.b + at);
            }
        }
    }
}

template <class Sink>
__device__ inline void enum_item(const EnumItem &item, const StageAhead &ahead, const EnumGraph &G, int64_t it,
                                 Sink &sink, EnumLds &L) {
    sink.begin(it);
    if (item.d < 0) enum_flat<true>(item, ahead, G, sink, L);
    else if (item.d <= CAP) enum_flat<false>(item, ahead, G, sink, L);
    else enum_long(item, G, sink);
    sink.end(it);
}

// (A queue of items or batches of items, handed to a chip's worth of wavefronts
// by one counter, was slower: atomics on one address take 11 ns each here, 0.54
// against 0.10 ms for 45,000 items.  Many blocks let the dispatcher balance.)
template <class Sink>
__global__ __launch_bounds__(BLK) __attribute__((amdgpu_waves_per_eu(4))) void k_tri_enum(EnumGraph G, int32_t NI,
                                                                                          Sink sink) {
    __shared__ EnumLds lds[WPB];
    const int w = wave_id();
    const int64_t stride = (int64_t)gridDim.x * WPB;
    int64_t it = (int64_t)blockIdx.x * WPB + w;
    // item headers run two items ahead and the first row and segment entries
    // one item ahead, so a wavefront starts each item with its data loaded
    const EnumItem none{};
    EnumItem h0 = it < NI ? G.item[it] : none;
    EnumItem h1 = it + stride < NI ? G.item[it + stride] : none;
    StageAhead a0 = stage_ahead<Sink::kRanges>(h0, G);
    for (; it < NI; it += stride) {
        const EnumItem cur = h0;
        const StageAhead ca = a0;
        h0 = h1;
        a0 = stage_ahead<Sink::kRanges>(h0, G);
        h1 = it + 2 * stride < NI ? G.item[it + 2 * stride] : none;
        enum_item(cur, ca, G, it, sink, lds[w]);
    }
    sink.finish();
}

// the filter over a cached triangle list, 64 triangles to a wavefront
template <class Sink>
__device__ inline void cached_triangles(const int32_t *__restrict__ tri, int64_t T, int64_t first, int64_t step,
                                        Sink &sink) {
    for (int64_t t0 = first * 64; t0 < T; t0 += step * 64) {
        const int64_t t = t0 + lane_id();
        bool h = t < T;
        int32_t a = 0, b = 0, c = 0;
        uint32_t n0 = 0, n1 = 0;
        uint2 rp = make_uint2(RNG_EMPTY, RNG_EMPTY);
        if (h) {
            a = tri[3 * t];
            b = tri[3 * t + 1];
            c = tri[3 * t + 2];
            const uint2 r = sink.rng[a];
            n0 = rng_near(r.x, sink.dq);
            n1 = rng_near(r.y, sink.dq);
            rp = sink.rng[c];
            h = sink.first(n0, n1, rp);
        }
        if (__ballot(h)) sink.found(h, n0, n1, rp, a, c, b); // as mode A: c probed, b in the owner's row
    }
}

template <class Sink>
__global__ __launch_bounds__(BLK) void k_filter_cached(const int32_t *__restrict__ tri, int64_t T, Sink sink) {
    cached_triangles(tri, T, (int64_t)blockIdx.x * WPB + wave_id(), (int64_t)gridDim.x * WPB, sink);
    sink.finish();
}

// ---------------------------------------------------------------------------
// a.6: scheduling the tests of the triangles the filter kept
// ---------------------------------------------------------------------------
// A wavefront takes a group of the filter's chunks, a triangle per lane, reads
// their records and finds the runs that can count and their tests.  The lanes
// stage their triangles' runs in LDS, and the work of triangles with at most
// LIGHT_TESTS tests, concatenated, is spread over the lanes: each finds its
// triangle by a search over 64 prefix sums and its run by the triangle's bits,
// and all lanes run one copy of the test whatever their run or predicate.
// (A copy per run, six in turn with part of the lanes each, took 2.2 ms where
// this takes 1.6 ms: 36.6M tests of the 70M-edge graph at one year.)  The
// per-edge counts take two tests per lane at a time (their first reads go together:
// 686,000 tests of 10M uniform edges 0.127 -> 0.079 ms), so neighbouring lanes take
// neighbouring tests of one run and their loads coalesce; the exists-exists-exists
// counting, whose window bookkeeping the tests of a run share, takes a few of them
// per lane.
// A triangle with more tests (a heavy one) gets an entry in a list and a range of
// piece numbers, both from one packed counter, so entries are in the order of
// their pieces; a second kernel runs piece p (tests [4 i, 4 i + 4) of its
// triangle) per thread, finding its entry by binary search over the entries'
// first pieces (the merge-path split of a long run over neighbouring threads).
// Heavy triangles past the list's capacity run where they were found, so any
// capacity gives the same result.
// Both kernels wait on dependent reads, so registers and LDS are kept small
// enough for four to eight wavefronts per SIMD.
// 70M-edge graph, one year (14.1M triangles, 36.6M tests) and a graph of
// 5,000-edge lists closed by short ones (2.9M triangles, 106M tests), both kernels:
// light limit 32 / 64 / 128 with pieces of 4: 1.60, 1.58, 1.56 and 1.12, 1.10, 1.11 ms;
// limit 64 with pieces of 2 / 8: 1.53, 1.67 and 1.19, 1.68 ms.
constexpr int64_t LIGHT_TESTS = 64;
constexpr int64_t PIECE_TESTS = 4;

struct Heavy {
    int64_t slot;  // slot in the filter's output
    int64_t first; // its first piece number
};
// the counter of heavy triangles: entries in bits 40-63, piece numbers in 0-39
constexpr int HEAVY_SHIFT = 40;
constexpr unsigned long long PIECE_MASK = (1ull << HEAVY_SHIFT) - 1;

// The filter's chunks as one sequence (a block's copy in LDS).
struct Chunks {
    int32_t start[MAX_REGIONS + 1]; // chunks of the regions before each, and of all
    int32_t total;
    // every thread of the block calls this
    __device__ void load(const CandBuf &B) {
        if (threadIdx.x < 64) {
            const int lane = lane_id();
            int32_t k = 0;
            if (lane < B.regions) {
                const uint32_t c = B.ctr[lane * CAND_STRIDE];
                k = c < (uint32_t)B.per_region ? (int32_t)c : B.per_region;
            }
            const int32_t incl = wave_scan(k);
            if (lane < MAX_REGIONS) start[lane + 1] = incl;
            if (lane == 0) start[0] = 0;
            if (lane == 63) total = incl;
        }
        __syncthreads();
    }
    // chunk g of the sequence, g < total
    __device__ int32_t at(const CandBuf &B, int32_t g) const {
        int r = 0; // the last region that starts at or before g (later empty ones start past it)
#pragma unroll
        for (int o = MAX_REGIONS / 2; o > 0; o >>= 1)
            if (start[r + o] <= g) r += o;
        return r * B.per_region + g - start[r];
    }
};

// The exact form of the filter's test on two edges: all lists' timestamps of each
// pair of edges come within dmax (in the records' units).
__device__ inline bool edges_meet(const TriLists &T, uint32_t dq) {
    auto lo = [](const Span &f, const Span &b) { return !f.n ? b.lo : !b.n || f.lo < b.lo ? f.lo : b.lo; };
    auto hi = [](const Span &f, const Span &b) { return !f.n ? b.hi : !b.n || f.hi > b.hi ? f.hi : b.hi; };
    const uint32_t l0 = lo(T.d01, T.d10), h0 = hi(T.d01, T.d10), l1 = lo(T.d02, T.d20), h1 = hi(T.d02, T.d20),
                   l2 = lo(T.d12, T.d21), h2 = hi(T.d12, T.d21);
    auto meet = [dq](uint32_t xl, uint32_t xh, uint32_t yl, uint32_t yh) {
        return (xl <= yh || xl - yh <= dq) && (yl <= xh || yl - xh <= dq);
    };
    return meet(l0, h0, l1, h1) && meet(l0, h0, l2, h2) && meet(l1, h1, l2, h2);
}

// list index of E_{x_a, x_b} in TriLists order (d01, d10, d02, d20, d12, d21)
constexpr int list_id(int a, int b) { return a == 0 ? (b == 1 ? 0 : 2) : a == 1 ? (b == 0 ? 1 : 4) : (b == 0 ? 3 : 5); }

// A wavefront's triangles in LDS: start and length of each directed list, the
// runs that can count (bit k: run k in the order of tri_live), and the inclusive
// prefix of the triangles' work.  SHORT: also the edges, for tests that read
// short lists from their records (see List).  SLOT: also their slots.
template <bool SHORT, bool SLOT = false> struct RunLds {
    int32_t incl[64];
    uint32_t live[64];
    int32_t n[6][64];
    int32_t s[6][64];
    int32_t e[SHORT ? 3 : 1][64];
    int64_t slot[SLOT ? 64 : 1];
};
template <bool SHORT, bool SLOT>
__device__ inline void stage_runs(RunLds<SHORT, SLOT> &F, int lane, const TriLists &T, const int32_t (&e)[3],
                                  uint32_t live, int64_t slot) {
    const Span *sp[6] = {&T.d01, &T.d10, &T.d02, &T.d20, &T.d12, &T.d21};
#pragma unroll
    for (int k = 0; k < 6; k++) {
        F.s[k][lane] = sp[k]->s;
        F.n[k][lane] = sp[k]->n;
    }
    if constexpr (SHORT)
        for (int k = 0; k < 3; k++) F.e[k][lane] = e[k];
    if constexpr (SLOT) F.slot[lane] = slot;
    F.live[lane] = live;
}

// The three lists of run k (order of tri_live's bits) under a predicate code, as
// indices in list_id's order: run k's own list is number k; the others sit three
// bits each in two words, the same for every lane.
struct RunLists {
    uint32_t l2, l3;
};
__host__ __device__ constexpr RunLists run_list_ids(int variant) {
    // for run (I, J) with third vertex C: the lists I -> C, C -> I, J -> C, C -> J
    constexpr int RI[6] = {0, 1, 0, 2, 1, 2}, RJ[6] = {1, 0, 2, 0, 2, 1};
    uint32_t ic = 0, ci = 0, jc = 0, cj = 0;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const int C = 3 - RI[k] - RJ[k];
        ic |= (uint32_t)list_id(RI[k], C) << (3 * k);
        ci |= (uint32_t)list_id(C, RI[k]) << (3 * k);
        jc |= (uint32_t)list_id(RJ[k], C) << (3 * k);
        cj |= (uint32_t)list_id(C, RJ[k]) << (3 * k);
    }
    const bool swap = (variant & 4) != 0; // L2 hangs off J, L3 off I
    const uint32_t x = (variant & 1) ? (swap ? cj : ci) : (swap ? jc : ic);
    const uint32_t y = (variant & 2) ? (swap ? ci : cj) : (swap ? ic : jc);
    return RunLists{x, y};
}

// list `id` of staged triangle si; rec: the edges' records when its end
// timestamps are exact, else null
template <bool SHORT>
__device__ inline List staged_list(const RunLds<SHORT> &F, int id, int si, const int64_t *__restrict__ ts,
                                   const EdgeRec *__restrict__ rec) {
    List l{ts + F.s[id][si], F.n[id][si], nullptr};
    if constexpr (SHORT)
        if (rec && l.n <= 2) l.ends = reinterpret_cast<const int64_t *>(rec + F.e[id >> 1][si]) + 2 + (id & 1);
    return l;
}

// Tests [r, r + cnt) of staged triangle si's runs in order (ONE: cnt = 1, and
// r is below their number).  SS: a run whose L2 is shorter than L1 has |L2|
// tests, the entries of L2, and is evaluated from them.
template <bool SS, bool ONE, class Op, bool SHORT>
__device__ inline void staged_tests(const RunLds<SHORT> &F, const RunLists &ids, int si, int64_t r, int32_t cnt,
                                    const int64_t *__restrict__ ts, const EdgeRec *__restrict__ rec, const Op &op) {
    uint32_t live = F.live[si];
    while (live) {
        const int k = __ffs((int)live) - 1;
        live &= live - 1;
        const int i2 = (int)(ids.l2 >> (3 * k)) & 7, i3 = (int)(ids.l3 >> (3 * k)) & 7;
        const int32_t n1 = F.n[k][si];
        const int32_t nt = SS && F.n[i2][si] < n1 ? F.n[i2][si] : n1;
        if (r >= nt) {
            r -= nt;
            continue;
        }
        const int32_t l1s = F.s[k][si];
        const List l2 = staged_list(F, i2, si, ts, rec), l3 = staged_list(F, i3, si, ts, rec);
        const int32_t first = (int32_t)r, m = ONE || cnt < nt - first ? (ONE ? 1 : cnt) : nt - first;
        bool done = false;
        if constexpr (SS) {
            if (nt < n1) {
                op.iv(List{ts + l1s, n1, nullptr}, l1s, first, m, l2, l3);
                done = true;
            }
        }
        if (!done) {
            int32_t c2 = 0, c3 = 0;
            for (int32_t q = 0; q < m; q++) {
                const int32_t e = l1s + first + q;
                const Probe p2 = l2.template at<SHORT>(c2), p3 = l3.template at<SHORT>(c3);
                int64_t win = 0;
                const TestEnd x = window_test(l2, l3, c2, c3, p2, p3, ts[e], op.most(), win);
                if (x == TEST_HIT) op.hit(e, win);
                if (x == TEST_END) break;
            }
        }
        cnt -= m;
        if (ONE || cnt == 0) return;
        r = 0;
    }
}

// One test, r of staged triangle si's runs, in two steps: its reads that depend on
// nothing else are issued when it is set up, so two tests' go together.
template <bool SHORT> struct OneTest {
    List l2, l3;
    Probe p2, p3;
    int64_t t;
    int32_t e;
    __device__ inline OneTest(const RunLds<SHORT> &F, const RunLists &ids, int si, int64_t r,
                              const int64_t *__restrict__ ts, const EdgeRec *__restrict__ rec) {
        int k = 0;
        for (uint32_t live = F.live[si];;) {
            k = __ffs((int)live) - 1;
            live &= live - 1;
            if (r < F.n[k][si] || !live) break;
            r -= F.n[k][si];
        }
        e = F.s[k][si] + (int32_t)r;
        l2 = staged_list(F, (int)(ids.l2 >> (3 * k)) & 7, si, ts, rec);
        l3 = staged_list(F, (int)(ids.l3 >> (3 * k)) & 7, si, ts, rec);
        p2 = l2.template at<SHORT>(0);
        p3 = l3.template at<SHORT>(0);
        t = ts[e];
    }
    template <class Op> __device__ inline void run(const Op &op) const {
        int32_t c2 = 0, c3 = 0;
        int64_t win = 0;
        if (window_test(l2, l3, c2, c3, p2, p3, t, op.most(), win) == TEST_HIT) op.hit(e, win);
    }
};

// Runs the tests of the per-edge counts (see k_tests_light): units() is a light
// triangle's work items, flat() runs one of them, piece() tests [r, r + cnt).
template <int VAR, class Op, bool SS> struct CountRunner {
    static constexpr bool kShort = !SS;
    using Lds = RunLds<kShort>;
    uint32_t dq;
    const int64_t *ts;
    Op op;
    const int32_t *sv; // the triangles as three oriented edges
    const EdgeRec *rec;
    bool inl; // timestamps are below 2^32, so the records' are exact
    __device__ inline uint32_t live(const TriLists &L) const { return tri_live<VAR>(L, dq); }
    __device__ inline int64_t work(const TriLists &L) const { return tri_work<VAR, SS>(L, dq); }
    __device__ inline int64_t units(const Lds &, int, int64_t tests) const { return tests; }
    __device__ inline const EdgeRec *ends() const { return inl ? rec : nullptr; }
    __device__ inline void flat(Lds &F, int si, int64_t r, bool on) {
        if (on) staged_tests<SS, true>(F, run_list_ids(VAR), si, r, 1, ts, ends(), op);
    }
    // items of two triangles; the second may be off
    static constexpr bool kTwo = !SS;
    __device__ inline void flat2(Lds &F, int s0, int64_t r0, int s1, int64_t r1, bool two) {
        const OneTest<kShort> a(F, run_list_ids(VAR), s0, r0, ts, ends());
        const OneTest<kShort> b(F, run_list_ids(VAR), two ? s1 : s0, two ? r1 : r0, ts, ends());
        a.run(op);
        if (two) b.run(op);
    }
    __device__ inline void piece(Lds &F, int si, int64_t r, int32_t cnt, bool on) {
        if (on) staged_tests<SS, false>(F, run_list_ids(VAR), si, r, cnt, ts, ends(), op);
    }
    __device__ inline void finish() {}
};

// Lanes with np > 0 (heavy triangles, np pieces each) take list entries and
// piece numbers for the whole wavefront with one atomic; returns which of them
// are listed.  The piece numbers that one past cap reserved follow every listed
// one.  `full` is set once this wavefront's atomic returned an entry count of cap
// or more, after which it lists nothing: each wavefront adds at most 64 entries
// past cap, so the entry count stays below cap + 64 x (the grid's wavefronts),
// below 2^24 (the static assertion at MOST_TEST_BLOCKS).
__device__ inline bool defer_heavy(int64_t slot, int64_t np, Heavy *__restrict__ heavy,
                                   unsigned long long *__restrict__ counter, int64_t cap, bool &full) {
    if (full || !__ballot(np > 0)) return false;
    const unsigned long long add = np > 0 ? (1ull << HEAVY_SHIFT) | (unsigned long long)np : 0ull;
    const unsigned long long incl = wave_inclusive_sum(add);
    unsigned long long at = 0;
    if (lane_id() == 63) at = atomicAdd(counter, incl);
    at = __shfl(at, 63);
    full = (int64_t)(at >> HEAVY_SHIFT) + 64 >= cap;
    if (np == 0) return false;
    const unsigned long long mine = at + incl - add;
    const int64_t e = (int64_t)(mine >> HEAVY_SHIFT);
    if (e >= cap) return false;
    heavy[e] = Heavy{slot, (int64_t)(mine & PIECE_MASK)};
    return true;
}

// the first of 64 ascending prefix sums that is above x (63 if none)
__device__ inline int staged_owner(const int32_t *incl, int32_t x) {
    int a = 0, b = 63;
    while (a < b) {
        const int mid = (a + b) >> 1;
        if (incl[mid] > x) b = mid;
        else a = mid + 1;
    }
    return a;
}

// The staged triangles' work over the lanes: flat(si, r, on) is item r of triangle
// si (called by all lanes together, with on false past the last item), this lane's
// triangle has `units` items (at most LIGHT_TESTS); triangles with `own` set (heavy,
// not listed) have alone(si) items each and go one after another.  TWO: a lane takes
// two items at a time, flat2(si, r, si', r', whether there is a second).
template <bool TWO, class Lds, class Flat, class Flat2, class Alone>
__device__ inline void spread_units(Lds &F, int32_t incl, bool own, const Flat &flat, const Flat2 &flat2,
                                    const Alone &alone) {
    const int lane = lane_id();
    int64_t total = __builtin_amdgcn_readlane(incl, 63);
    unsigned long long left = __ballot(own);
    int src = -1;
    auto item = [&](int64_t t, int &si, int64_t &r) {
        si = src;
        r = t;
        if (src < 0) { // the triangle whose items hold t
            si = staged_owner(F.incl, (int32_t)t);
            r = t - (si ? F.incl[si - 1] : 0);
        }
    };
    for (;;) {
        if constexpr (TWO) {
            for (int64_t t = lane; t < total; t += 128) {
                int s0, s1;
                int64_t r0, r1;
                item(t, s0, r0);
                item(t + 64, s1, r1);
                flat2(s0, r0, s1, r1, t + 64 < total);
            }
        } else {
            for (int64_t t0 = 0; t0 < total; t0 += 64) {
                int si;
                int64_t r;
                item(t0 + lane, si, r);
                flat(si, r, t0 + lane < total);
            }
        }
        if (!left) break;
        src = __builtin_ctzll(left);
        left &= left - 1;
        total = alone(src);
    }
}

// A wavefront's group of chunks as a dense sequence of slots: narrow windows
// leave most chunks with an entry or two, and their triangles are taken 64 at a
// time across chunks.  Groups of up to 64 chunks, fewer when that would leave
// less than GROUPS_WANTED groups (8,192 and 4,096 of them: 1.69 and 1.94 ms against
// 1.58 on the 70M-edge graph at one year, 0.079 and 0.097 against 0.079 for 10M uniform
// edges, but 0.061 and 0.056 against 0.084 for 10M renewal edges at 4 weeks); with few
// chunks each is shared by two or eight wavefronts, since a wavefront's tests are a
// chain of dependent reads.  Temporal step with one / two / four / eight wavefronts
// per chunk, us: 165 triangles in 164 chunks 14.8 / 13.6 / 13.3 / 13.4; 1,002 in 828
// 18.7 / 18.9 / 22.5 / 28.9; 17,400 in 2,050 38.7 / 30.1 / 32.9 / 46.3; 38,600 in
// 4,640 40.4 / 41.2 / 49.7 / 76.2; 17,800 in 5,120 36.3 / 44.2 / 59.6 / 87.8.
constexpr int32_t GROUPS_WANTED = 16384;
__device__ inline int32_t group_chunks(int32_t total) {
    const int32_t k = total / GROUPS_WANTED;
    return k < 1 ? 1 : k > 64 ? 64 : k;
}
__device__ inline int32_t chunk_parts(int32_t total) {
    return total >= GROUPS_WANTED / 4 ? 1 : total >= GROUPS_WANTED / 32 ? 2 : 8;
}
struct GroupLds {
    int32_t incl[64];  // slots of the group's chunks up to this one
    int32_t chunk[64];
};
// chunks [g0, g1) of the sequence into the LDS; returns their slots
__device__ inline int32_t stage_group(const CandBuf &B, const Chunks &C, int32_t g0, int32_t g1, GroupLds &L) {
    const int lane = lane_id();
    int32_t n = 0;
    if (lane < g1 - g0) {
        const int32_t chunk = C.at(B, g0 + lane);
        L.chunk[lane] = chunk;
        n = B.cnt[chunk];
    }
    const int32_t incl = wave_scan(n);
    L.incl[lane] = incl;
    wave_sync();
    return __builtin_amdgcn_readlane(incl, 63);
}
// slot number q of a staged group
__device__ inline int64_t group_slot(const GroupLds &L, int32_t q) {
    int a = 0, b = 63;
    while (a < b) {
        const int mid = (a + b) >> 1;
        if (L.incl[mid] > q) b = mid;
        else a = mid + 1;
    }
    return (int64_t)L.chunk[a] * 64 + (q - (a ? L.incl[a - 1] : 0));
}

// The regions' tests and kept triangles receive those of the chunks (one atomic each per block).
template <class R>
__global__ __launch_bounds__(BLK) void k_tests_light(CandBuf B, R runner, Heavy *__restrict__ heavy,
                                                     unsigned long long *__restrict__ counter, int64_t cap,
                                                     unsigned long long *__restrict__ scal) {
    __shared__ typename R::Lds flds[WPB];
    __shared__ GroupLds glds[WPB];
    __shared__ Chunks C;
    const int w = wave_id();
    const int lane = lane_id();
    typename R::Lds &F = flds[w];
    C.load(B);
    const int32_t per = group_chunks(C.total), parts = chunk_parts(C.total); // one of them is 1
    bool full = false;
    int64_t mine = 0;
    int32_t kept = 0;
    const int64_t units = (int64_t)C.total * parts;
    for (int64_t x = ((int64_t)blockIdx.x * WPB + w) * per; x < units; x += (int64_t)gridDim.x * WPB * per) {
        const int32_t g0 = (int32_t)(x / parts), part = (int32_t)(x % parts), wide = 64 / parts;
        const int32_t all = stage_group(B, C, g0, g0 + per < C.total ? g0 + per : C.total, glds[w]);
        // this wavefront's slots: the group's, or a part of its one chunk's
        const int32_t slots = parts == 1 || all < (part + 1) * wide ? all : (part + 1) * wide;
        if (part == 0) kept += all;
        for (int32_t q0 = part * wide; q0 < slots; q0 += 64) {
            int64_t slot = 0, wk = 0, np = 0;
            int32_t e[3] = {0, 0, 0};
            TriLists T{};
            uint32_t live = 0;
            if (q0 + lane < slots) {
                slot = group_slot(glds[w], q0 + lane);
                for (int k = 0; k < 3; k++) e[k] = runner.sv[3 * slot + k];
                T = load_lists(runner.rec, e[0], e[1], e[2]);
                if (edges_meet(T, runner.dq)) {
                    live = runner.live(T);
                    wk = runner.work(T);
                }
            }
            if (wk > LIGHT_TESTS) np = (wk + PIECE_TESTS - 1) / PIECE_TESTS;
            mine += wk;
            const bool listed = defer_heavy(slot, np, heavy, counter, cap, full);
            stage_runs(F, lane, T, e, live, slot);
            const int32_t incl = wave_scan(np ? 0 : (int32_t)runner.units(F, lane, wk));
            F.incl[lane] = incl;
            wave_sync();
            spread_units<R::kTwo>(
                F, incl, np && !listed,
                [&](int si, int64_t r, bool on) { runner.flat(F, si, r, on); },
                [&](int s0, int64_t r0, int s1, int64_t r1, bool two) {
                    if constexpr (R::kTwo) runner.flat2(F, s0, r0, s1, r1, two);
                },
                [&](int si) { return runner.units(F, si, __shfl(wk, si)); }); // si: the same in every lane
            wave_sync(); // the LDS is rewritten by the next triangles
        }
        wave_sync(); // the group's LDS is rewritten by the next group
    }
    runner.finish();
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
    __shared__ unsigned long long s_tests[WPB];
    __shared__ int32_t s_kept[WPB];
    if (lane == 0) {
        s_tests[w] = (unsigned long long)mine;
        s_kept[w] = kept;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0, k = 0;
        for (int i = 0; i < WPB; i++) {
            t += s_tests[i];
            k += (unsigned long long)s_kept[i];
        }
        if (t) region_add(scal, REGION_TESTS, t);
        if (k) region_add(scal, REGION_KEPT, k);
    }
}

// the entry of piece p: the last whose first piece is <= p (entry 0 starts at piece 0)
__device__ inline Heavy heavy_of(const Heavy *__restrict__ heavy, int64_t ne, int64_t p) {
    int64_t a = 0, b = ne - 1;
    while (a < b) {
        const int64_t mid = (a + b + 1) >> 1;
        if (heavy[mid].first <= p) a = mid;
        else b = mid - 1;
    }
    return heavy[a];
}

template <class R>
__global__ __launch_bounds__(BLK) void k_tests_pieces(const Heavy *__restrict__ heavy,
                                                      const unsigned long long *__restrict__ counter, int64_t cap,
                                                      R runner) {
    __shared__ typename R::Lds flds[WPB];
    typename R::Lds &F = flds[wave_id()];
    const int lane = lane_id();
    const unsigned long long c = *counter;
    const int64_t ne = (int64_t)(c >> HEAVY_SHIFT) < cap ? (int64_t)(c >> HEAVY_SHIFT) : cap;
    const int64_t np = (int64_t)(c & PIECE_MASK);
    if (ne > 0) {
        for (int64_t p0 = (int64_t)blockIdx.x * BLK + 64 * wave_id(); p0 < np; p0 += (int64_t)gridDim.x * BLK) {
            const int64_t p = p0 + lane;
            const bool on = p < np;
            const Heavy h = heavy_of(heavy, ne, on ? p : p0);
            int32_t e[3];
            for (int k = 0; k < 3; k++) e[k] = runner.sv[3 * h.slot + k];
            const TriLists T = load_lists(runner.rec, e[0], e[1], e[2]);
            stage_runs(F, lane, T, e, runner.live(T), h.slot); // this lane's own column
            // pieces past the last listed triangle's belong to ones that ran
            // where they were found: they lie past every run, nothing is tested
            runner.piece(F, lane, (p - h.first) * PIECE_TESTS, PIECE_TESTS, on);
        }
    }
    runner.finish();
}

constexpr int64_t MAX_HEAVY = 1 << 22; // 64 MB of entries at most
constexpr int64_t MIN_HEAVY = 1 << 16; // room for this many however few triangles are kept
constexpr int64_t LIGHT_BLOCKS = 4096; // a group per wavefront or two; 16,384 blocks mostly started for nothing
constexpr int64_t PIECE_BLOCKS = 8192;
// A plan's block count may come from a file: more than this many could take the count
// of heavy triangles past its 24 bits (and have no use: tried shapes end at 16,384).
constexpr int64_t MOST_TEST_BLOCKS = 32768;
static_assert(MAX_HEAVY + 64 * WPB * MOST_TEST_BLOCKS < (int64_t)1 << (64 - HEAVY_SHIFT) && LIGHT_BLOCKS <= MOST_TEST_BLOCKS,
              "entries of the heavy list's counter");

// the heavy list's capacity limit: MAX_HEAVY, or FOLTY_MAX_HEAVY (>= 1) when set
inline int64_t max_heavy() {
    static const int64_t v = [] {
        const char *e = getenv("FOLTY_MAX_HEAVY");
        const long long x = e ? atoll(e) : 0;
        return x >= 1 ? (int64_t)std::min<long long>(x, MAX_HEAVY) : MAX_HEAVY;
    }();
    return v;
}

// Entries a query's heavy list holds: at most one per slot of the filter's
// output (at least MIN_HEAVY, at most the limit).
inline int64_t heavy_slots(int64_t slots) {
    return std::max<int64_t>(1, std::min<int64_t>(std::max<int64_t>(slots + 1, MIN_HEAVY), max_heavy()));
}

// The tests of the triangles the last filter kept (see k_tests_light): chunks is
// the number of its chunks, or an upper bound.
template <class R>
void launch_tests(Workspace &ws, const CandBuf &B, const R &runner, int64_t chunks, hipStream_t s) {
    // any capacity gives the same result: a fixed scratch takes the smallest, or what it has left
    const int64_t left = arena_left();
    const int64_t cap = left < 0 ? heavy_slots(ws.kept_most)
                                 : std::max<int64_t>(1, std::min(heavy_slots(0), (left - 256) / (int64_t)sizeof(Heavy)));
    ws.pieces.ensure(sizeof(Heavy) * (size_t)cap);
    unsigned long long *np = ws.scal.as<unsigned long long>() + SCAL_HEAVY;
    // up to eight wavefronts per chunk (chunk_parts)
    const unsigned lb = (unsigned)std::max<int64_t>(1, std::min<int64_t>((8 * chunks + WPB - 1) / WPB, LIGHT_BLOCKS));
    k_tests_light<<<lb, BLK, 0, s>>>(B, runner, ws.pieces.as<Heavy>(), np, cap, ws.scal.as<unsigned long long>());
    FOLTY_LAUNCHED();
    // the pieces are numbered on the device
    const unsigned pb = (unsigned)std::max<int64_t>(1, std::min<int64_t>(chunks * 16, PIECE_BLOCKS));
    k_tests_pieces<<<pb, BLK, 0, s>>>(ws.pieces.as<Heavy>(), np, cap, runner);
    FOLTY_LAUNCHED();
}

inline EnumGraph enum_graph(const Index &ix) {
    return EnumGraph{ix.item.as<EnumItem>(), ix.oadj.as<int32_t>(),  ix.seg.as<int4>(),
                     ix.srng.as<uint2>(),    ix.owner.as<int32_t>(), ix.ooff.as<int32_t>(),
                     ix.n <= (1 << 22)};
}

// Chunks that hold every triangle of a graph, `waves` wavefronts filling them: a
// wavefront leaves at most one chunk partly filled, and none empty.
inline int64_t most_chunks(int64_t triangles, int64_t waves) { return std::min(triangles, triangles / 64 + waves); }
constexpr int64_t CHUNK_BYTES = 3 * 4 * 64 + 4;
} // namespace

// query.hip: the single-query filter and its scalars
void clear_query(const Index &ix, Workspace &ws, bool counts, hipStream_t s);
void read_scalars(Workspace &ws, hipStream_t s, bool pairs);
int64_t chunks_taken(const Workspace &ws, const CandBuf &B);
int64_t region_sum(const Workspace &ws, int what);
CandBuf filter_triangles(Index &ix, int variant, int64_t dmax, Workspace &ws, hipStream_t s, bool one_pass);
void after_filter(Index &ix, Workspace &ws, int64_t delta, bool one_pass);

} // namespace folty
