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

// runtime predicate code (one code per job in a batch)
__device__ inline int64_t tri_work_rt(int variant, const TriLists &T, uint32_t dq) {
    switch (variant) {
    case 0: return tri_work<0>(T, dq);
    case 1: return tri_work<1>(T, dq);
    case 2: return tri_work<2>(T, dq);
    case 3: return tri_work<3>(T, dq);
    case 4: return tri_work<4>(T, dq);
    case 5: return tri_work<5>(T, dq);
    case 6: return tri_work<6>(T, dq);
    default: return tri_work<7>(T, dq);
    }
}

// first position p in [from, n) with L[p] >= key (n if none)
__device__ inline int32_t lower_bound_from(const int64_t *__restrict__ L, int32_t from, int32_t n, int64_t key) {
    if (from >= n || L[from] >= key) return from;
    int32_t a = from + 1, b = n;
    while (a < b) {
        int32_t mid = (a + b) >> 1;
        if (L[mid] < key) a = mid + 1;
        else b = mid;
    }
    return a;
}

// Entry k of a list of at most two entries, from its record's first and last
// timestamps (exact when the timestamps fit 32 bits, tshift = 0).
__device__ inline int64_t short_at(const Span &l, int32_t k) { return (int64_t)(k == 0 ? l.lo : l.hi); }
__device__ inline int32_t short_lower_bound(const Span &l, int32_t from, int64_t key) {
    int32_t p = from;
    while (p < l.n && short_at(l, p) < key) p++;
    return p;
}

// cnt consecutive temporal edges of L1 starting at l1s against (L2, L3).  With
// SHORT and `inl` (timestamps below 2^32) a list of one or two entries is read
// from its span's first and last timestamps instead of ts: most lists are that
// short, and their entries are scattered reads that no neighbouring test
// shares.  (A compile-time switch: the branches cost registers where unused.)
template <bool SHORT> struct DirectOpT {
    static constexpr bool kShort = SHORT;
    int64_t delta;
    uint32_t *count;
    int32_t *diff = nullptr; // per sorted edge + 1: +1 / -1 at the ends of edge ranges (interval evaluation)
    bool inl = false;
    __device__ inline void operator()(const int64_t *__restrict__ ts, int32_t l1s, int32_t cnt, const Span &l2,
                                      const Span &l3) const {
        const int64_t *L2 = ts + l2.s, *L3 = ts + l3.s;
        const bool s2 = SHORT && inl && l2.n <= 2, s3 = SHORT && inl && l3.n <= 2;
        int32_t c2 = 0, c3 = 0;
        for (int32_t q = 0; q < cnt; q++) {
            int32_t e = l1s + q;
            int64_t t = ts[e];
            c2 = s2 ? short_lower_bound(l2, c2, t) : lower_bound_from(L2, c2, l2.n, t);
            if (c2 == l2.n) break; // later edges are no earlier: no t2 for them either
            int64_t t2 = s2 ? short_at(l2, c2) : L2[c2];
            if (t2 - t > delta) continue;
            c3 = s3 ? short_lower_bound(l3, c3, t2) : lower_bound_from(L3, c3, l3.n, t2);
            if (c3 == l3.n) break;
            if ((s3 ? short_at(l3, c3) : L3[c3]) - t <= delta) atomicAdd(&count[e], 1u);
        }
    }

    // The same run evaluated from L2 (paper, the in-neighbour theorem: e forms
    // a triangle with w iff some entry t2 of L2, with t3 the first entry of L3
    // at or after t2 and t3 - t2 <= delta, has t3 - delta <= t(e) <= t2).
    // Those intervals have non-decreasing ends, so entry j adds exactly the
    // times in [max(t3 - delta, t2' + 1), t2] (t2' the entry before it) to the
    // union of the earlier ones; each such piece is a range of L1 marked +1 / -1
    // in diff, whose prefix sum over the sorted edges adds one per third vertex.
    // Entries [j0, j0 + cnt) of L2.
    __device__ inline void iv(const int64_t *__restrict__ ts, const Span &l1, int32_t j0, int32_t cnt,
                              const Span &l2, const Span &l3) const {
        const int64_t *L1 = ts + l1.s, *L2 = ts + l2.s, *L3 = ts + l3.s;
        int32_t c3 = 0, a = 0, b = 0;
        for (int32_t q = 0; q < cnt; q++) {
            const int32_t j = j0 + q;
            const int64_t t2 = L2[j];
            c3 = lower_bound_from(L3, c3, l3.n, t2);
            if (c3 == l3.n) break; // no t3 for this or any later entry
            const int64_t t3 = L3[c3];
            if (t3 - t2 > delta) continue; // an empty interval
            int64_t lo = t3 - delta;
            if (j > 0 && L2[j - 1] + 1 > lo) lo = L2[j - 1] + 1;
            if (lo > t2) continue;
            a = lower_bound_from(L1, a, l1.n, lo);
            b = lower_bound_from(L1, a > b ? a : b, l1.n, t2 + 1);
            if (a < b) {
                atomicAdd(&diff[l1.s + a], 1);
                atomicAdd(&diff[l1.s + b], -1);
            }
        }
    }
};
using DirectOp = DirectOpT<false>;      // plain tests (also the interval evaluation)
using DirectShortOp = DirectOpT<true>;  // short lists from their spans' end timestamps

// the smallest window per (e, w) into a histogram over sorted window levels:
// level j counts w whose smallest window lies in (lv[j-1], lv[j]]
struct PoolOp {
    const int64_t *lv;
    int nl, nls;
    uint32_t *hist;
    unsigned long long *tmask; // per tile of 64 edges: bit e & 63 set once a counter of edge e is non-zero
    __device__ inline void operator()(const int64_t *__restrict__ ts, int32_t l1s, int32_t cnt, const Span &l2,
                                      const Span &l3) const {
        const int64_t *L2 = ts + l2.s, *L3 = ts + l3.s;
        const int64_t dmax = lv[nl - 1];
        int32_t c2 = 0, c3 = 0;
        for (int32_t q = 0; q < cnt; q++) {
            int32_t e = l1s + q;
            int64_t t = ts[e];
            c2 = lower_bound_from(L2, c2, l2.n, t);
            if (c2 == l2.n) break;
            int64_t t2 = L2[c2];
            if (t2 - t > dmax) continue;
            c3 = lower_bound_from(L3, c3, l3.n, t2);
            if (c3 == l3.n) break;
            int64_t win = L3[c3] - t;
            if (win > dmax) continue;
            int a = 0, b = nl;
            while (a < b) {
                int mid = (a + b) >> 1;
                if (lv[mid] < win) a = mid + 1;
                else b = mid;
            }
            if (atomicAdd(&hist[hist_at(e, a, nls)], 1u) == 0u) atomicOr(&tmask[e >> 6], 1ull << (e & 63));
        }
    }
};

// one run of a surviving triangle within the chunk [k, k1); r = tests of this
// triangle still to skip.  Returns false once the chunk is used up.  With SS (and
// a filter that counted tests the same way) a run whose L2 is shorter than L1
// has |L2| tests, the entries of L2, and is evaluated from them.
template <int VAR, int I, int J, class Op, bool SS = false>
__device__ inline bool chunk_run(const TriLists &T, uint32_t dq, const int64_t *ts, int64_t &r, int64_t &k,
                                 int64_t k1, const Op &op) {
    Span l1, l2, l3;
    if (!run_lists<VAR, I, J>(T, dq, l1, l2, l3)) return true;
    const int32_t w = run_tests<SS>(l1, l2);
    if (r >= w) {
        r -= w;
        return true;
    }
    int64_t cnt = w - r;
    if (cnt > k1 - k) cnt = k1 - k;
    if constexpr (SS) {
        if (w < l1.n) op.iv(ts, l1, (int32_t)r, (int32_t)cnt, l2, l3);
        else op(ts, l1.s + (int32_t)r, (int32_t)cnt, l2, l3);
    } else {
        op(ts, l1.s + (int32_t)r, (int32_t)cnt, l2, l3);
    }
    k += cnt;
    r = 0;
    return k < k1;
}

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
// low and high half, timestamps >> rshift (RNG_BITS bits); an empty list is
// (-32768, -32768).  In this form the tests below are packed additions whose
// signs decide, and an empty list fails every one of them.
constexpr int RNG_BITS = 14;
constexpr uint32_t RNG_EMPTY = 0x80008000u;
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
            const uint32_t i = __builtin_amdgcn_mbcnt_hi(w1, __builtin_amdgcn_mbcnt_lo(w0, (uint32_t)seg0));
            ek[k] = L.sg[i];
            if constexpr (LOOSE) ik[k] = i;
            seg0 += __builtin_popcount(w0) + __builtin_popcount(w1);
            vk[k] = q < nq;
            pk[k] = ek[k].x + (uint32_t)q;
        }
        if constexpr (Sink::kAll) {
#pragma unroll
            for (int k = 0; k < ENUM_UNROLL; k++) xk[k] = vk[k] ? oadj[pk[k]] : -1;
        }
        if constexpr (Sink::kRanges) {
#pragma unroll
            for (int k = 0; k < ENUM_UNROLL; k++) rk[k] = vk[k] ? sink.rng[pk[k]] : make_uint2(RNG_EMPTY, RNG_EMPTY);
        }
        if constexpr (Sink::kRanges && !Sink::kAll) {
            bool any = false;
#pragma unroll
            for (int k = 0; k < ENUM_UNROLL; k++) {
                vk[k] = sink.first(ek[k].z, ek[k].w, rk[k]); // false past the item's probes
                any = any || vk[k];
            }
            if (!__ballot(any)) continue;
            if (!built) {
                tab_build(L, oadj, b, d, ahead.v, tlog);
                built = true;
            }
#pragma unroll
            for (int k = 0; k < ENUM_UNROLL; k++) xk[k] = vk[k] ? oadj[pk[k]] : -1;
        }
#pragma unroll
        for (int k = 0; k < ENUM_UNROLL; k++) {
            if (!__ballot(vk[k])) continue;
            bool h = false;
            int32_t pw = 0;
            if (vk[k]) h = find(LOOSE ? ik[k] : 0u, xk[k], pw);
            if constexpr (!Sink::kRanges) {
                int32_t e01 = 0, e02 = 0, e12 = 0;
                if (h) tri_edges((int32_t)ek[k].y, (int32_t)pk[k], pw, e01, e02, e12);
                sink.hit(h, e01, e02, e12);
            } else {
                if constexpr (Sink::kHits) sink.nhit += (unsigned long long)__popcll(__ballot(h));
                if constexpr (Sink::kAll && Sink::kFirst) h = h && sink.first(ek[k].z, ek[k].w, rk[k]);
                if (__ballot(h)) sink.found(h, ek[k].z, ek[k].w, rk[k], (int32_t)ek[k].y, (int32_t)pk[k], pw);
            }
        }
    }
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

template <int VAR, class Op, bool SS = false>
__device__ inline void chunk_runs(const TriLists &L, uint32_t dq, const int64_t *ts, int64_t &r, int64_t &k, int64_t k1,
                                  const Op &op) {
    if (chunk_run<VAR, 0, 1, Op, SS>(L, dq, ts, r, k, k1, op) && chunk_run<VAR, 1, 0, Op, SS>(L, dq, ts, r, k, k1, op) &&
        chunk_run<VAR, 0, 2, Op, SS>(L, dq, ts, r, k, k1, op) && chunk_run<VAR, 2, 0, Op, SS>(L, dq, ts, r, k, k1, op) &&
        chunk_run<VAR, 1, 2, Op, SS>(L, dq, ts, r, k, k1, op))
        chunk_run<VAR, 2, 1, Op, SS>(L, dq, ts, r, k, k1, op);
}

template <class Op>
__device__ inline void chunk_runs_rt(int variant, const TriLists &L, uint32_t dq, const int64_t *ts, int64_t &r,
                                     int64_t &k, int64_t k1, const Op &op) {
    switch (variant) {
    case 0: chunk_runs<0>(L, dq, ts, r, k, k1, op); break;
    case 1: chunk_runs<1>(L, dq, ts, r, k, k1, op); break;
    case 2: chunk_runs<2>(L, dq, ts, r, k, k1, op); break;
    case 3: chunk_runs<3>(L, dq, ts, r, k, k1, op); break;
    case 4: chunk_runs<4>(L, dq, ts, r, k, k1, op); break;
    case 5: chunk_runs<5>(L, dq, ts, r, k, k1, op); break;
    case 6: chunk_runs<6>(L, dq, ts, r, k, k1, op); break;
    default: chunk_runs<7>(L, dq, ts, r, k, k1, op); break;
    }
}

// ---------------------------------------------------------------------------
// a.6: scheduling the tests of the triangles the filter kept
// ---------------------------------------------------------------------------
// A wavefront takes one chunk of the filter's output, a triangle per lane, reads
// their records and finds the runs that can count and their tests.  A triangle
// with at most LIGHT_TESTS tests is run by the wavefront.  One with more (a
// heavy triangle) gets an entry in a list and a range of piece numbers, both
// from one packed counter, so entries are in the order of their pieces; a second
// kernel runs piece p (tests [4 i, 4 i + 4) of its triangle) per thread, finding
// its entry by binary search over the entries' first pieces and starting its L2
// and L3 cursors with one binary search each (the merge-path split of a long run
// over neighbouring threads).  Heavy triangles past the list's capacity run where
// they were found, so any capacity gives the same result.
//
// How a wavefront runs its light tests depends on the runner.  Flat runners (the
// per-edge counts): the lanes stage their triangles' six list spans in LDS, and
// the tests, concatenated, go one per lane, so neighbouring lanes take
// neighbouring tests of one run and their loads coalesce; each test finds its
// triangle by a search over 64 prefix sums in LDS and its cursors by binary
// search.  Other runners (the exists-exists-exists counting, whose window
// bookkeeping is shared by the tests of a run): each lane runs its own
// triangle's tests in order.
// 70M-edge graph, one year (36.8M tests) and a graph of 5,000-edge lists closed
// by short ones (104M tests): light limit 16 / pieces of 32: 2.45 and 3.2 ms;
// 64 / 8: 1.97 and 1.74 ms; 64 / 4: 1.85 and 1.15 ms; 64 / 2: 1.83 and 1.30 ms
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

// One light group's survivors in LDS: start and length of each directed list,
// the runs that can count (bit k: run k in the order of chunk_runs), and the
// inclusive prefix of the survivors' tests.
// SHORT also keeps each list's first and last timestamp (3 KB more per
// wavefront), for tests that read short lists from them.
template <bool SHORT> struct FlatLds;
template <> struct FlatLds<false> {
    int32_t incl[64];
    int32_t ls[6][64];
    int32_t ln[6][64];
    uint32_t live[64];
};
template <> struct FlatLds<true> : FlatLds<false> {
    uint32_t lo[6][64]; // first and last timestamp >> tshift
    uint32_t hi[6][64];
};

// run k = (I, J) of survivor si holds test r (r < that run's tests): run it
template <int VAR, int I, int J, bool SS, class Op, bool SHORT>
__device__ inline bool flat_run(const FlatLds<SHORT> &F, int si, int k, int64_t &r, const int64_t *__restrict__ ts,
                                const Op &op) {
    if (!((F.live[si] >> k) & 1u)) return false;
    using P = Pick<VAR, I, J>;
    constexpr int i1 = list_id(I, J), i2 = list_id(P::L2a, P::L2b), i3 = list_id(P::L3a, P::L3b);
    const int32_t n1 = F.ln[i1][si], n2 = F.ln[i2][si];
    const int32_t nt = SS && n2 < n1 ? n2 : n1;
    if (r >= nt) {
        r -= nt;
        return false;
    }
    Span l1{}, l2{}, l3{};
    l1.s = F.ls[i1][si];
    l1.n = n1;
    l2.s = F.ls[i2][si];
    l2.n = n2;
    l3.s = F.ls[i3][si];
    l3.n = F.ln[i3][si];
    if constexpr (SHORT) {
        l2.lo = F.lo[i2][si];
        l2.hi = F.hi[i2][si];
        l3.lo = F.lo[i3][si];
        l3.hi = F.hi[i3][si];
    }
    if (SS && nt < n1) op.iv(ts, l1, (int32_t)r, 1, l2, l3);
    else op(ts, l1.s + (int32_t)r, 1, l2, l3);
    return true;
}

// The three lists of run k (order of tri_live's bits) under a predicate code, as
// indices in list_id's order: run k's own list is number k; the others sit three
// bits each in two words, the same for every lane.
struct RunLists {
    uint32_t l2, l3;
};
__device__ inline RunLists run_list_ids(int variant) {
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

// test r of triangle si's live runs, from the staged spans, for a predicate code
// read at run time
template <class Op>
__device__ inline void flat_run_rt(const FlatLds<false> &F, const RunLists &R, int si, int32_t r,
                                   const int64_t *__restrict__ ts, const Op &op) {
    uint32_t live = F.live[si];
    while (live) {
        const int k = __ffs((int)live) - 1;
        live &= live - 1;
        const int32_t n1 = F.ln[k][si];
        if (r >= n1) {
            r -= n1;
            continue;
        }
        const int i2 = (int)(R.l2 >> (3 * k)) & 7, i3 = (int)(R.l3 >> (3 * k)) & 7;
        Span l2{}, l3{};
        l2.s = F.ls[i2][si];
        l2.n = F.ln[i2][si];
        l3.s = F.ls[i3][si];
        l3.n = F.ln[i3][si];
        op(ts, F.ls[k][si] + r, 1, l2, l3);
        return;
    }
}

// Runs the tests of the per-edge counts: work() is a survivor's number of
// tests, run() takes tests [r, k1) of it in order, flat() its test r alone,
// from the spans stage() put in LDS.
template <int VAR, class Op, bool SS> struct CountRunner {
    static constexpr bool kFlat = true;
    static constexpr bool kShort = Op::kShort && !SS; // staging keeps the lists' end timestamps
    static_assert(!(Op::kShort && SS), "short lists are read only by the plain evaluation");
    using Flat = FlatLds<kShort>;
    using Surv = TriLists;
    uint32_t dq;
    const int64_t *ts;
    Op op;
    const int32_t *sv; // survivors as three oriented edges
    const EdgeRec *rec;
    __device__ inline TriLists load(int64_t slot) const {
        return load_lists(rec, sv[3 * slot], sv[3 * slot + 1], sv[3 * slot + 2]);
    }
    __device__ inline int64_t work(const TriLists &L) const { return tri_work<VAR, SS>(L, dq); }
    __device__ inline void run(const TriLists &L, int64_t, int64_t r, int64_t k1) {
        int64_t k = r;
        chunk_runs<VAR, Op, SS>(L, dq, ts, r, k, k1, op);
    }
    __device__ inline void stage(Flat &F, int lane, const TriLists &T, bool light) const {
        const Span *sp[6] = {&T.d01, &T.d10, &T.d02, &T.d20, &T.d12, &T.d21};
#pragma unroll
        for (int k = 0; k < 6; k++) {
            F.ls[k][lane] = sp[k]->s;
            F.ln[k][lane] = sp[k]->n;
            if constexpr (kShort) {
                F.lo[k][lane] = sp[k]->lo;
                F.hi[k][lane] = sp[k]->hi;
            }
        }
        F.live[lane] = light ? tri_live<VAR>(T, dq) : 0u;
    }
    __device__ inline void flat(const Flat &F, int si, int64_t r) const {
        flat_run<VAR, 0, 1, SS>(F, si, 0, r, ts, op) || flat_run<VAR, 1, 0, SS>(F, si, 1, r, ts, op) ||
            flat_run<VAR, 0, 2, SS>(F, si, 2, r, ts, op) || flat_run<VAR, 2, 0, SS>(F, si, 3, r, ts, op) ||
            flat_run<VAR, 1, 2, SS>(F, si, 4, r, ts, op) || flat_run<VAR, 2, 1, SS>(F, si, 5, r, ts, op);
    }
    __device__ inline void finish() {}
};

// Lanes with np > 0 (heavy survivors, np pieces each) take list entries and
// piece numbers for the whole wavefront with one atomic.  A survivor whose
// entry lies past cap runs here; the piece numbers it reserved follow every
// listed one.  `full` is set once this wavefront's atomic returned an entry
// count of cap or more, after which it lists nothing: each wavefront adds at
// most 64 entries past cap, so the entry count stays below cap + 64 x (the
// grid's wavefronts), far below 2^24.
template <class R>
__device__ inline void defer_heavy(R &runner, const typename R::Surv &S, int64_t slot, int64_t w, int64_t np,
                                   Heavy *__restrict__ heavy, unsigned long long *__restrict__ counter, int64_t cap,
                                   bool &full) {
    if (!__ballot(np > 0)) return;
    if (full) {
        if (np > 0) runner.run(S, slot, 0, w);
        return;
    }
    const unsigned long long add = np > 0 ? (1ull << HEAVY_SHIFT) | (unsigned long long)np : 0ull;
    const unsigned long long incl = wave_inclusive_sum(add);
    unsigned long long at = 0;
    if (lane_id() == 63) at = atomicAdd(counter, incl);
    at = __shfl(at, 63);
    full = (int64_t)(at >> HEAVY_SHIFT) + 64 >= cap;
    if (np == 0) return;
    const unsigned long long mine = at + incl - add;
    const int64_t e = (int64_t)(mine >> HEAVY_SHIFT);
    if (e < cap) heavy[e] = Heavy{slot, (int64_t)(mine & PIECE_MASK)};
    else runner.run(S, slot, 0, w);
}

// A wavefront's group of chunks as a dense sequence of slots: narrow windows
// leave most chunks with an entry or two, and their triangles are taken 64 at a
// time across chunks.  Groups of up to 64 chunks, fewer when that would leave
// less than GROUPS_WANTED groups; with few chunks each is shared by up to eight
// wavefronts, since a wavefront's tests are a chain of dependent reads.
constexpr int32_t GROUPS_WANTED = 16384;
__device__ inline int32_t group_chunks(int32_t total) {
    const int32_t k = total / GROUPS_WANTED;
    return k < 1 ? 1 : k > 64 ? 64 : k;
}
__device__ inline int32_t chunk_parts(int32_t total) {
    return total >= GROUPS_WANTED / 2 ? 1 : total >= GROUPS_WANTED / 4 ? 2 : total >= GROUPS_WANTED / 8 ? 4 : 8;
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
    __shared__ typename R::Flat flds[R::kFlat ? WPB : 1];
    __shared__ GroupLds glds[WPB];
    __shared__ Chunks C;
    __shared__ unsigned long long s_tests[WPB];
    __shared__ int32_t s_kept[WPB];
    const int w = wave_id();
    const int lane = lane_id();
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
            const bool on = q0 + lane < slots;
            int64_t slot = 0, wk = 0, np = 0;
            typename R::Surv S{};
            if (on) {
                slot = group_slot(glds[w], q0 + lane);
                S = runner.load(slot);
                if (edges_meet(S, runner.dq)) wk = runner.work(S);
                if (wk > LIGHT_TESTS) np = (wk + PIECE_TESTS - 1) / PIECE_TESTS;
            }
            mine += wk;
            defer_heavy(runner, S, slot, wk, np, heavy, counter, cap, full);
            const int64_t light = np ? 0 : wk;
            if constexpr (R::kFlat) {
                typename R::Flat &F = flds[w];
                const int32_t incl = wave_scan((int32_t)light);
                const int32_t total = __builtin_amdgcn_readlane(incl, 63);
                if (total == 0) continue;
                F.incl[lane] = incl;
                runner.stage(F, lane, S, light != 0);
                wave_sync();
                for (int32_t t = lane; t < total; t += 64) {
                    // the triangle whose tests hold t: the first si with incl[si] > t
                    int a = 0, b = 63;
                    while (a < b) {
                        const int mid = (a + b) >> 1;
                        if (F.incl[mid] > t) b = mid;
                        else a = mid + 1;
                    }
                    runner.flat(F, a, (int64_t)(t - (a ? F.incl[a - 1] : 0)));
                }
                wave_sync(); // the LDS is rewritten by the next triangles
            } else {
                if (light) runner.run(S, slot, 0, light);
            }
        }
        wave_sync(); // the group's LDS is rewritten by the next group
    }
    runner.finish();
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
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

template <class R>
__global__ __launch_bounds__(BLK) void k_tests_pieces(const Heavy *__restrict__ heavy,
                                                      const unsigned long long *__restrict__ counter, int64_t cap,
                                                      R runner) {
    const unsigned long long c = *counter;
    const int64_t ne = (int64_t)(c >> HEAVY_SHIFT) < cap ? (int64_t)(c >> HEAVY_SHIFT) : cap;
    const int64_t np = (int64_t)(c & PIECE_MASK);
    if (ne > 0) {
        for (int64_t p = (int64_t)blockIdx.x * BLK + threadIdx.x; p < np; p += (int64_t)gridDim.x * BLK) {
            // the last entry whose first piece is <= p (entry 0 starts at piece 0)
            int64_t a = 0, b = ne - 1;
            while (a < b) {
                const int64_t mid = (a + b + 1) >> 1;
                if (heavy[mid].first <= p) a = mid;
                else b = mid - 1;
            }
            const Heavy h = heavy[a];
            const int64_t k0 = (p - h.first) * PIECE_TESTS;
            // pieces past the last listed survivor's belong to ones that ran
            // where they were found: k0 lies past every run, nothing is tested
            runner.run(runner.load(h.slot), h.slot, k0, k0 + PIECE_TESTS);
        }
    }
    runner.finish();
}

constexpr int64_t MAX_HEAVY = 1 << 22; // 64 MB of heavy-survivor entries at most
constexpr int64_t MIN_HEAVY = 1 << 16; // room for this many whatever the survivors
constexpr int64_t LIGHT_BLOCKS = 16384;
constexpr int64_t PIECE_BLOCKS = 8192;

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
    // any capacity gives the same result: a fixed scratch keeps it small
    const int64_t cap = heavy_slots(arena_left() >= 0 ? 0 : 64 * chunks);
    ws.pieces.ensure(sizeof(Heavy) * (size_t)cap);
    unsigned long long *np = ws.scal.as<unsigned long long>() + SCAL_HEAVY;
    // up to eight wavefronts per chunk
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
