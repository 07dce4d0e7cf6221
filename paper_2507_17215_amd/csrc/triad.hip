// The exists-exists-exists triadic query: solution triples and temporal
// triangles (paper, Definition of a solution; Section 1, where this prefix is
// identified with temporal triangle counting).
//
// It shares the index and the time-range filter of the exists-exists-forall
// query: the filter keeps the static triangles with a run (triangle, directed
// list E_{a,b}) whose three lists can hold t <= t2 <= t3 <= t + delta, and a lane
// takes a run or a piece of one:
//   - solutions: the first-entry search of Theorems 3.1 and 3.2 per edge of
//     E_{a,b}, stopping at the first edge with a triangle, sets the run's bit;
//     a run is the ordered triple (a, b, w), so the set bits are the solutions;
//   - temporal triangles (optional): for an edge at time t, with L2[lo, hi) the
//     entries of L2 in [t, t + delta], h3 the first entry of L3 after t + delta
//     and f(j) the first entry of L3 at or after L2[j], the edge closes
//     sum_{j in [lo, hi)} (h3 - f(j)) = (hi - lo) h3 - (F(hi) - F(lo)) pairs,
//     F the running sum of f.  lo, hi, h3 and the two search cursors for f only
//     move forward over a piece's time-sorted edges, so a piece costs its edges
//     plus the entries its windows pass, each with a search (range_sum).
// The set bits are then counted chunk by chunk over the kept triangles, and listed
// as (a, b, w) in original ids, sorted by two stable radix sorts (w, then
// the pair key a n + b).
#include <algorithm>
#include <cstring>

#include "tri_device.h"

namespace folty {
namespace {

// first position p in [from, n) with L[p] - t > d (n if none); L ascending
__device__ inline int32_t past_window(const int64_t *__restrict__ L, int32_t from, int32_t n, int64_t t, int64_t d) {
    if (from >= n || L[from] - t > d) return from;
    int32_t a = from + 1, b = n;
    while (a < b) { // four entries per step, as in lower_bound
        const int32_t q = probe_step(b - a);
        const Probe P = probe(L, a, b);
        const int c = (P.x[0] - t <= d) + (a + q < b && P.x[1] - t <= d) + (a + 2 * q < b && P.x[2] - t <= d) +
                      (a + 3 * q < b && P.x[3] - t <= d);
        if (c == 0) return a;
        if (c < 4 && a + c * q < b) b = a + c * q;
        a += (c - 1) * q + 1;
    }
    return b;
}

struct TriadOut {
    int64_t delta;
    uint32_t *flag;                // bit run of byte (slot & 3) of word slot >> 2
    unsigned long long *inst;      // temporal triangles per input edge, or null
    const int32_t *perm;           // input position of each sorted edge (with inst)
};

// LDS of a wavefront: its staged triangles, and the ranges that its lanes sum together
struct TriadLds : RunLds<false, true> {
    int32_t cum[64];            // entries of the lanes' ranges up to this one
    int32_t j0[64];             // first entry of the range, in ts
    int32_t l3[64], n3[64];     // its L3
    unsigned long long sum[64];
};

// Sum over entries j in [a, b) of L2 of f(j) = entries of L3 before L2[j], for each
// lane's own lists and range (all lanes together; a lane without a range passes
// a >= b).  f0: a position that no f(j) lies before.  A range's entries go one
// after another with a moving cursor when the lanes' ranges are about as long;
// otherwise all lanes' entries are spread over the wavefront, each with a search of
// its own: a window holds a few entries mostly and hundreds at times, and the
// wavefront would wait for that one lane.
__device__ inline unsigned long long range_sum(TriadLds &F, const int64_t *__restrict__ ts, int32_t l2s, int32_t l3s,
                                               int32_t n3, int32_t a, int32_t b, int32_t &f0) {
    const int lane = lane_id();
    const int32_t len = b > a ? b - a : 0;
    const int32_t incl = wave_scan(len);
    const int32_t total = __builtin_amdgcn_readlane(incl, 63);
    if (!__ballot(len > 0)) return 0;
    // (the prefix sums of ranges below 2^24 fit 32 bits)
    if (__ballot(len >= 1 << 24) || !__ballot(len > 4 + 4 * (total >> 6))) {
        unsigned long long s = 0;
        for (int32_t j = a; j < b; j++) {
            f0 = lower_bound_from(ts + l3s, f0, n3, ts[l2s + j]);
            s += (unsigned)f0;
        }
        return s;
    }
    wave_sync();
    F.cum[lane] = incl;
    F.j0[lane] = l2s + a;
    F.l3[lane] = l3s;
    F.n3[lane] = n3;
    F.sum[lane] = 0;
    wave_sync();
    for (int32_t t = lane; t < total; t += 64) {
        const int o = staged_owner(F.cum, t);
        const int64_t x = ts[F.j0[o] + (t - (o ? F.cum[o - 1] : 0))];
        atomicAdd(&F.sum[o], (unsigned long long)(unsigned)lower_bound_from(ts + F.l3[o], 0, F.n3[o], x));
    }
    wave_sync();
    return F.sum[lane];
}

// Temporal triangles of edges [l1s, l1s + cnt) of each lane's run (all lanes
// together; cnt = 0: none) against its lists (L2, L3).
__device__ inline void triad_instances(TriadLds &F, const TriadOut &o, const int64_t *__restrict__ ts, int32_t l1s,
                                       int32_t cnt, const Span &l2, const Span &l3, int64_t slot, int run,
                                       unsigned long long &acc, bool &ovf) {
    const int64_t *L2 = ts + l2.s, *L3 = ts + l3.s;
    const int64_t d = o.delta;
    // the window's entries of L2, [lo, hi), and the sum of f over them
    int32_t lo = 0, hi = 0, fin = 0, fout = 0, h3 = 0;
    unsigned long long S = 0;
    bool any = false;
    for (int32_t q = 0; __ballot(q < cnt); q++) {
        int32_t nlo = lo, nhi = hi;
        int64_t t = 0;
        if (q < cnt) {
            t = ts[l1s + q];
            nlo = lower_bound_from(L2, lo, l2.n, t);
            nhi = past_window(L2, nlo > hi ? nlo : hi, l2.n, t, d);
        }
        S += range_sum(F, ts, l2.s, l3.s, l3.n, nlo > hi ? nlo : hi, nhi, fin);
        if (__ballot(nlo < nhi)) S -= range_sum(F, ts, l2.s, l3.s, l3.n, lo, nlo < hi ? nlo : hi, fout);
        lo = nlo;
        hi = nhi;
        if (lo == hi) {
            S = 0;
            if (lo == l2.n) cnt = 0; // no t2 at or after t for this or any later edge
        } else if (q < cnt) {
            h3 = past_window(L3, h3, l3.n, t, d);
            const unsigned long long pairs = (unsigned long long)(hi - lo) * (unsigned)h3 - S;
            if (pairs) {
                any = true;
                if (o.inst) atomicAdd(&o.inst[o.perm[l1s + q]], pairs);
                const unsigned long long x = acc + pairs;
                ovf |= x < acc;
                acc = x;
            }
        }
    }
    if (any) atomicOr(&o.flag[slot >> 2], 1u << (((int)(slot & 3) << 3) + run));
}

// Does any of edges [l1s, l1s + cnt) close a triangle?
__device__ inline void triad_any(const TriadOut &o, const int64_t *__restrict__ ts, int32_t l1s, int32_t cnt,
                                 const Span &l2, const Span &l3, int64_t slot, int run) {
    const List a{ts + l2.s, l2.n, nullptr}, b{ts + l3.s, l3.n, nullptr};
    int32_t c2 = 0, c3 = 0;
    for (int32_t q = 0; q < cnt; q++) {
        const Probe p2 = probe(a.p, c2, a.n), p3 = probe(b.p, c3, b.n);
        int64_t win;
        const TestEnd x = window_test(a, b, c2, c3, p2, p3, ts[l1s + q], o.delta, win);
        if (x == TEST_HIT) atomicOr(&o.flag[slot >> 2], 1u << (((int)(slot & 3) << 3) + run));
        if (x != TEST_MISS) return;
    }
}

// The triangles' runs, scheduled as the count's (k_tests_light, a run
// or a few tests of one per lane; then the pieces of triangles with many tests); total[0] += temporal triangles,
// total[1] = 1 on a 64-bit overflow.
template <int VAR, bool INST> struct TriadRunner {
    using Lds = TriadLds;
    static constexpr bool kTwo = false;
    uint32_t dq;
    const int64_t *ts;
    TriadOut o;
    unsigned long long *total;
    const int32_t *sv;  // the triangles as three oriented edges
    const EdgeRec *rec;
    unsigned long long acc = 0;
    bool ovf = false;
    __device__ inline uint32_t live(const TriLists &L) const { return tri_live<VAR>(L, dq); }
    __device__ inline int64_t work(const TriLists &L) const { return tri_work<VAR, false>(L, dq); }
    // A light triangle's items are its runs, which stop at the first edge that closes
    // a triangle; when all are counted, pieces of them: a whole run of 64 tests is then
    // a chain of some hundred dependent reads, which its wavefront waits for.
    __device__ inline int64_t units(const Lds &F, int si, int64_t) const {
        if (!INST) return __popc(F.live[si]);
        int64_t c = 0;
        for (uint32_t live = F.live[si]; live; live &= live - 1)
            c += (F.n[__ffs((int)live) - 1][si] + (int32_t)PIECE_TESTS - 1) / (int32_t)PIECE_TESTS;
        return c;
    }
    // edges [first, first + cnt) of each lane's run k (cnt = 0: none)
    __device__ inline void run(Lds &F, int si, int k, int32_t first, int32_t cnt) {
        constexpr RunLists ids = run_list_ids(VAR);
        const int i2 = (int)(ids.l2 >> (3 * k)) & 7, i3 = (int)(ids.l3 >> (3 * k)) & 7;
        const Span l2{F.s[i2][si], F.n[i2][si], 0, 0}, l3{F.s[i3][si], F.n[i3][si], 0, 0};
        if constexpr (INST) triad_instances(F, o, ts, F.s[k][si] + first, cnt, l2, l3, F.slot[si], k, acc, ovf);
        else triad_any(o, ts, F.s[k][si] + first, cnt, l2, l3, F.slot[si], k);
    }
    __device__ inline void flat(Lds &F, int si, int64_t r, bool on) {
        int k = 0;
        int32_t first = 0, cnt = 0;
        for (uint32_t live = on ? F.live[si] : 0u; live; live &= live - 1) {
            k = __ffs((int)live) - 1;
            const int32_t n1 = F.n[k][si], piece = INST ? (int32_t)PIECE_TESTS : n1, c = INST ? (n1 + piece - 1) / piece : 1;
            if (r < c) {
                first = (int32_t)r * piece;
                cnt = n1 - first < piece ? n1 - first : piece;
                break;
            }
            r -= c;
        }
        run(F, si, k, first, cnt);
    }
    __device__ inline void piece(Lds &F, int si, int64_t r, int32_t cnt, bool on) {
        uint32_t live = on ? F.live[si] : 0u;
        while (__ballot(live != 0u && cnt > 0)) { // each lane's next run with tests of the piece
            int k = 0;
            int32_t first = 0, m = 0;
            while (live && cnt > 0 && m == 0) {
                k = __ffs((int)live) - 1;
                live &= live - 1;
                const int32_t n1 = F.n[k][si];
                if (r >= n1) {
                    r -= n1;
                } else {
                    first = (int32_t)r;
                    m = cnt < n1 - first ? cnt : n1 - first;
                    cnt -= m;
                    r = 0;
                }
            }
            run(F, si, k, first, m);
        }
    }
    // every lane of the wavefront calls this once, at the end
    __device__ inline void finish() {
        if constexpr (INST) {
            for (int off = 32; off > 0; off >>= 1) {
                const unsigned long long y = __shfl_xor(acc, off);
                const int oy = __shfl_xor((int)ovf, off);
                const unsigned long long s = acc + y;
                ovf = ovf || oy || s < acc;
                acc = s;
            }
            if (lane_id() == 0 && (acc || ovf)) {
                const unsigned long long old = atomicAdd(&total[0], acc);
                if (ovf || old + acc < old) atomicOr(&total[1], 1ull);
            }
        }
    }
};

// The passes below go over the chunks of triangles the filter kept, a wavefront
// per chunk; slot p's bits are byte p of the flag array.
__global__ __launch_bounds__(BLK) void k_triad_clear(CandBuf B, uint32_t *__restrict__ flag) {
    __shared__ Chunks C;
    C.load(B);
    for (int32_t g = (int32_t)blockIdx.x * WPB + wave_id(); g < C.total; g += (int32_t)gridDim.x * WPB) {
        const int32_t chunk = __builtin_amdgcn_readfirstlane(C.at(B, g));
        if (lane_id() < 16) flag[(int64_t)chunk * 16 + lane_id()] = 0;
    }
}

// solutions of a chunk's triangles
__device__ inline uint32_t slot_bits(const CandBuf &B, const uint8_t *__restrict__ flag8, int32_t chunk) {
    return lane_id() < B.cnt[chunk] ? flag8[(int64_t)chunk * 64 + lane_id()] & 0x3fu : 0u;
}

// solutions per chunk, in the chunks' sequence (optional), and their total
__global__ __launch_bounds__(BLK) void k_triad_count(CandBuf B, const uint8_t *__restrict__ flag8,
                                                     int32_t *__restrict__ ccnt, unsigned long long *total) {
    __shared__ Chunks C;
    C.load(B);
    unsigned long long c = 0;
    for (int32_t g = (int32_t)blockIdx.x * WPB + wave_id(); g < C.total; g += (int32_t)gridDim.x * WPB) {
        const int32_t x = wave_scan(__popc(slot_bits(B, flag8, __builtin_amdgcn_readfirstlane(C.at(B, g)))));
        if (lane_id() == 63) {
            if (ccnt) ccnt[g] = x;
            c += (unsigned)x;
        }
    }
    if (!total) return;
    __shared__ unsigned long long s_c[WPB];
    if (lane_id() == 63) s_c[wave_id()] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long sum = 0;
        for (int i = 0; i < WPB; i++) sum += s_c[i];
        if (sum) atomicAdd(total, sum);
    }
}

// the endpoints (original ids) of oriented edge q: tail, head
__device__ inline void oriented_ends(const uint32_t *__restrict__ oeid, const int32_t *__restrict__ slo,
                                     const int32_t *__restrict__ shi, int32_t q, int32_t &tail, int32_t &head) {
    const uint32_t x = oeid[q];
    const uint32_t s = x & 0x7fffffffu;
    const int32_t lo = slo[s], hi = shi[s];
    tail = (x >> 31) ? lo : hi;
    head = (x >> 31) ? hi : lo;
}

// each set bit as (w, its index, pair key a n + b), from the chunk's offset
__global__ __launch_bounds__(BLK) void k_triad_emit(CandBuf B, const int64_t *__restrict__ coff,
                                                    const uint8_t *__restrict__ flag8,
                                                    const uint32_t *__restrict__ oeid, const int32_t *__restrict__ slo,
                                                    const int32_t *__restrict__ shi, int64_t n,
                                                    uint32_t *__restrict__ wkey, int32_t *__restrict__ idx,
                                                    unsigned long long *__restrict__ pkey) {
    __shared__ Chunks C;
    C.load(B);
    for (int32_t g = (int32_t)blockIdx.x * WPB + wave_id(); g < C.total; g += (int32_t)gridDim.x * WPB) {
        const int32_t chunk = __builtin_amdgcn_readfirstlane(C.at(B, g));
        const uint32_t bits = slot_bits(B, flag8, chunk);
        const int32_t mine = __popc(bits);
        int64_t o = coff[g] + wave_scan(mine) - mine;
        if (!bits) continue;
        const int32_t *e = B.sv + 3 * ((int64_t)chunk * 64 + lane_id());
        int32_t x0, x1, x2, t;
        oriented_ends(oeid, slo, shi, e[0], x0, x1);
        oriented_ends(oeid, slo, shi, e[1], t, x2);
        // run -> (a, b, w): (x0,x1,x2) (x1,x0,x2) (x0,x2,x1) (x2,x0,x1) (x1,x2,x0) (x2,x1,x0)
        const int32_t A[6] = {x0, x1, x0, x2, x1, x2};
        const int32_t Bv[6] = {x1, x0, x2, x0, x2, x1};
        const int32_t W[6] = {x2, x2, x1, x1, x0, x0};
#pragma unroll
        for (int run = 0; run < 6; run++) {
            if (!((bits >> run) & 1u)) continue;
            wkey[o] = (uint32_t)W[run];
            idx[o] = (int32_t)o;
            pkey[o] = (unsigned long long)A[run] * (unsigned long long)n + (unsigned long long)Bv[run];
            o++;
        }
    }
}

__global__ void k_gather_u64(const unsigned long long *__restrict__ in, const int32_t *__restrict__ idx, int64_t k,
                             unsigned long long *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < k) out[i] = in[idx[i]];
}

__global__ void k_triad_unpack(const unsigned long long *__restrict__ pkey, const uint32_t *__restrict__ w, int64_t k,
                               int64_t n, int32_t *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= k) return;
    const unsigned long long key = pkey[i];
    out[3 * i] = (int32_t)(key / (unsigned long long)n);
    out[3 * i + 1] = (int32_t)(key % (unsigned long long)n);
    out[3 * i + 2] = (int32_t)w[i];
}


void check_triad(const Graph *g, const folty_triad_query &q) {
    if (!g->ix.built) fail(FOLTY_ENOTBUILT, "folty_build_index has not been called for this graph");
    if (q.delta < 0) fail(FOLTY_EINVAL, "delta must be >= 0 (got %lld)", (long long)q.delta);
    if (q.variant > 7) fail(FOLTY_EINVAL, "variant must be 0..7 (got %u)", (unsigned)q.variant);
    if (q.flags & ~(FOLTY_TRIAD_TRIPLES | FOLTY_TRIAD_INSTANCES | FOLTY_TRIAD_EDGE_INSTANCES))
        fail(FOLTY_EINVAL, "unknown triad flags 0x%x", (unsigned)q.flags);
    for (int i = 0; i < 6; i++)
        if (q.reserved[i]) fail(FOLTY_EINVAL, "reserved fields of the triad query must be 0");
}

unsigned chunk_grid(int64_t chunks) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((chunks + WPB - 1) / WPB, 1024));
}

// the listed triples, sorted by (a, b, w), copied to res->trip; the filter took
// `chunks` chunks
void list_triples(const Index &ix, const Workspace &ws, const CandBuf &B, int64_t chunks, int64_t nsol, Result *res,
                  hipStream_t s) {
    if (nsol > INT32_MAX) fail(FOLTY_EOVERFLOW, "%lld solution triples exceed the listing limit of 2^31 - 1",
                               (long long)nsol);
    DevBuf ccnt, coff, wk, ix0, pk, wk2, ix2, pk2, trip;
    ccnt.ensure(4 * (size_t)chunks + 4);
    coff.ensure(8 * (size_t)chunks + 8);
    k_triad_count<<<chunk_grid(chunks), BLK, 0, s>>>(B, ws.tflag.as<uint8_t>(), ccnt.as<int32_t>(), nullptr);
    FOLTY_LAUNCHED();
    DevBuf cub;
    size_t need = exclusive_scan_i32_to_i64(nullptr, 0, ccnt.as<int32_t>(), coff.as<int64_t>(), chunks, s);
    const size_t k = (size_t)nsol;
    const int endw = std::max(1, bit_length((uint64_t)ix.n - 1));
    const int endp = std::max(1, bit_length((uint64_t)ix.n * (uint64_t)ix.n - 1));
    need = std::max(need, sort_pairs_u32_i32(nullptr, 0, nullptr, nullptr, nullptr, nullptr, (int64_t)k, endw, s));
    need = std::max(need, sort_pairs_u64_i32(nullptr, 0, nullptr, nullptr, nullptr, nullptr, (int64_t)k, endp, s));
    cub.ensure(need);
    exclusive_scan_i32_to_i64(cub.p, need, ccnt.as<int32_t>(), coff.as<int64_t>(), chunks, s);
    wk.ensure(4 * k);
    ix0.ensure(4 * k);
    pk.ensure(8 * k);
    wk2.ensure(4 * k);
    ix2.ensure(4 * k);
    pk2.ensure(8 * k);
    trip.ensure(12 * k);
    k_triad_emit<<<chunk_grid(chunks), BLK, 0, s>>>(B, coff.as<int64_t>(), ws.tflag.as<uint8_t>(),
                                                    ix.oeid.as<uint32_t>(), ix.slo.as<int32_t>(), ix.shi.as<int32_t>(),
                                                    ix.n, wk.as<uint32_t>(), ix0.as<int32_t>(),
                                                    pk.as<unsigned long long>());
    FOLTY_LAUNCHED();
    // by w, then stably by the pair key: (a, b, w) order
    sort_pairs_u32_i32(cub.p, need, wk.as<uint32_t>(), wk2.as<uint32_t>(), ix0.as<int32_t>(), ix2.as<int32_t>(),
                       (int64_t)k, endw, s);
    k_gather_u64<<<grid_for((int64_t)k, BLK), BLK, 0, s>>>(pk.as<unsigned long long>(), ix2.as<int32_t>(),
                                                           (int64_t)k, pk2.as<unsigned long long>());
    FOLTY_LAUNCHED();
    sort_pairs_u64_i32(cub.p, need, pk2.as<uint64_t>(), pk.as<uint64_t>(), wk2.as<int32_t>(), wk.as<int32_t>(),
                       (int64_t)k, endp, s);
    k_triad_unpack<<<grid_for((int64_t)k, BLK), BLK, 0, s>>>(pk.as<unsigned long long>(), wk.as<uint32_t>(),
                                                             (int64_t)k, ix.n, trip.as<int32_t>());
    FOLTY_LAUNCHED();
    res->trip.resize(3 * k);
    FOLTY_HIP(hipMemcpyAsync(res->trip.data(), trip.p, 12 * k, hipMemcpyDeviceToHost, s));
    FOLTY_HIP(hipStreamSynchronize(s));
}

} // namespace

Result *run_triad_query(Graph *g, const folty_triad_query &q, Workspace &ws) {
    check_triad(g, q);
    if (hipSetDevice(g->device) != hipSuccess) fail(FOLTY_EDEVICE, "hipSetDevice failed");
    Index &ix = g->ix;
    hipStream_t s = g->stream;
    const bool edge = (q.flags & FOLTY_TRIAD_EDGE_INSTANCES) != 0;
    const bool inst = edge || (q.flags & FOLTY_TRIAD_INSTANCES) != 0;
    std::unique_ptr<Result> res(new Result());
    StreamScope sc(s); // an error waits for the copies into res before res goes
    res->triad = true;
    res->device = g->device;
    ws.ensure_events();
    FOLTY_HIP(hipEventRecord(ws.ev[0], s));
    clear_query(ix, ws, false, s);
    unsigned long long *tot = ws.scal.as<unsigned long long>() + SCAL_TRIAD; // triangles, overflow, solutions
    if (edge) {
        // counted straight into input order (self-loops keep their 0)
        ws.tinst.ensure(8 * (size_t)ix.m_input + 8);
        if (ix.m_input > 0) {
            k_fill<unsigned long long><<<grid_for(ix.m_input, BLK, PERSIST_BLOCKS), BLK, 0, s>>>(
                ws.tinst.as<unsigned long long>(), 0ull, ix.m_input);
            FOLTY_LAUNCHED();
        }
    }
    const bool one = ix.one_pass_at(q.delta);
    CandBuf B{};
    FOLTY_HIP(hipEventRecord(ws.ev[4], s));
    if (ix.NI > 0) {
        B = filter_triangles(ix, q.variant, q.delta, ws, s, one);
        FOLTY_HIP(hipEventRecord(ws.ev[5], s));
        const int64_t chunks = ws.kept_chunks;
        if (chunks > 0) {
            ws.tflag.ensure(64 * (size_t)B.regions * (size_t)B.per_region);
            k_triad_clear<<<chunk_grid(chunks), BLK, 0, s>>>(B, ws.tflag.as<uint32_t>());
            FOLTY_LAUNCHED();
            TriadOut o{q.delta, ws.tflag.as<uint32_t>(), edge ? ws.tinst.as<unsigned long long>() : nullptr,
                       ix.perm.as<int32_t>()};
            const uint32_t dq = run_slack(range_slack(q.delta, ix.tshift));
            dispatch_variant(q.variant, [&](auto V) {
                constexpr int VAR = decltype(V)::value;
                const int32_t *sv = ws.sv.as<int32_t>();
                const EdgeRec *rec = ix.rec.as<EdgeRec>();
                if (inst) launch_tests(ws, B, TriadRunner<VAR, true>{dq, ix.ts.as<int64_t>(), o, tot, sv, rec}, chunks, s);
                else launch_tests(ws, B, TriadRunner<VAR, false>{dq, ix.ts.as<int64_t>(), o, tot, sv, rec}, chunks, s);
            });
            FOLTY_LAUNCHED();
            k_triad_count<<<chunk_grid(chunks), BLK, 0, s>>>(B, ws.tflag.as<uint8_t>(), nullptr, tot + 2);
            FOLTY_LAUNCHED();
        }
    } else {
        FOLTY_HIP(hipEventRecord(ws.ev[5], s));
    }
    FOLTY_HIP(hipEventRecord(ws.ev[2], s));
    read_scalars(ws, s, false);
    FOLTY_HIP(hipStreamSynchronize(s));
    if (ix.NI > 0) after_filter(ix, ws, q.delta, one);
    else ix.T = 0;
    const unsigned long long *h = ws.host.as<unsigned long long>() + SCAL_TRIAD;
    if (h[1] || h[0] > (unsigned long long)INT64_MAX)
        fail(FOLTY_EOVERFLOW, "the temporal triangles number 2^63 or more");
    res->n_triads = (int64_t)h[2];
    res->n_tinst = inst ? (int64_t)h[0] : -1;
    if ((q.flags & FOLTY_TRIAD_TRIPLES) && res->n_triads > 0)
        list_triples(ix, ws, B, chunks_taken(ws, B), res->n_triads, res.get(), s);
    FOLTY_HIP(hipEventRecord(ws.ev[3], s));
    if (edge) {
        res->tinst.resize((size_t)ix.m_input);
        if (ix.m_input > 0)
            FOLTY_HIP(hipMemcpyAsync(res->tinst.data(), ws.tinst.p, 8 * (size_t)ix.m_input, hipMemcpyDeviceToHost,
                                     s));
    }
    FOLTY_HIP(hipStreamSynchronize(s));
    fill_stats_from_index(ix, &res->stats);
    res->stats.tests = region_sum(ws, REGION_TESTS);
    res->stats.wedge_ms = ev_ms(ws.ev[4], ws.ev[5]);
    res->stats.temporal_ms = ev_ms(ws.ev[5], ws.ev[2]);
    res->stats.threshold_ms = ev_ms(ws.ev[2], ws.ev[3]);
    res->stats.query_ms = ev_ms(ws.ev[0], ws.ev[3]);
    res->stats.filter_passes = ix.NI > 0 ? ws.filter_passes : 0;
    return res.release();
}

} // namespace folty
