// Query kernels for the thresholded exists-exists-forall triadic query.
//
//  a.5  wedge enumeration + closing probe (paper, Algorithm OutNeighbours:
//       (u, v) in G->_pi and w in N+(u), test whether v and w are adjacent).
//       Each oriented edge (u, v) probes the shorter of N+(v) and the part of
//       N+(u) past v for membership in the other's row, which its wavefront holds
//       as a hash table in LDS.  Each static triangle is found once, from its
//       lowest-ranked vertex, as three oriented edges.
//  a.6  temporal tests (paper, Theorems 3.1 and 3.2): a temporal edge e on list
//       L1 forms a delta-temporal triangle with the third vertex w iff, with
//       t2 = the first entry of L2 at or after t(e) and t3 = the first entry of
//       L3 at or after t2, both exist and t3 - t(e) <= delta.  The first-entry
//       searches are binary searches over the time-sorted lists (the log
//       sigma_max factor).  A (triangle, directed list) pair is a run of tests.
//       A run is skipped when the time ranges of its three lists already rule
//       out t <= t2 <= t3 <= t + delta (a necessary condition, so no result
//       changes).  The tests left are spread over the lanes of the wavefront
//       that holds their triangles, or in pieces over the chip.
//  a.7  threshold (paper, Algorithm ExistExistForAll, final loop) with the exact
//       rational theta, then per-pair certificate counts by a wavefront
//       segmented reduction and a ballot/prefix compaction of the pairs.
#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>

#include "tri_device.h"

namespace folty {

namespace {

// ---------------------------------------------------------------------------
// index helpers
// ---------------------------------------------------------------------------
// The records of the static edges in their own order, lists lo -> hi first:
// soff, smid and the lists' end timestamps are read in the order they are
// stored, so this pass streams.
__global__ void k_static_recs(const int32_t *__restrict__ soff, const int32_t *__restrict__ smid,
                              const int64_t *__restrict__ ts, int32_t S, int32_t tshift,
                              EdgeRec *__restrict__ srec) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= S) return;
    const int32_t a = soff[e], mid = smid[e], b = soff[e + 1];
    EdgeRec r;
    r.fs = a;
    r.fn = mid - a;
    r.bs = mid;
    r.bn = b - mid;
    r.flo = r.fn ? (uint32_t)(ts[a] >> tshift) : 0;
    r.fhi = r.fn ? (uint32_t)(ts[mid - 1] >> tshift) : 0;
    r.blo = r.bn ? (uint32_t)(ts[mid] >> tshift) : 0;
    r.bhi = r.bn ? (uint32_t)(ts[b - 1] >> tshift) : 0;
    srec[e] = r;
}

// Oriented edge p (static edge e, tail lo when bit 31 of its id is set): one
// 32-byte read of e's record, lists swapped when the tail is hi.  shift: the
// ranges' shift beyond the records' own.
__global__ void k_edge_recs(const uint32_t *__restrict__ oeid, const EdgeRec *__restrict__ srec, int32_t S,
                            int32_t shift, uint32_t rbase, EdgeRec *__restrict__ rec,
                            uint2 *__restrict__ erng) {
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= S) return;
    const uint32_t id = oeid[p];
    const EdgeRec q = srec[id & 0x7fffffffu];
    EdgeRec r = q;
    if (!(id >> 31)) {
        r.fs = q.bs, r.fn = q.bn, r.flo = q.blo, r.fhi = q.bhi;
        r.bs = q.fs, r.bn = q.fn, r.blo = q.flo, r.bhi = q.fhi;
    }
    rec[p] = r;
    erng[p] = make_uint2(r.fn ? rng_pack(rng_code(r.flo, rbase, shift), rng_code(r.fhi, rbase, shift)) : RNG_EMPTY,
                         r.bn ? rng_pack(rng_code(r.blo, rbase, shift), rng_code(r.bhi, rbase, shift)) : RNG_EMPTY);
}

// Probe segments: for the oriented edge (u, v) at position p, the candidates
// x > v are the entries of N+(v), or those of N+(u) past p; the shorter list is
// the segment (mode A or B), and the other row's vertex owns it.  Sort key: the
// owner; an edge with an empty side closes no triangle and gets key n, past all
// owners.
__global__ void k_seg_keys(const int32_t *__restrict__ ooff, const int32_t *__restrict__ oadj,
                           const int32_t *__restrict__ otail, int32_t S, int32_t n, uint32_t *__restrict__ key,
                           uint32_t *__restrict__ val) {
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= S) return;
    const int32_t u = otail[p], v = oadj[p];
    const int32_t past = ooff[u + 1] - 1 - (int32_t)p, dv = ooff[v + 1] - ooff[v];
    const bool mode_b = past < dv;
    key[p] = past == 0 || dv == 0 ? (uint32_t)n : (uint32_t)(mode_b ? v : u);
    val[p] = (uint32_t)p | (mode_b ? MODE_B : 0u);
}

// seg[j] = (segment start, length, oriented edge | mode B << 31, 0), with its ranges;
// run[w] = the owner's first segment and the one past its last (owners without
// segments are not written and never read); *ng = segments
__global__ void k_seg_recs(const uint32_t *__restrict__ key, const uint32_t *__restrict__ val,
                           const int32_t *__restrict__ ooff, const int32_t *__restrict__ oadj,
                           const int32_t *__restrict__ otail, const uint2 *__restrict__ erng, int32_t S, int32_t n,
                           int4 *__restrict__ seg, uint2 *__restrict__ srng, int32_t *__restrict__ owner, int32_t *__restrict__ len, int2 *__restrict__ run, int32_t *__restrict__ ng) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= S) return;
    const uint32_t k = key[j];
    const bool first = j == 0 || key[j - 1] != k;
    if (k == (uint32_t)n) {
        if (first) *ng = (int32_t)j;
        len[j] = 0;
        return;
    }
    const uint32_t id = val[j];
    const int32_t p = (int32_t)(id & ~MODE_B);
    int32_t rs, re;
    if (id & MODE_B) {
        rs = p + 1;
        re = ooff[otail[p] + 1];
    } else {
        const int32_t v = oadj[p];
        rs = ooff[v];
        re = ooff[v + 1];
    }
    seg[j] = make_int4(rs, re - rs, (int32_t)id, 0);
    srng[j] = erng[p];
    owner[j] = (int32_t)k;
    len[j] = re - rs;
    if (first) run[k].x = (int32_t)j;
    if (j == S - 1 || key[j + 1] != k) {
        run[k].y = (int32_t)j + 1;
        if (j == S - 1) *ng = S;
    }
}

// Owners with fewer than LOOSE_PROBES probes share items (their rows are searched
// in global memory, so a wavefront's 64 lanes are filled across owners); the
// others have items of their own.
constexpr int64_t LOOSE_PROBES = 128;
constexpr int64_t LOOSE_CHUNK = 1024;
static_assert(LOOSE_CHUNK + LOOSE_PROBES <= CHUNK + CAP, "a loose item's probes fit the marks");

// An item starts at the first segment of each owner with items of its own and
// of each run of loose owners, and wherever the run's probe count crosses a
// multiple of CHUNK or its segment count a multiple of ITEM_SEGS (loose runs: the
// global counts, and LOOSE_CHUNK); both indices only grow, so segments of equal
// value are contiguous.
__global__ void k_item_flags(const uint32_t *__restrict__ key, const int64_t *__restrict__ P,
                             const int2 *__restrict__ run, int32_t G, int32_t *__restrict__ flag) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= G) return;
    const int2 r = run[key[j]];
    const int64_t Pj = P[j], P0 = P[r.x];
    const bool loose = P[r.y] - P0 < LOOSE_PROBES;
    int f = j == 0;
    if (j > 0) {
        const int64_t Pp = P[j - 1];
        if (loose) {
            f = Pj / LOOSE_CHUNK != Pp / LOOSE_CHUNK || j % ITEM_SEGS == 0;
            if (!f && j == r.x) {
                const int2 rp = run[key[j - 1]];
                f = P[rp.y] - P[rp.x] >= LOOSE_PROBES;
            }
        } else {
            f = j == r.x ||
                (Pj - P0) / CHUNK + (j - r.x) / ITEM_SEGS != (Pp - P0) / CHUNK + (j - 1 - r.x) / ITEM_SEGS;
        }
    }
    flag[j] = f;
}

__global__ void k_item_starts(const int32_t *__restrict__ flag, const int32_t *__restrict__ fid, int32_t G,
                              int32_t *__restrict__ start) {
    int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < G && flag[j]) start[fid[j] - 1] = (int32_t)j;
}

__global__ void k_items(const int32_t *__restrict__ start, const int32_t *__restrict__ owner, const int64_t *__restrict__ P,
                        const int2 *__restrict__ run, const int32_t *__restrict__ ooff, int32_t NI,
                        EnumItem *__restrict__ items) {
    int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (it >= NI) return;
    const int32_t g0 = start[it], g1 = start[it + 1];
    const int32_t w = owner[g0];
    const int2 r = run[w];
    EnumItem e{};
    e.g0 = g0;
    e.ng = g1 - g0;
    e.nq = (int32_t)(P[g1] - P[g0]);
    e.b = ooff[w];
    e.d = P[r.y] - P[r.x] < LOOSE_PROBES ? -1 : ooff[w + 1] - e.b;
    items[it] = e;
}

// ---------------------------------------------------------------------------
// a.7 threshold + per-pair certificate counts
// ---------------------------------------------------------------------------
struct ThreshArgs {
    const uint32_t *count;
    const int32_t *sid, *smid, *slo, *shi, *deg, *tcnt;
    int32_t m;
    uint32_t num, den;
    int universe, excl;
    int zero_never;                  // theta > 0 and |U| >= 1 for every edge: count 0 never certifies
    int any;                         // the inner exists of a vertex query: count >= 1 qualifies
    uint32_t *ncert;                 // [2S]: 2 s + dir
    unsigned long long *scal;        // the query's scalars (certificates per region)
};

// A block takes many tiles of edges, so that its one atomic on the certificate
// total is a rare one.
constexpr int64_t THRESHOLD_BLOCKS = 8192;
__global__ __launch_bounds__(BLK) void k_threshold(ThreshArgs A) {
    __shared__ unsigned long long s_tot[BLK / 64];
    unsigned long long sum = 0;
    for (int64_t k0 = (int64_t)blockIdx.x * BLK; k0 < A.m; k0 += (int64_t)gridDim.x * BLK) {
        const int64_t k = k0 + threadIdx.x;
        bool in = k < A.m;
        int64_t key = -1;
        bool cert = false;
        const uint32_t cnt = in ? A.count[k] : 0u;
        // a wavefront whose edges all count 0 has no certificate when 0 cannot
        // reach theta * |U|
        if (A.zero_never && !__ballot(cnt != 0u)) continue;
        if (in) {
            int32_t s = A.sid[k];
            int dir = k >= A.smid[s] ? 1 : 0;
            if (A.any) {
                cert = cnt >= 1u;
            } else if (cnt != 0u || !A.zero_never) {
                int32_t a = dir ? A.shi[s] : A.slo[s];
                int32_t b = dir ? A.slo[s] : A.shi[s];
                int64_t U;
                if (A.universe == FOLTY_UNIVERSE_DST) U = (int64_t)A.deg[b] - A.excl;
                else if (A.universe == FOLTY_UNIVERSE_SRC) U = (int64_t)A.deg[a] - A.excl;
                else U = A.tcnt[s];
                cert = (uint64_t)cnt * A.den >= (uint64_t)A.num * (uint64_t)U;
            }
            key = 2 * (int64_t)s + dir;
        }
        // segmented count of certificates over runs of equal keys inside the wave
        int lane = lane_id();
        int64_t prev = __shfl_up(key, 1);
        int64_t next = __shfl_down(key, 1);
        bool head = lane == 0 || prev != key;
        bool tail = lane == 63 || next != key;
        unsigned long long heads = __ballot(head && in);
        unsigned long long certs = __ballot(cert);
        if (in && tail) {
            unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
            unsigned long long h = heads & upto;
            int start = 63 - __clzll((long long)h);
            unsigned long long seg = upto & ~((1ull << start) - 1ull);
            int c = __popcll(certs & seg);
            if (c) atomicAdd(&A.ncert[key], (uint32_t)c);
        }
        sum += (unsigned long long)__popcll(certs);
    }
    if (lane_id() == 0) s_tot[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int i = 0; i < BLK / 64; i++) t += s_tot[i];
        if (t) region_add(A.scal, REGION_CERTS, t);
    }
}

// bits of a vertex id in a pair key (at least 1)
__host__ __device__ inline int pair_bits(int32_t n) {
    int b = 1;
    while (b < 31 && ((int64_t)1 << b) < (int64_t)n) b++;
    return b;
}

// Directed pairs with certificates, as keys (a << nbits) | b with their counts.
// Each block takes BLK x PAIR_ITEMS entries (2 s + dir) and claims its output
// range with one atomic, so a dense result does not serialise on the counter.
constexpr int PAIR_ITEMS = 32;
__global__ __launch_bounds__(BLK) void k_pairs_compact(const uint32_t *__restrict__ ncert, int32_t S,
                                                       const int32_t *__restrict__ slo, const int32_t *__restrict__ shi,
                                                       int nbits, uint64_t *__restrict__ keys,
                                                       uint32_t *__restrict__ vals, int32_t *__restrict__ npairs) {
    __shared__ int32_t s_wave[BLK / 64];
    __shared__ int32_t s_base;
    const int64_t n2 = 2 * (int64_t)S;
    const int64_t tile = (int64_t)blockIdx.x * BLK * PAIR_ITEMS;
    uint32_t c[PAIR_ITEMS];
    int32_t mine = 0;
#pragma unroll
    for (int j = 0; j < PAIR_ITEMS; j++) {
        const int64_t i = tile + (int64_t)j * BLK + threadIdx.x;
        c[j] = i < n2 ? ncert[i] : 0u;
        mine += c[j] > 0;
    }
    const int w = threadIdx.x >> 6;
    const int32_t incl = wave_inclusive_sum(mine);
    if (lane_id() == 63) s_wave[w] = incl;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t tot = 0;
        for (int k = 0; k < BLK / 64; k++) {
            const int32_t x = s_wave[k];
            s_wave[k] = tot;
            tot += x;
        }
        s_base = tot ? atomicAdd(npairs, tot) : 0;
    }
    __syncthreads();
    int32_t pos = s_base + s_wave[w] + incl - mine;
#pragma unroll
    for (int j = 0; j < PAIR_ITEMS; j++) {
        if (!c[j]) continue;
        const int64_t i = tile + (int64_t)j * BLK + threadIdx.x;
        const int32_t e = (int32_t)(i >> 1);
        const uint64_t a = (uint64_t)((i & 1) ? shi[e] : slo[e]);
        const uint64_t b = (uint64_t)((i & 1) ? slo[e] : shi[e]);
        keys[pos] = (a << nbits) | b;
        vals[pos] = c[j];
        pos++;
    }
}

__global__ void k_pairs_unpack(const uint64_t *__restrict__ keys, int32_t np, int nbits, int32_t *__restrict__ u,
                               int32_t *__restrict__ v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= np) return;
    const uint64_t k = keys[i];
    u[i] = (int32_t)(k >> nbits);
    v[i] = (int32_t)(k & ((1ull << nbits) - 1));
}

// Sorts a small result (at most SMALL_PAIRS pairs, otherwise nothing is done): one
// block, each pair's rank counted against all keys in LDS, u, v and the
// certificates written behind the scalars.  Launched before the host knows the
// number of pairs, so a small query is one stream of launches and one copy.
constexpr int SMALL_BLK = 1024;
__global__ __launch_bounds__(SMALL_BLK) void k_pairs_small(const uint64_t *__restrict__ keys,
                                                           const uint32_t *__restrict__ vals,
                                                           const int32_t *__restrict__ npairs, int nbits,
                                                           int32_t *__restrict__ out) {
    __shared__ uint64_t s_k[SMALL_PAIRS];
    static_assert(SMALL_PAIRS == SMALL_BLK, "a pair per thread");
    const int np = *npairs, i = threadIdx.x;
    if (np > SMALL_PAIRS) return;
    const uint64_t k = i < np ? keys[i] : ~0ull;
    s_k[i] = k;
    __syncthreads();
    if (i >= np) return;
    int r = 0;
    for (int j = 0; j < np; j++) r += s_k[j] < k; // keys differ
    out[r] = (int32_t)(k >> nbits);
    out[SMALL_PAIRS + r] = (int32_t)(k & ((1ull << nbits) - 1));
    out[2 * SMALL_PAIRS + r] = (int32_t)vals[i];
}

// count[e] += the prefix sum of the interval marks at e
__global__ void k_add_counts(const int32_t *__restrict__ ps, int32_t m, uint32_t *__restrict__ count) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x)
        count[e] += (uint32_t)ps[e];
}

__global__ void k_counts_scatter(const uint32_t *__restrict__ count, const int32_t *__restrict__ perm, int32_t m,
                                 uint32_t *__restrict__ out) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < m) out[perm[k]] = count[k];
}

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------

} // namespace

double ev_ms(hipEvent_t a, hipEvent_t b) {
    float ms = 0;
    FOLTY_HIP(hipEventElapsedTime(&ms, a, b));
    return ms;
}

namespace {

unsigned enum_grid(int32_t n) {
    int64_t g = ((int64_t)n + WPB - 1) / WPB;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(g, ENUM_BLOCKS));
}

// clears per-edge counts, per-pair counts and the query's scalars in one launch
__global__ __launch_bounds__(BLK) void k_query_clear(uint32_t *__restrict__ count, int64_t m,
                                                     uint32_t *__restrict__ ncert, int64_t np,
                                                     unsigned long long *__restrict__ scal) {
    const int64_t i0 = (int64_t)blockIdx.x * BLK + threadIdx.x, stride = (int64_t)gridDim.x * BLK;
    uint4 *c4 = reinterpret_cast<uint4 *>(count), *n4 = reinterpret_cast<uint4 *>(ncert);
    const uint4 zero = make_uint4(0, 0, 0, 0);
    for (int64_t i = i0; i < (m + 3) / 4; i += stride) c4[i] = zero;
    for (int64_t i = i0; i < (np + 3) / 4; i += stride) n4[i] = zero;
    for (int64_t i = i0; i < SCAL_WORDS; i += stride) scal[i] = 0;
}

} // namespace

// makes the workspace's scalars, and per-edge and per-pair counts if asked for,
// and clears them
void clear_query(const Index &ix, Workspace &ws, bool counts, hipStream_t s) {
    ws.scal.ensure(SCAL_ALL_BYTES);
    ws.host.ensure(SCAL_ALL_BYTES);
    int64_t m = 0, np = 0;
    if (counts) {
        m = ix.m;
        np = 2 * (int64_t)ix.S;
        ws.count.ensure(4 * (size_t)m + 16);
        ws.ncert.ensure(4 * (size_t)np + 16);
    }
    const int64_t n4 = std::max<int64_t>((std::max(m, np) + 3) / 4, SCAL_WORDS);
    k_query_clear<<<grid_for(n4, BLK, 8192), BLK, 0, s>>>(ws.count.as<uint32_t>(), m, ws.ncert.as<uint32_t>(), np,
                                                          ws.scal.as<unsigned long long>());
    FOLTY_LAUNCHED();
}

// the query's scalars (and a small result's pairs) into ws.host; read them after
// the stream is synchronised
void read_scalars(Workspace &ws, hipStream_t s, bool pairs) {
    FOLTY_HIP(hipMemcpyAsync(ws.host.p, ws.scal.p, pairs ? SCAL_ALL_BYTES : SCAL_BYTES, hipMemcpyDeviceToHost, s));
}

int64_t chunks_taken(const Workspace &ws, const CandBuf &B) {
    const uint32_t *c = reinterpret_cast<const uint32_t *>(ws.host.as<unsigned long long>() + SCAL_REGIONS);
    int64_t k = 0;
    for (int r = 0; r < B.regions; r++) k += std::min<int64_t>(c[r * CAND_STRIDE], B.per_region);
    return k;
}

// the sum of a counter over the regions
int64_t region_sum(const Workspace &ws, int what) {
    const unsigned long long *h = ws.host.as<unsigned long long>() + SCAL_REGIONS;
    unsigned long long k = 0;
    for (int r = 0; r < MAX_REGIONS; r++) k += h[r * REGION_WORDS + what];
    return (int64_t)k;
}

namespace {

// Up to this many chunks (50 MB) are allocated whatever the window keeps, so that
// no pass has to be repeated and the host reads nothing back in between.
constexpr int64_t SAFE_CHUNKS = 1 << 16;

// Chunks allocated at first for a graph of at most `triangles` triangles, in a
// workspace that has some: the safe ones or an eighth of what all would take, and all
// beside a cached list, which is as large (10M edges, the first query without a
// window: 2.13 ms with the pass repeated, now 1.04).  More than the safe ones only
// out of plenty, so that the rest of the query has room, and otherwise none (the
// pass then counts what it needs).
int64_t first_chunks(int64_t triangles, int64_t waves, bool cached, const Workspace &ws) {
    const int64_t most = most_chunks(triangles, waves), have = (int64_t)ws.sv.bytes / (CHUNK_BYTES - 4);
    const int64_t chunks = std::min(most, std::max({SAFE_CHUNKS, cached ? most : most / 8, have}));
    if (chunks > SAFE_CHUNKS && chunks > have) {
        size_t fr = 0, tot = 0;
        if (hipMemGetInfo(&fr, &tot) != hipSuccess) {
            (void)hipGetLastError();
            fr = 0;
        }
        if (chunks * CHUNK_BYTES > (int64_t)((fr + dev_cached()) / 4)) return have;
    }
    return chunks;
}

// What a filter pass goes over: the index's enumeration items, or groups of 64
// cached triangles.
int64_t filter_units(const Index &ix) { return ix.tri_cached ? (ix.T.load() + 63) / 64 : ix.NI; }

// `chunks` of them (or up to one per region more) in the workspace
CandBuf make_chunks(Workspace &ws, unsigned grid, int64_t chunks) {
    CandBuf B{};
    B.regions = (int32_t)std::min<unsigned>(MAX_REGIONS, grid);
    B.per_region = (int32_t)((chunks + B.regions - 1) / B.regions);
    const size_t total = (size_t)B.regions * (size_t)B.per_region;
    ws.sv.ensure((CHUNK_BYTES - 4) * total);
    ws.svn.ensure(4 * total);
    unsigned long long *scal = ws.scal.as<unsigned long long>();
    B.sv = ws.sv.as<int32_t>();
    B.cnt = ws.svn.as<int32_t>();
    B.ctr = reinterpret_cast<uint32_t *>(scal + SCAL_REGIONS);
    B.dropped = reinterpret_cast<uint32_t *>(scal + SCAL_DROPPED);
    ws.kept_chunks = (int64_t)total;
    ws.kept_most = 64 * (int64_t)total;
    return B;
}

// Wavefronts of a bounded workspace's filter when all that it keeps is much: their
// partly filled chunks take at most 36 bytes per item then, and all chunks together
// at most bounded_chunks.
int64_t bounded_waves(const Index &ix) { return std::max<int64_t>(WPB, 36 * (int64_t)ix.NI / CHUNK_BYTES); }
int64_t bounded_chunks(const Index &ix, int64_t T) { return T / 64 + bounded_waves(ix); }

// The filter over units [u0, u0 + nu), which appends to B; T: the triangles, -1 if
// they are counted by this pass.
void launch_filter(const Index &ix, int variant, int64_t dmax, const Workspace &ws, const CandBuf &B, int64_t T,
                   bool one_pass, unsigned grid, int64_t u0, int64_t nu, hipStream_t s) {
    auto run = [&](auto V, auto M) {
        FilterSink<decltype(V)::value, decltype(M)::value> sink{};
        sink.rng = ix.erng.as<uint2>();
        sink.dq = rng_slack(dmax, ix.rshift);
        sink.out = B;
        sink.scal = ws.scal.as<unsigned long long>();
        if (ix.tri_cached) {
            k_filter_cached<<<grid, BLK, 0, s>>>(ix.tri.as<int32_t>() + 192 * u0, std::min(T - 64 * u0, 64 * nu), sink);
        } else {
            EnumGraph G = enum_graph(ix);
            G.item += u0;
            k_tri_enum<<<grid, BLK, 0, s>>>(G, (int32_t)nu, sink);
        }
        FOLTY_LAUNCHED();
    };
    dispatch_variant(variant, [&](auto V) {
        if (T < 0) run(V, std::integral_constant<FilterMode, FILTER_COUNT>{});
        else if (one_pass) run(V, std::integral_constant<FilterMode, FILTER_WIDE>{});
        else run(V, std::integral_constant<FilterMode, FILTER_NARROW>{});
    });
}

// the chunks are free again; the other scalars stay
__global__ void k_chunks_reset(unsigned long long *__restrict__ scal) {
    const int i = threadIdx.x;
    if (i < MAX_REGIONS) scal[SCAL_REGIONS + i * REGION_WORDS + REGION_CHUNKS] = 0;
    if (i == 0) scal[SCAL_DROPPED] = scal[SCAL_HEAVY] = 0;
}
void reset_chunks(Workspace &ws, hipStream_t s) {
    k_chunks_reset<<<1, MAX_REGIONS, 0, s>>>(ws.scal.as<unsigned long long>());
    FOLTY_LAUNCHED();
}

} // namespace

// a.5 for one predicate code and window bound: one pass over the enumeration
// items (or the cached triangles) appends the triangles it keeps to the
// workspace's chunks.  The first pass over an index also counts its triangles.
// When the chunks do not suffice, or there is no memory for the first of them, they
// grow to what the pass would have needed and it is repeated.  The scalars have
// been cleared.
CandBuf filter_triangles(Index &ix, int variant, int64_t dmax, Workspace &ws, hipStream_t s, bool one_pass) {
    int64_t T = ix.T.load();
    const int64_t units = filter_units(ix);
    unsigned grid = enum_grid((int32_t)std::min<int64_t>(units, INT32_MAX));
    const int64_t waves = std::min<int64_t>((int64_t)grid * WPB, units);
    int64_t most = most_chunks(T >= 0 ? T : ix.probes, waves);
    int64_t chunks = first_chunks(T >= 0 ? T : ix.probes, waves, ix.tri_cached, ws);
    // a bounded workspace takes no more than query_footprint says, or keeps what it has
    const int64_t bound = !ws.bounded || T < 0
                              ? INT64_MAX
                              : std::max(bounded_chunks(ix, T), (int64_t)ws.sv.bytes / (CHUNK_BYTES - 4));
    chunks = std::min(chunks, bound);
    for (bool counted = false;; counted = true) {
        CandBuf B;
        try {
            B = make_chunks(ws, grid, chunks);
        } catch (const Error &e) {
            if (e.code != FOLTY_ENOMEM || counted) throw;
            chunks = 0;
            B = make_chunks(ws, grid, 0);
        }
        if (T >= 0) ws.kept_most = std::min(ws.kept_most, T);
        launch_filter(ix, variant, dmax, ws, B, T, one_pass, grid, 0, units, s);
        // (a cached list's many chunks are mostly not taken: the tests' grids follow their number)
        if (chunks >= most && !(ix.tri_cached && chunks > SAFE_CHUNKS)) return B;
        read_scalars(ws, s, false);
        FOLTY_HIP(hipStreamSynchronize(s));
        const unsigned long long *h = ws.host.as<unsigned long long>();
        const int64_t taken = chunks_taken(ws, B);
        const uint32_t dropped = (uint32_t)h[SCAL_DROPPED];
        ws.kept_chunks = taken;
        ws.kept_most = std::min(ws.kept_most, 64 * taken);
        if (dropped == 0) return B;
        if (T < 0) {
            T = region_sum(ws, REGION_HITS);
            ix.T = T;
        }
        chunks = taken + (int64_t)dropped;
        if (chunks > bound) { // fewer wavefronts, and then every triangle fits
            grid = (unsigned)(bounded_waves(ix) / WPB);
            most = chunks = most_chunks(T, (int64_t)grid * WPB);
        }
        reset_chunks(ws, s);
    }
}

namespace {

// The filter and the tests with a fixed scratch: chunks take what is left of it,
// and when they do not suffice the units are gone over in parts (the tests add up
// in the per-edge counts, so any split gives the same), each half as long as what
// did not fit or less.  Afterwards the chunks' part of the scratch is free again.
constexpr unsigned ARENA_ENUM_BLOCKS = 1024; // fewer partly filled chunks
template <class Tests>
void filter_in_arena(Index &ix, const folty_query &q, Workspace &ws, hipStream_t s, bool one_pass, const Tests &tests) {
    int64_t T = ix.T.load();
    const int64_t units = filter_units(ix);
    const size_t mark = arena_mark();
    auto free_chunks = [&] {
        ws.sv.forget();
        ws.svn.forget();
        ws.pieces.forget();
        arena_rewind(mark);
        reset_chunks(ws, s);
    };
    for (int64_t u0 = 0, step = units; u0 < units;) {
        const int64_t nu = std::min(step, units - u0), left = arena_left();
        // the list of heavy triangles takes what the chunks leave
        const int64_t room = (left - std::max<int64_t>(left / 16, 1024)) / CHUNK_BYTES;
        // half of the chunks may be partly filled, one by each wavefront
        const unsigned grid = (unsigned)std::max<int64_t>(
            1, std::min({(int64_t)enum_grid((int32_t)std::min<int64_t>(nu, INT32_MAX)), (int64_t)ARENA_ENUM_BLOCKS,
                         room / (2 * WPB)}));
        const int64_t most = most_chunks(T >= 0 ? T : ix.probes, std::min<int64_t>((int64_t)grid * WPB, nu));
        // make_chunks gives every region as many
        const int64_t chunks = std::min(most, room + 1 - std::min<int64_t>(MAX_REGIONS, grid));
        if (chunks < most && chunks < 1)
            fail(FOLTY_ENOMEM, "this call needs more than its fixed device scratch: %lld bytes are left for triangles",
                 (long long)left);
        const CandBuf B = make_chunks(ws, grid, chunks);
        launch_filter(ix, q.variant, q.delta, ws, B, T, one_pass, grid, u0, nu, s);
        if (chunks < most) {
            read_scalars(ws, s, false);
            FOLTY_HIP(hipStreamSynchronize(s));
            if (T < 0) { // the first part is all of it
                T = region_sum(ws, REGION_HITS);
                ix.T = T;
            }
            const uint32_t dropped = (uint32_t)ws.host.as<unsigned long long>()[SCAL_DROPPED];
            if (dropped) {
                const int64_t need = chunks_taken(ws, B) + dropped;
                if (nu == 1)
                    fail(FOLTY_ENOMEM, "this call needs more than its fixed device scratch: %lld bytes for one part of "
                         "the triangles, %lld left", (long long)(need * CHUNK_BYTES), (long long)left);
                step = std::max<int64_t>(1, std::min(nu / 2, nu * chunks / (2 * need)));
                free_chunks();
                continue;
            }
        }
        if (ws.kept_chunks > 0) tests(B);
        free_chunks();
        u0 += nu;
    }
}

} // namespace

// After the query's scalars are on the host: the number of triangles on the first
// query, the filter's passes, and the switch to one pass for later queries.
// By default the filter tests a probe's two known edges first and the whole
// triangle after (two passes).  When a window keeps at least one triangle in 12,
// the first test drops too little, and later queries of about that window or wider
// (from half of it) look every probe up and test triangles once.  Filter with two
// passes and one: 70M edges, 1 hour 1.28 and 3.45 ms (none kept), 1 year 3.41 and
// 3.95 ms (0.028 kept); 10M edges of the medium graph, 4 weeks 0.18 and 0.25 ms
// (0.005), 13 weeks 0.26 and 0.28 ms (0.05), half a year 0.34 and 0.29 ms (0.15), 1
// year 0.40 and 0.31 ms (0.30); 10M uniform edges 0.10 and 0.07 ms (0.34-0.44).
// The rule depends only on the graph and the queries, never on timing.
void after_filter(Index &ix, Workspace &ws, int64_t delta, bool one_pass) {
    if (ix.T.load() < 0) ix.T = region_sum(ws, REGION_HITS);
    const int64_t kept = region_sum(ws, REGION_KEPT);
    ws.filter_passes = one_pass ? 1 : 2;
    if (!one_pass && kept > 0 && 12 * kept >= ix.T.load() &&
        delta / 2 < ix.one_pass_from.load(std::memory_order_relaxed))
        ix.one_pass_from.store(delta / 2, std::memory_order_relaxed);
}

bool use_one_pass(Graph *g, const folty_query &q) {
    if (q.flags & FOLTY_QUERY_ONE_PASS) {
        ensure_triangles(g);
        return true;
    }
    return g->ix.one_pass_at(q.delta);
}

namespace {

// per-edge counts of the kept triangles' runs (a.6)
template <bool SS>
void launch_temporal(const Index &ix, int variant, int64_t dmax, Workspace &ws, const CandBuf &B, const DirectOp &op,
                     hipStream_t s) {
    const uint32_t dq = run_slack(range_slack(dmax, ix.tshift));
    dispatch_variant(variant, [&](auto V) {
        launch_tests(ws, B,
                     CountRunner<decltype(V)::value, DirectOp, SS>{dq, ix.ts.as<int64_t>(), op, ws.sv.as<int32_t>(),
                                                                   ix.rec.as<EdgeRec>(), ix.tshift == 0},
                     ws.kept_chunks, s);
    });
}

// threshold + pairs for one query given device counts (sorted edge order)
// ---------------------------------------------------------------------------
// vertex queries: per vertex u, its neighbours v with a qualifying edge u -> v
// ---------------------------------------------------------------------------
// good[u] = the pairs (u, v), from the result's pairs sorted by u: the last pair
// of a run writes its length (no atomics: a hub's thousands of pairs would queue at
// one address; 1.4M pairs 0.31 ms, now 0.01 ms)
__global__ void k_vertex_starts(const int32_t *__restrict__ pu, int32_t np, uint32_t *__restrict__ good) {
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < np && (i == 0 || pu[i - 1] != pu[i])) good[pu[i]] = (uint32_t)i;
}
__global__ void k_vertex_good(const int32_t *__restrict__ pu, int32_t np, uint32_t *__restrict__ good) {
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < np && (i == np - 1 || pu[i + 1] != pu[i])) good[pu[i]] = (uint32_t)i + 1 - good[pu[i]];
}

// u is a solution: |N(u)| >= 1 and good[u] * den >= num * |N(u)|
__global__ void k_vertex_flags(const uint32_t *__restrict__ good, const int32_t *__restrict__ deg, int32_t n,
                               uint32_t num, uint32_t den, int32_t *__restrict__ flag) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n) return;
    const int32_t d = deg[u];
    flag[u] = d >= 1 && (uint64_t)good[u] * den >= (uint64_t)num * (uint64_t)d;
}

// the solutions in id order, at their exclusive-scan positions
__global__ void k_vertex_compact(const int32_t *__restrict__ flag, const int32_t *__restrict__ pos,
                                 const uint32_t *__restrict__ good, int32_t n, int32_t *__restrict__ vert,
                                 uint32_t *__restrict__ vgood) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= n || !flag[u]) return;
    vert[pos[u]] = (int32_t)u;
    vgood[pos[u]] = good[u];
}

// the vertex step after the edge-level threshold (pu: its np pairs' first vertices,
// ascending)
void finish_vertex(const Graph *g, const folty_vertex_query &vq, Workspace &ws, const int32_t *pu, int32_t np,
                   Result *res, hipStream_t s) {
    const Index &ix = g->ix;
    const int32_t n = ix.n;
    ws.vtmp.ensure(20 * (size_t)n + 16);
    uint32_t *good = ws.vtmp.as<uint32_t>();
    int32_t *flag = reinterpret_cast<int32_t *>(good + n);
    int32_t *pos = flag + n;
    int32_t *vert = pos + n;
    uint32_t *vgood = reinterpret_cast<uint32_t *>(vert + n);
    k_fill<uint32_t><<<grid_for(n, BLK), BLK, 0, s>>>(good, 0u, n);
    FOLTY_LAUNCHED();
    if (np > 0) {
        k_vertex_starts<<<grid_for(np, BLK), BLK, 0, s>>>(pu, np, good);
        k_vertex_good<<<grid_for(np, BLK), BLK, 0, s>>>(pu, np, good);
        FOLTY_LAUNCHED();
    }
    k_vertex_flags<<<grid_for(n, BLK), BLK, 0, s>>>(good, ix.deg.as<int32_t>(), n, vq.theta_num, vq.theta_den, flag);
    FOLTY_LAUNCHED();
    size_t need = exclusive_scan_i32(nullptr, 0, flag, pos, n, s);
    ws.cub.ensure(need);
    exclusive_scan_i32(ws.cub.p, need, flag, pos, n, s);
    k_vertex_compact<<<grid_for(n, BLK), BLK, 0, s>>>(flag, pos, good, n, vert, vgood);
    FOLTY_LAUNCHED();
    int32_t *last = reinterpret_cast<int32_t *>(ws.host.as<char>() + SCAL_BYTES); // the pairs have been taken
    FOLTY_HIP(hipMemcpyAsync(&last[0], pos + n - 1, 4, hipMemcpyDeviceToHost, s));
    FOLTY_HIP(hipMemcpyAsync(&last[1], flag + n - 1, 4, hipMemcpyDeviceToHost, s));
    FOLTY_HIP(hipStreamSynchronize(s));
    const int32_t nv = last[0] + last[1];
    res->vert.resize(nv);
    res->vgood.resize(nv);
    if (nv > 0) {
        FOLTY_HIP(hipMemcpyAsync(res->vert.data(), vert, 4 * (size_t)nv, hipMemcpyDeviceToHost, s));
        FOLTY_HIP(hipMemcpyAsync(res->vgood.data(), vgood, 4 * (size_t)nv, hipMemcpyDeviceToHost, s));
        FOLTY_HIP(hipStreamSynchronize(s));
    }
}

struct PairCounts {
    int64_t ncerts;
    int32_t npairs;
};

// Threshold step: certificates, per-pair certificate counts and the compacted
// pair keys (unsorted, in ws); a small result is sorted behind the scalars.
// any: qualify edges with count >= 1 (the inner exists of a vertex query)
void threshold_pairs(const Graph *g, const folty_query &q, const uint32_t *count, Workspace &ws,
                           hipStream_t s, bool any) {
    const Index &ix = g->ix;
    const int32_t S = ix.S, m = ix.m;
    int32_t *np = reinterpret_cast<int32_t *>(ws.scal.as<unsigned long long>() + SCAL_PAIRS);
    if (m > 0) {
        ThreshArgs A;
        A.count = count;
        A.sid = ix.sid.as<int32_t>();
        A.smid = ix.smid.as<int32_t>();
        A.slo = ix.slo.as<int32_t>();
        A.shi = ix.shi.as<int32_t>();
        A.deg = ix.deg.as<int32_t>();
        A.tcnt = ix.tcnt.as<int32_t>();
        A.m = m;
        A.num = q.theta_num;
        A.den = q.theta_den;
        A.universe = q.universe;
        A.excl = q.exclude_other ? 1 : 0;
        // N(b) and N(a) hold the other endpoint, so |U| >= 1 unless it is left out
        A.zero_never = any || (q.theta_num > 0 && !q.exclude_other &&
                               (q.universe == FOLTY_UNIVERSE_DST || q.universe == FOLTY_UNIVERSE_SRC));
        A.any = any ? 1 : 0;
        A.ncert = ws.ncert.as<uint32_t>();
        A.scal = ws.scal.as<unsigned long long>();
        k_threshold<<<grid_for(m, BLK, THRESHOLD_BLOCKS), BLK, 0, s>>>(A);
        FOLTY_LAUNCHED();
        ws.pairs_k.ensure(16 * (size_t)S + 16);
        ws.pairs_v.ensure(8 * (size_t)S + 8);
        k_pairs_compact<<<grid_for(2 * (int64_t)S, BLK * PAIR_ITEMS), BLK, 0, s>>>(
            ws.ncert.as<uint32_t>(), S, ix.slo.as<int32_t>(), ix.shi.as<int32_t>(), pair_bits(ix.n),
            ws.pairs_k.as<uint64_t>(), ws.pairs_v.as<uint32_t>(), np);
        k_pairs_small<<<1, SMALL_BLK, 0, s>>>(ws.pairs_k.as<uint64_t>(), ws.pairs_v.as<uint32_t>(), np,
                                              pair_bits(ix.n), reinterpret_cast<int32_t *>(ws.scal.as<char>() + SCAL_BYTES));
        FOLTY_LAUNCHED();
    }
}

// |Sol| and the number of pairs, from the scalars on the host
PairCounts pair_counts(const Workspace &ws) {
    int32_t npairs;
    memcpy(&npairs, ws.host.as<unsigned long long>() + SCAL_PAIRS, 4);
    return PairCounts{region_sum(ws, REGION_CERTS), npairs};
}

// sort the pair keys of threshold_pairs and unpack them: u, v and the
// certificate counts, sorted by (u, v), in ws
void sort_pairs(const Graph *g, Workspace &ws, int32_t npairs, hipStream_t s, int32_t **du, int32_t **dv,
                uint32_t **dn) {
    const Index &ix = g->ix;
    ws.pairs_k2.ensure(8 * (size_t)npairs);
    ws.pairs_v2.ensure(4 * (size_t)npairs);
    const int nb = pair_bits(ix.n);
    size_t need = sort_pairs_u64_u32(nullptr, 0, ws.pairs_k.as<uint64_t>(), ws.pairs_k2.as<uint64_t>(),
                                     ws.pairs_v.as<uint32_t>(), ws.pairs_v2.as<uint32_t>(), npairs, 2 * nb, s);
    ws.cub.ensure(need);
    sort_pairs_u64_u32(ws.cub.p, need, ws.pairs_k.as<uint64_t>(), ws.pairs_k2.as<uint64_t>(),
                       ws.pairs_v.as<uint32_t>(), ws.pairs_v2.as<uint32_t>(), npairs, 2 * nb, s);
    // the unsorted keys are no longer needed: u and v go where they were
    *du = reinterpret_cast<int32_t *>(ws.pairs_k.p);
    *dv = *du + npairs;
    *dn = ws.pairs_v2.as<uint32_t>();
    k_pairs_unpack<<<grid_for(npairs, BLK), BLK, 0, s>>>(ws.pairs_k2.as<uint64_t>(), npairs, nb, *du, *dv);
    FOLTY_LAUNCHED();
}

// per-edge counts in input order (0xFFFFFFFF for self-loops) into out
void scatter_counts(const Graph *g, const uint32_t *count, uint32_t *out, hipStream_t s) {
    const Index &ix = g->ix;
    if (ix.m_input > 0) {
        k_fill<uint32_t><<<grid_for(ix.m_input, BLK), BLK, 0, s>>>(out, 0xffffffffu, ix.m_input);
        FOLTY_LAUNCHED();
    }
    if (ix.m > 0) {
        k_counts_scatter<<<grid_for(ix.m, BLK), BLK, 0, s>>>(count, ix.perm.as<int32_t>(), ix.m, out);
        FOLTY_LAUNCHED();
    }
}

void keep_counts(const Graph *g, const uint32_t *count, Result *res, hipStream_t s);

// threshold, pairs and (kept) per-edge counts into res.  The stream is idle after
// it; ev[3] follows the pair step.  Returns the pairs' first vertices on the device.
const int32_t *finish_query(const Graph *g, const folty_query &q, const uint32_t *count, Workspace &ws, Result *res,
                  hipStream_t s, bool any) {
    threshold_pairs(g, q, count, ws, s, any);
    read_scalars(ws, s, true);
    FOLTY_HIP(hipEventRecord(ws.ev[3], s));
    if (!(q.flags & FOLTY_QUERY_NO_COUNTS)) keep_counts(g, count, res, s);
    FOLTY_HIP(hipStreamSynchronize(s));
    const PairCounts pc = pair_counts(ws);
    const int32_t npairs = pc.npairs;
    res->n_certificates = pc.ncerts;
    res->u.resize(npairs);
    res->v.resize(npairs);
    res->n_cert.resize(npairs);
    const int32_t *first = reinterpret_cast<const int32_t *>(ws.scal.as<char>() + SCAL_BYTES);
    if (npairs > SMALL_PAIRS) {
        int32_t *du, *dv;
        uint32_t *dn;
        sort_pairs(g, ws, npairs, s, &du, &dv, &dn);
        FOLTY_HIP(hipMemcpyAsync(res->u.data(), du, 4 * (size_t)npairs, hipMemcpyDeviceToHost, s));
        FOLTY_HIP(hipMemcpyAsync(res->v.data(), dv, 4 * (size_t)npairs, hipMemcpyDeviceToHost, s));
        FOLTY_HIP(hipMemcpyAsync(res->n_cert.data(), dn, 4 * (size_t)npairs, hipMemcpyDeviceToHost, s));
        FOLTY_HIP(hipEventRecord(ws.ev[3], s));
        FOLTY_HIP(hipStreamSynchronize(s));
        first = du;
    } else if (npairs > 0) {
        const int32_t *p = reinterpret_cast<const int32_t *>(ws.host.as<char>() + SCAL_BYTES);
        memcpy(res->u.data(), p, 4 * (size_t)npairs);
        memcpy(res->v.data(), p + SMALL_PAIRS, 4 * (size_t)npairs);
        memcpy(res->n_cert.data(), p + 2 * SMALL_PAIRS, 4 * (size_t)npairs);
    }
    return first;
}

void keep_counts(const Graph *g, const uint32_t *count, Result *res, hipStream_t s) {
    res->counts_dev.ensure(4 * (size_t)g->ix.m_input + 4);
    scatter_counts(g, count, res->counts_dev.as<uint32_t>(), s);
    res->has_counts = true;
    res->device = g->device;
}

} // namespace

// one pass of a sink over every item
template <class Sink> static void enumerate_all(const Index &ix, const Sink &sink, hipStream_t s) {
    k_tri_enum<<<enum_grid(ix.NI), BLK, 0, s>>>(enum_graph(ix), ix.NI, sink);
    FOLTY_LAUNCHED();
}

static void count_triangles(Index &ix, DevBuf &base, hipStream_t s);

void index_triangles(Index &ix, bool cache, DevBuf &cub, hipStream_t s) {
    const int32_t n = ix.n, S = ix.S;
    ix.rec.ensure(sizeof(EdgeRec) * ((size_t)S + 1));
    ix.erng.ensure(sizeof(uint2) * ((size_t)S + 1));
    ix.tcnt_ready = false;
    if (S > 0) {
        DevBuf srec;
        srec.ensure(sizeof(EdgeRec) * (size_t)S);
        k_static_recs<<<grid_for(S, BLK), BLK, 0, s>>>(ix.soff.as<int32_t>(), ix.smid.as<int32_t>(),
                                                       ix.ts.as<int64_t>(), S, ix.tshift, srec.as<EdgeRec>());
        k_edge_recs<<<grid_for(S, BLK), BLK, 0, s>>>(ix.oeid.as<uint32_t>(), srec.as<EdgeRec>(), S,
                                                     ix.rshift - ix.tshift, ix.rbase, ix.rec.as<EdgeRec>(),
                                                     ix.erng.as<uint2>());
        FOLTY_LAUNCHED();
    }
    // probe segments grouped by owner, their probe prefix, and items
    ix.seg.ensure(sizeof(int4) * ((size_t)S + 1));
    ix.srng.ensure(sizeof(uint2) * ((size_t)S + 1));
    ix.owner.ensure(4 * ((size_t)S + 1));
    int32_t ni = 0, ng = 0;
    int64_t probes = 0;
    {
        PinnedBuf hb;
        hb.ensure(64);
        DevBuf key, key2, val, val2, run, len, P, flag, fid, start, cnt;
        key.ensure(4 * (size_t)S + 4);
        key2.ensure(4 * (size_t)S + 4);
        val.ensure(4 * (size_t)S + 4);
        val2.ensure(4 * (size_t)S + 4);
        len.ensure(4 * ((size_t)S + 1));
        P.ensure(8 * ((size_t)S + 1));
        flag.ensure(4 * (size_t)S + 4);
        fid.ensure(4 * (size_t)S + 4);
        start.ensure(4 * ((size_t)S + 1));
        run.ensure(8 * ((size_t)n + 1));
        cnt.ensure(4);
        if (S > 0) {
            k_seg_keys<<<grid_for(S, BLK), BLK, 0, s>>>(ix.ooff.as<int32_t>(), ix.oadj.as<int32_t>(),
                                                        ix.otail.as<int32_t>(), S, n, key.as<uint32_t>(),
                                                        val.as<uint32_t>());
            FOLTY_LAUNCHED();
            const int kb = bit_length((uint64_t)n);
            size_t need = sort_pairs_u32_i32(nullptr, 0, key.as<uint32_t>(), key2.as<uint32_t>(), val.as<int32_t>(),
                                             val2.as<int32_t>(), S, kb, s);
            cub.ensure(need);
            sort_pairs_u32_i32(cub.p, need, key.as<uint32_t>(), key2.as<uint32_t>(), val.as<int32_t>(),
                               val2.as<int32_t>(), S, kb, s);
            k_seg_recs<<<grid_for(S, BLK), BLK, 0, s>>>(key2.as<uint32_t>(), val2.as<uint32_t>(), ix.ooff.as<int32_t>(),
                                                        ix.oadj.as<int32_t>(), ix.otail.as<int32_t>(),
                                                        ix.erng.as<uint2>(), S, n, ix.seg.as<int4>(),
                                                        ix.srng.as<uint2>(), ix.owner.as<int32_t>(), len.as<int32_t>(), run.as<int2>(),
                                                        cnt.as<int32_t>());
            k_fill<int32_t><<<1, 1, 0, s>>>(len.as<int32_t>() + S, 0, 1);
            FOLTY_LAUNCHED();
            need = exclusive_scan_i32_to_i64(nullptr, 0, len.as<int32_t>(), P.as<int64_t>(), (int64_t)S + 1, s);
            cub.ensure(need);
            exclusive_scan_i32_to_i64(cub.p, need, len.as<int32_t>(), P.as<int64_t>(), (int64_t)S + 1, s);
            FOLTY_HIP(hipMemcpyAsync(hb.p, cnt.p, 4, hipMemcpyDeviceToHost, s));
            FOLTY_HIP(hipMemcpyAsync(hb.as<int64_t>() + 1, P.as<int64_t>() + S, 8, hipMemcpyDeviceToHost, s));
            FOLTY_HIP(hipStreamSynchronize(s));
            ng = *hb.as<int32_t>();
            probes = hb.as<int64_t>()[1];
        }
        if (ng > 0) {
            k_item_flags<<<grid_for(ng, BLK), BLK, 0, s>>>(key2.as<uint32_t>(), P.as<int64_t>(), run.as<int2>(), ng,
                                                           flag.as<int32_t>());
            FOLTY_LAUNCHED();
            size_t need = inclusive_scan_i32(nullptr, 0, flag.as<int32_t>(), fid.as<int32_t>(), ng, s);
            cub.ensure(need);
            inclusive_scan_i32(cub.p, need, flag.as<int32_t>(), fid.as<int32_t>(), ng, s);
            k_item_starts<<<grid_for(ng, BLK), BLK, 0, s>>>(flag.as<int32_t>(), fid.as<int32_t>(), ng,
                                                            start.as<int32_t>());
            FOLTY_LAUNCHED();
            FOLTY_HIP(hipMemcpyAsync(hb.p, fid.as<int32_t>() + (ng - 1), 4, hipMemcpyDeviceToHost, s));
            FOLTY_HIP(hipStreamSynchronize(s));
            ni = *hb.as<int32_t>();
            k_fill<int32_t><<<1, 1, 0, s>>>(start.as<int32_t>() + ni, ng, 1);
            FOLTY_LAUNCHED();
        }
        ix.item.ensure(sizeof(EnumItem) * ((size_t)ni + 1));
        if (ni > 0) {
            k_items<<<grid_for(ni, BLK), BLK, 0, s>>>(start.as<int32_t>(), ix.owner.as<int32_t>(), P.as<int64_t>(),
                                                      run.as<int2>(), ix.ooff.as<int32_t>(), ni,
                                                      ix.item.as<EnumItem>());
            FOLTY_LAUNCHED();
        }
        FOLTY_HIP(hipStreamSynchronize(s)); // the temporaries go back to the pool
    }
    ix.otail.release();
    ix.NI = ni;
    ix.G = ng;
    ix.probes = probes;
    // counted by the first query, or by what needs them before (plans, the server's
    // memory estimate, the cached list)
    ix.T = -1;
    ix.triangles_asked.store(cache, std::memory_order_release);
    ix.tri_cached = false;
    ix.tri.release();
    if (cache) {
        DevBuf base;
        count_triangles(ix, base, s);
        if (ix.T > 0) {
            ix.tri.ensure(12 * (size_t)ix.T);
            CacheSink sink{base.as<int64_t>(), ix.tri.as<int32_t>(), 0};
            enumerate_all(ix, sink, s);
            FOLTY_LAUNCHED();
            ix.tri_cached = true;
        }
    }
}


// counts the triangles (ix.T); base: int64[NI + 1], each item's first slot in a list of them all
static void count_triangles(Index &ix, DevBuf &base, hipStream_t s) {
    const int32_t ni = ix.NI;
    DevBuf tri_it, cub;
    tri_it.ensure(4 * ((size_t)ni + 1));
    base.ensure(8 * ((size_t)ni + 1));
    if (ni > 0) enumerate_all(ix, CountSink{tri_it.as<int32_t>(), 0}, s);
    k_fill<int32_t><<<1, 1, 0, s>>>(tri_it.as<int32_t>() + ni, 0, 1);
    FOLTY_LAUNCHED();
    size_t need = exclusive_scan_i32_to_i64(nullptr, 0, tri_it.as<int32_t>(), base.as<int64_t>(), (int64_t)ni + 1, s);
    cub.ensure(need);
    exclusive_scan_i32_to_i64(cub.p, need, tri_it.as<int32_t>(), base.as<int64_t>(), (int64_t)ni + 1, s);
    PinnedBuf hb;
    hb.ensure(8);
    FOLTY_HIP(hipMemcpyAsync(hb.p, base.as<int64_t>() + ni, 8, hipMemcpyDeviceToHost, s));
    FOLTY_HIP(hipStreamSynchronize(s));
    ix.T = *hb.as<int64_t>();
}

void ensure_triangles(Graph *g) {
    std::lock_guard<std::mutex> lk(g->lazy_mu);
    Index &ix = g->ix;
    if (!ix.built) return;
    if (ix.T.load() < 0) {
        FOLTY_HIP(hipSetDevice(g->device));
        StreamScope sc(g->stream);
        HookScope hs(&g->hook);
        DevBuf base;
        count_triangles(ix, base, g->stream);
    }
    ix.triangles_asked.store(true, std::memory_order_release);
}

void ensure_tcnt(Index &ix, hipStream_t s) {
    if (ix.tcnt_ready) return;
    ix.tcnt.ensure(4 * (size_t)ix.S + 4);
    if (ix.S > 0) {
        k_fill<int32_t><<<grid_for(ix.S, BLK), BLK, 0, s>>>(ix.tcnt.as<int32_t>(), 0, ix.S);
        FOLTY_LAUNCHED();
        TcntSink sink{ix.oeid.as<uint32_t>(), ix.tcnt.as<int32_t>()};
        enumerate_all(ix, sink, s);
        FOLTY_LAUNCHED();
    }
    ix.tcnt_ready = true;
}

void check_query(const Graph *g, const folty_query &q) {
    if (!g->ix.built) fail(FOLTY_ENOTBUILT, "folty_build_index has not been called for this graph");
    if (q.delta < 0) fail(FOLTY_EINVAL, "delta must be >= 0 (got %lld)", (long long)q.delta);
    if (q.theta_den == 0) fail(FOLTY_EINVAL, "theta_den must be > 0");
    if (q.theta_num > q.theta_den) fail(FOLTY_EINVAL, "theta must lie in [0, 1]");
    if (q.variant > 7) fail(FOLTY_EINVAL, "variant must be 0..7 (got %u)", (unsigned)q.variant);
    if (q.universe > 2) fail(FOLTY_EINVAL, "unknown universe %u", (unsigned)q.universe);
    if (q.exclude_other > 1) fail(FOLTY_EINVAL, "exclude_other must be 0 or 1");
    if (q.exclude_other && q.universe == FOLTY_UNIVERSE_COMMON)
        fail(FOLTY_EINVAL, "exclude_other applies to the N(a) and N(b) universes only");
    if (q.flags & ~(FOLTY_QUERY_NO_COUNTS | FOLTY_QUERY_SMALLER_SIDE | FOLTY_QUERY_ONE_PASS))
        fail(FOLTY_EINVAL, "unknown query flags 0x%x", (unsigned)q.flags);
}

Result *run_query(Graph *g, const folty_query &q, Workspace &ws) { return run_query_on(g, q, ws, g->stream); }

static Result *run_query_impl(Graph *g, const folty_query &q, Workspace &ws, hipStream_t s,
                              const folty_vertex_query *vq);

Result *run_query_on(Graph *g, const folty_query &q, Workspace &ws, hipStream_t s) {
    check_query(g, q);
    return run_query_impl(g, q, ws, s, nullptr);
}

Result *run_vertex_query(Graph *g, const folty_vertex_query &vq, Workspace &ws) {
    if (vq.inner > FOLTY_INNER_EXISTS) fail(FOLTY_EINVAL, "unknown inner quantifier %u", (unsigned)vq.inner);
    for (int i = 0; i < 7; i++)
        if (vq.reserved[i]) fail(FOLTY_EINVAL, "reserved fields of the vertex query must be 0");
    if (vq.theta_den == 0) fail(FOLTY_EINVAL, "theta_den must be > 0");
    if (vq.theta_num > vq.theta_den) fail(FOLTY_EINVAL, "theta must lie in [0, 1]");
    folty_query q = vq.edge;
    if (vq.inner == FOLTY_INNER_EXISTS) { // the edge threshold is not read
        q.theta_num = 1;
        q.theta_den = 1;
    }
    check_query(g, q);
    return run_query_impl(g, q, ws, g->stream, &vq);
}

// The counts of a query (paper, Algorithm ExistExistForAll, the out- and
// in-count arrays summed): filter, temporal tests, per-edge counts in sorted
// edge order in ws.count.  Events: ev[0] start, ev[4]/ev[5] around the filter,
// ev[2] after the tests.  The scalars are on the device.
static const uint32_t *query_counts(Graph *g, const folty_query &q, Workspace &ws, hipStream_t s, bool *one_pass) {
    Index &ix = g->ix;
    ws.ensure_events();
    *one_pass = use_one_pass(g, q);
    FOLTY_HIP(hipEventRecord(ws.ev[0], s));
    clear_query(ix, ws, true, s);
    uint32_t *count = ws.count.as<uint32_t>();
    if (ix.NI > 0) {
        const bool ss = (q.flags & FOLTY_QUERY_SMALLER_SIDE) != 0;
        int32_t *diff = nullptr;
        // runs with a shorter L2 mark edge ranges in diff; its prefix sum is added at the end
        auto clear_marks = [&] {
            if (!ss) return;
            ws.diff.ensure(4 * (2 * (size_t)ix.m + 1));
            diff = ws.diff.as<int32_t>();
            k_fill<int32_t><<<grid_for(ix.m + 1, BLK, PERSIST_BLOCKS), BLK, 0, s>>>(diff, 0, ix.m + 1);
            FOLTY_LAUNCHED();
        };
        auto add_marks = [&] {
            if (!ss) return;
            int32_t *ps = diff + ix.m + 1;
            size_t need = inclusive_scan_i32(nullptr, 0, diff, ps, ix.m, s);
            ws.cub.ensure(need);
            inclusive_scan_i32(ws.cub.p, need, diff, ps, ix.m, s);
            k_add_counts<<<grid_for(ix.m, BLK, PERSIST_BLOCKS), BLK, 0, s>>>(ps, ix.m, count);
            FOLTY_LAUNCHED();
        };
        auto tests = [&](const CandBuf &B) {
            if (ss) launch_temporal<true>(ix, q.variant, q.delta, ws, B, DirectOp{q.delta, count, diff}, s);
            else launch_temporal<false>(ix, q.variant, q.delta, ws, B, DirectOp{q.delta, count, nullptr}, s);
        };
        FOLTY_HIP(hipEventRecord(ws.ev[4], s));
        if (arena_left() >= 0) {
            clear_marks();
            filter_in_arena(ix, q, ws, s, *one_pass, tests);
            FOLTY_HIP(hipEventRecord(ws.ev[5], s));
            add_marks();
        } else {
            const CandBuf B = filter_triangles(ix, q.variant, q.delta, ws, s, *one_pass);
            FOLTY_HIP(hipEventRecord(ws.ev[5], s));
            if (ws.kept_chunks > 0) {
                clear_marks();
                tests(B);
                add_marks();
            }
        }
    } else {
        FOLTY_HIP(hipEventRecord(ws.ev[4], s));
        FOLTY_HIP(hipEventRecord(ws.ev[5], s));
    }
    FOLTY_HIP(hipEventRecord(ws.ev[2], s));
    return count;
}

// Rows of the oriented graph by the edges (u, v) that meet them: out[0] += rows u with
// an edge to a row v that is no longer; a bit is set per row v with an edge from a
// shorter row u.
__global__ __launch_bounds__(BLK) void k_row_sides(const int32_t *__restrict__ ooff, const int32_t *__restrict__ oadj,
                                                   int32_t n, uint32_t *__restrict__ bits,
                                                   unsigned long long *__restrict__ out) {
    unsigned long long c = 0;
    for (int64_t u = (int64_t)blockIdx.x * BLK + threadIdx.x; u < n; u += (int64_t)gridDim.x * BLK) {
        const int32_t b = ooff[u], e = ooff[u + 1];
        bool any = false;
        for (int32_t p = b; p < e; p++) {
            const int32_t v = oadj[p];
            if (ooff[v + 1] - ooff[v] <= e - b) any = true;
            else if (bits) atomicOr(&bits[v >> 5], 1u << (v & 31));
        }
        c += any;
    }
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane_id() == 0 && c) atomicAdd(out, c);
}
__global__ __launch_bounds__(BLK) void k_count_bits(const uint32_t *__restrict__ bits, int64_t words,
                                                    unsigned long long *__restrict__ out) {
    unsigned long long c = 0;
    for (int64_t i = (int64_t)blockIdx.x * BLK + threadIdx.x; i < words; i += (int64_t)gridDim.x * BLK)
        c += __popc(bits[i]);
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane_id() == 0 && c) atomicAdd(out, c);
}

// The graphs that a fixed scratch takes are a matter of their sizes alone, the same
// for every window (folty.h): 4 bytes per edge, 32 per static edge and 36 per side of
// a row have to fit.  That is a promise, and more than the buffers need: the sides
// are counted only for graphs near the limit.
static void check_scratch(const Index &ix, Workspace &ws, hipStream_t s) {
    const int64_t cap = arena_left(), edges = 4 * (int64_t)ix.m + 32 * (int64_t)ix.S;
    int64_t need = edges;
    if (edges <= cap && edges + 36 * (int64_t)ix.S > cap) { // at least one edge to a side
        ws.scal.ensure(SCAL_ALL_BYTES);
        ws.host.ensure(SCAL_ALL_BYTES);
        unsigned long long *out = ws.scal.as<unsigned long long>();
        k_fill<unsigned long long><<<1, 1, 0, s>>>(out, 0ull, 1);
        const size_t mark = arena_mark();
        const int64_t words = ((int64_t)ix.n + 31) / 32;
        DevBuf bits;
        if (4 * words + 256 <= arena_left()) {
            bits.ensure(4 * (size_t)words);
            k_fill<uint32_t><<<grid_for(words, BLK, 1024), BLK, 0, s>>>(bits.as<uint32_t>(), 0u, words);
        }
        k_row_sides<<<grid_for(ix.n, BLK, 256), BLK, 0, s>>>(ix.ooff.as<int32_t>(), ix.oadj.as<int32_t>(), ix.n,
                                                             bits.as<uint32_t>(), out);
        if (bits.p) k_count_bits<<<grid_for(words, BLK, 256), BLK, 0, s>>>(bits.as<uint32_t>(), words, out);
        FOLTY_LAUNCHED();
        bits.forget();
        arena_rewind(mark);
        FOLTY_HIP(hipMemcpyAsync(ws.host.p, out, 8, hipMemcpyDeviceToHost, s));
        FOLTY_HIP(hipStreamSynchronize(s));
        need += 36 * *ws.host.as<int64_t>();
    }
    if (need > cap)
        fail(FOLTY_ENOMEM, "this call needs more than the %lld bytes of its fixed device scratch (%lld)", (long long)cap,
             (long long)need);
}

void run_query_into(Graph *g, const folty_query &q, Workspace &ws, int32_t *pair_u, int32_t *pair_v,
                    uint32_t *n_cert, int64_t pair_cap, uint32_t *edge_count, int64_t *n_pairs,
                    int64_t *n_certificates) {
    check_query(g, q);
    if (pair_cap < 0) fail(FOLTY_EINVAL, "pair_cap must be >= 0");
    if (pair_cap > 0 && (!pair_u || !pair_v || !n_cert)) fail(FOLTY_EINVAL, "null pair output array");
    if (hipSetDevice(g->device) != hipSuccess) fail(FOLTY_EDEVICE, "hipSetDevice failed");
    Index &ix = g->ix;
    if (q.universe == FOLTY_UNIVERSE_COMMON && !ix.tcnt_ready)
        fail(FOLTY_EINVAL, "the universe N(a) & N(b) needs the graph's per-edge triangle counts, which this call "
                           "does not build: run one query with that universe through folty_run_fol_query first");
    if ((q.flags & FOLTY_QUERY_ONE_PASS) && !ix.triangles_asked.load(std::memory_order_acquire))
        fail(FOLTY_EINVAL, "FOLTY_QUERY_ONE_PASS needs the graph's triangles, which this call does not count "
                           "beforehand: run one query with that flag through folty_run_fol_query first");
    hipStream_t s = g->stream;
    if (arena_left() >= 0) check_scratch(ix, ws, s);
    bool one_pass = false;
    const uint32_t *count = query_counts(g, q, ws, s, &one_pass);
    threshold_pairs(g, q, count, ws, s, false);
    read_scalars(ws, s, false);
    FOLTY_HIP(hipStreamSynchronize(s));
    const PairCounts pc = pair_counts(ws);
    if (ix.T.load() < 0) ix.T = region_sum(ws, REGION_HITS);
    *n_pairs = pc.npairs;
    *n_certificates = pc.ncerts;
    if (edge_count) scatter_counts(g, count, edge_count, s);
    if (pc.npairs > pair_cap) {
        FOLTY_HIP(hipStreamSynchronize(s));
        fail(FOLTY_EOVERFLOW, "%d solution pairs do not fit the %lld the caller's arrays hold", pc.npairs,
             (long long)pair_cap);
    }
    if (pc.npairs > 0) {
        int32_t *du, *dv;
        uint32_t *dn;
        sort_pairs(g, ws, pc.npairs, s, &du, &dv, &dn);
        FOLTY_HIP(hipMemcpyAsync(pair_u, du, 4 * (size_t)pc.npairs, hipMemcpyDeviceToDevice, s));
        FOLTY_HIP(hipMemcpyAsync(pair_v, dv, 4 * (size_t)pc.npairs, hipMemcpyDeviceToDevice, s));
        FOLTY_HIP(hipMemcpyAsync(n_cert, dn, 4 * (size_t)pc.npairs, hipMemcpyDeviceToDevice, s));
    }
    FOLTY_HIP(hipStreamSynchronize(s));
}

static Result *run_query_impl(Graph *g, const folty_query &q, Workspace &ws, hipStream_t s,
                              const folty_vertex_query *vq) {
    if (hipSetDevice(g->device) != hipSuccess) fail(FOLTY_EDEVICE, "hipSetDevice failed");
    Index &ix = g->ix;
    if (q.universe == FOLTY_UNIVERSE_COMMON) {
        std::lock_guard<std::mutex> lk(g->lazy_mu);
        HookScope hs(&g->hook);
        ensure_tcnt(ix, s);
        FOLTY_HIP(hipStreamSynchronize(s));
    }
    std::unique_ptr<Result> res(new Result());
    StreamScope sc(s); // an error waits for the copies into res before res goes
    bool one_pass = false;
    const uint32_t *count = query_counts(g, q, ws, s, &one_pass);
    const int32_t *first = finish_query(g, q, count, ws, res.get(), s, vq && vq->inner == FOLTY_INNER_EXISTS);
    if (vq) {
        finish_vertex(g, *vq, ws, first, (int32_t)res->u.size(), res.get(), s);
        FOLTY_HIP(hipEventRecord(ws.ev[3], s));
        FOLTY_HIP(hipStreamSynchronize(s));
    }
    if (ix.NI > 0) after_filter(ix, ws, q.delta, one_pass);
    else ix.T = 0;
    fill_stats_from_index(ix, &res->stats);
    res->stats.tests = region_sum(ws, REGION_TESTS);
    res->stats.n_pairs = (int64_t)res->u.size();
    res->stats.n_certificates = res->n_certificates;
    res->stats.wedge_ms = ev_ms(ws.ev[4], ws.ev[5]);
    res->stats.temporal_ms = ev_ms(ws.ev[5], ws.ev[2]);
    res->stats.threshold_ms = ev_ms(ws.ev[2], ws.ev[3]);
    res->stats.query_ms = ev_ms(ws.ev[0], ws.ev[3]);
    res->stats.filter_passes = ix.NI > 0 ? ws.filter_passes : 0;
    return res.release();
}

// Device bytes one single query in a bounded workspace takes beyond the resident
// index: per-edge counts, the chunks of the triangles its filter keeps, the
// smaller-side difference array, per-pair certificate counts, pair keys and their
// sorted copies, sort and scan scratch, and the per-edge counts handed back.
int64_t query_footprint(const Graph *g, const folty_query &q) {
    const Index &ix = g->ix;
    const int64_t T = std::max<int64_t>(0, ix.T.load());
    // counts; the filter's chunks (every triangle kept); heavy triangles; pair step
    int64_t b = 4 * (int64_t)ix.m + CHUNK_BYTES * bounded_chunks(ix, T) +
                (int64_t)sizeof(Heavy) * heavy_slots(T) + 56 * (int64_t)ix.S;
    if (q.flags & FOLTY_QUERY_SMALLER_SIDE) b += 8 * (int64_t)ix.m + 4;
    if (!(q.flags & FOLTY_QUERY_NO_COUNTS)) b += 4 * ix.m_input;
    // the library scratch the query's sorts and scans ask for (sizes only)
    const int64_t S2 = 2 * (int64_t)ix.S;
    const size_t scratch = std::max({sort_pairs_u64_u32(nullptr, 0, nullptr, nullptr, nullptr, nullptr, S2,
                                                        2 * pair_bits(ix.n), nullptr),
                                     inclusive_scan_i32(nullptr, 0, nullptr, nullptr, ix.m, nullptr),
                                     exclusive_scan_i32(nullptr, 0, nullptr, nullptr, ix.n, nullptr)});
    // scalars, and what allocations are rounded up by
    return b + (int64_t)scratch + (1 << 20);
}

void fill_stats_from_index(const Index &ix, folty_stats *s) {
    s->n = ix.n;
    s->m_input = ix.m_input;
    s->m = ix.m;
    s->self_loops = ix.self_loops;
    s->static_edges = ix.S;
    s->directed_pairs = ix.P;
    s->max_core = ix.max_core;
    s->max_out_degree = ix.max_out;
    s->wedges = ix.W;
    s->triangles = ix.T;
    s->max_multiplicity = ix.sigma_max;
    s->peel_rounds = ix.peel_rounds;
    s->core_sweeps = ix.core_sweeps;
    s->closing_probes = ix.probes;
    s->enum_items = ix.NI;
    s->build_ms = ix.build_ms;
}

Workspace::~Workspace() {
    if (events)
        for (auto &e : ev) (void)hipEventDestroy(e);
}

size_t Workspace::device_bytes() const {
    const DevBuf *b[] = {&count, &sv, &svn, &pieces, &ncert, &pairs_k, &pairs_v,
                         &pairs_k2, &pairs_v2, &scal, &cub, &vtmp, &diff, &tflag, &tinst};
    size_t t = 0;
    for (auto *x : b) t += x->bytes;
    return t;
}

void Workspace::forget_buffers() {
    DevBuf *b[] = {&count, &sv, &svn, &pieces, &ncert, &pairs_k, &pairs_v,
                   &pairs_k2, &pairs_v2, &scal, &cub, &vtmp, &diff, &tflag, &tinst};
    for (auto *x : b) x->forget();
}

void Workspace::ensure_events() {
    if (events) return;
    for (auto &e : ev) FOLTY_HIP(hipEventCreate(&e));
    events = true;
}

} // namespace folty
