// Graph formats built on the device (Section 4.1: the in-CSR for g-SpMM, the
// reverse graph's CSR for the backward pass; Appendix B: the reverse graph
// keeps the edge ids).
//
// A CSR is a stable sort of the edge list by row key: sorting the pairs
// (row of edge e, e) by row with a stable LSD radix sort leaves the edges of
// every row in ascending edge id, which is the order the kernels and the
// oracle reduce in.  Row offsets are then binary searches in the sorted keys
// (no atomics: every result is a pure function of the edge list), and a third
// stable sort, on (capacity - degree, row), gives the rows by descending
// degree with ties in ascending row id.
//
// Radix pass: digits of up to 9 bits, the passes of a sort sharing its bits
// evenly (18-bit row ids take two passes), 8,192 keys per workgroup.  Each
// wavefront ranks its 1,024 keys in 16 steps of 64: lanes with equal digits
// find each other with one ballot per digit bit, take their rank within the
// step from a popcount, and read the running count of their digit from the
// wavefront's LDS counters.  Counts of all workgroups are scanned
// digit-major, so equal digits keep their input order across workgroups as
// well.  A workgroup puts its keys, and then each array of values, in digit
// order in LDS before it stores them, so that the stores of a wavefront
// cover runs of consecutive addresses (16 keys of a digit on average at 9
// bits) rather than 64 lines: the pass is bound by its reads and writes of
// memory.  Two arrays of values can travel with the keys (an edge's id and
// its other endpoint), which leaves no random gather of endpoints after the
// sort.
#include <algorithm>

#include "device.h"

namespace gnnk {
namespace {

constexpr int RS_WAVES = 8;
constexpr int RS_BLOCK = RS_WAVES * 64;
constexpr int RS_BITS = 9;                         // most bits of a digit
constexpr int RS_DIGITS = 1 << RS_BITS;
static_assert(RS_DIGITS == RS_BLOCK, "thread d of a workgroup handles digit d");
// keys per workgroup: 16 steps of 64 per wavefront, or 4 where 64 workgroups
// of those hold every key (a sort of 100,000 keys then runs on 49 workgroups
// rather than 13)
constexpr int rs_tile(int steps) { return RS_BLOCK * steps; }
// up to this many workgroups per sort, each adds up the counts of the others
// itself and the scan kernels are left out
constexpr int RS_DIRECT = 64;
constexpr int SCAN_BLOCK = 1024;
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;

inline unsigned tiles_of(int64_t n, int64_t per) { return (unsigned)((n + per - 1) / per); }

inline unsigned grid_1d(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    return (unsigned)(b > 0 ? b : 1);
}

// ---------------------------------------------------------------------------
// radix sort

// One pass of up to two sorts at once (the in-CSR's and the reverse CSR's are
// independent): workgroups [0, tiles of the first) take the first.
struct RsJob {
    const uint32_t* key;
    const uint32_t* v0;  // nullptr: 0..n-1
    const uint32_t* v1;
    uint32_t* key_out;
    uint32_t* out0;
    uint32_t* out1;
    int64_t n;
    int64_t hist;        // first word of the sort's counts
    uint32_t before;     // keys of the sort before it in the same scan
    int32_t n_tiles, shift, bits;
};
struct RsArgs {
    RsJob job[2];
    uint32_t* hist;
    int32_t direct;
};

// direct: counts by (workgroup, digit); else by (digit, workgroup), the order
// in which the scan gives each its first output position
template <int STEPS>
__global__ __launch_bounds__(RS_BLOCK) void rs_count_kernel(RsArgs A) {
    __shared__ uint32_t c[RS_DIGITS];
    const bool second = (int)blockIdx.x >= A.job[0].n_tiles;
    const RsJob& J = A.job[second];
    const int tile = (int)blockIdx.x - (second ? A.job[0].n_tiles : 0);
    const uint32_t mask = (1u << J.bits) - 1u;
    c[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t base = (int64_t)tile * rs_tile(STEPS);
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const int64_t i = base + j * RS_BLOCK + threadIdx.x;
        if (i < J.n) atomicAdd(&c[(J.key[i] >> J.shift) & mask], 1u);
    }
    __syncthreads();
    if (threadIdx.x <= mask)
        A.hist[J.hist + (A.direct ? ((int64_t)tile << J.bits) + threadIdx.x
                                  : (int64_t)threadIdx.x * J.n_tiles + tile)] = c[threadIdx.x];
}

// exclusive prefix of v over the threads of the workgroup
__device__ uint32_t rs_exclusive(uint32_t v, uint32_t* wsum) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0u;
#pragma unroll
    for (int i = 0; i < RS_WAVES; ++i) off += i < w ? wsum[i] : 0u;
    return off + inc - v;
}

// NV: arrays of values that move with the keys
template <int NV, int STEPS>
__global__ __launch_bounds__(RS_BLOCK) void rs_scatter_kernel(RsArgs A) {
    __shared__ uint32_t cnt[RS_WAVES][RS_DIGITS];
    __shared__ uint32_t first[RS_DIGITS];  // output position of a digit's first key less its place in the tile
    __shared__ uint32_t wsum[2][RS_WAVES];
    __shared__ uint32_t stage[rs_tile(STEPS)];
    const bool second = (int)blockIdx.x >= A.job[0].n_tiles;
    const RsJob& J = A.job[second];
    const int tile = (int)blockIdx.x - (second ? A.job[0].n_tiles : 0);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int shift = J.shift, bits = J.bits;
    const int64_t n = J.n;
    const uint32_t mask = (1u << bits) - 1u;
    const int64_t tile0 = (int64_t)tile * rs_tile(STEPS);
    const int64_t base = tile0 + (int64_t)w * (64 * STEPS);
    const int m = (int)(n - tile0 < rs_tile(STEPS) ? n - tile0 : rs_tile(STEPS));  // keys of this tile
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint32_t k[STEPS], a[STEPS], b[STEPS], at[STEPS];
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const int64_t i = base + j * 64 + lane;
        const bool ok = i < n;
        k[j] = ok ? J.key[i] : 0u;
        a[j] = ok ? (J.v0 ? J.v0[i] : (uint32_t)i) : 0u;
        b[j] = NV > 1 && ok ? J.v1[i] : 0u;
    }
    // thread d: the output position of the tile's first key of digit d
    uint32_t pos = 0u;
    if (A.direct) {
        const uint32_t d = threadIdx.x;
        uint32_t all = 0u;
        if (d <= mask) {
            const uint32_t* h = A.hist + J.hist + d;
#pragma unroll 16
            for (int t = 0; t < J.n_tiles; ++t) {
                const uint32_t c = h[(int64_t)t << bits];
                pos += t < tile ? c : 0u;
                all += c;
            }
        }
        pos += rs_exclusive(all, wsum[0]);
    } else if (threadIdx.x <= mask) {
        pos = A.hist[J.hist + (int64_t)threadIdx.x * J.n_tiles + tile] - J.before;
    }
    for (int i = threadIdx.x; i < RS_WAVES * RS_DIGITS; i += RS_BLOCK) (&cnt[0][0])[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const bool ok = base + j * 64 + lane < n;
        const uint32_t d = (k[j] >> shift) & mask;
        uint64_t peers = __ballot(ok);
        for (int t = 0; t < bits; ++t) {
            const uint64_t bm = __ballot((d >> t) & 1u);
            peers &= ((d >> t) & 1u) ? bm : ~bm;
        }
        // every lane reads its digit's count before the last lane of each
        // digit group advances it (one LDS read, then one LDS write, in the
        // wavefront's program order)
        const uint32_t start = cnt[w][d];
        at[j] = start + (uint32_t)__popcll(peers & below);
        __builtin_amdgcn_wave_barrier();
        if (ok && (peers >> lane) == 1ull) cnt[w][d] = start + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {
        const uint32_t d = threadIdx.x;
        uint32_t tot = 0u;
#pragma unroll
        for (int ww = 0; ww < RS_WAVES; ++ww) tot += cnt[ww][d];
        uint32_t run = rs_exclusive(tot, wsum[1]);
        first[d] = pos - run;
#pragma unroll
        for (int ww = 0; ww < RS_WAVES; ++ww) {
            const uint32_t c = cnt[ww][d];
            cnt[ww][d] = run;
            run += c;
        }
    }
    __syncthreads();
    // the keys in digit order; at becomes a key's place in the tile, and `to`
    // the output position of the keys this thread stores
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        if (base + j * 64 + lane < n) {
            at[j] += cnt[w][(k[j] >> shift) & mask];
            stage[at[j]] = k[j];
        }
    }
    __syncthreads();
    uint32_t to[STEPS];
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const int i = j * RS_BLOCK + (int)threadIdx.x;
        to[j] = 0u;
        if (i < m) {
            const uint32_t key = stage[i];
            to[j] = first[(key >> shift) & mask] + (uint32_t)i;
            J.key_out[to[j]] = key;
        }
    }
    auto put = [&](const uint32_t* v, uint32_t* out) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < STEPS; ++j)
            if (base + j * 64 + lane < n) stage[at[j]] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            const int i = j * RS_BLOCK + (int)threadIdx.x;
            if (i < m) out[to[j]] = stage[i];
        }
    };
    put(a, J.out0);
    if constexpr (NV > 1) put(b, J.out1);
}

// ---------------------------------------------------------------------------
// exclusive scan of uint32 counts (in place)

__device__ uint32_t block_exclusive(uint32_t v, uint32_t* total) {
    __shared__ uint32_t wsum[SCAN_BLOCK / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0u, tot = 0u;
#pragma unroll
    for (int i = 0; i < SCAN_BLOCK / 64; ++i) {
        const uint32_t t = wsum[i];
        if (i < w) off += t;
        tot += t;
    }
    __syncthreads();  // wsum is reused by the next call
    *total = tot;
    return off + inc - v;
}

__device__ uint32_t scan_tile(uint32_t* x, int64_t n, int64_t tile, uint32_t carry) {
    const int64_t b = tile + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS], s = 0u;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        v[j] = b + j < n ? x[b + j] : 0u;
        s += v[j];
    }
    uint32_t total;
    uint32_t pre = block_exclusive(s, &total) + carry;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        if (b + j < n) x[b + j] = pre;
        pre += v[j];
    }
    return total;
}

__global__ __launch_bounds__(SCAN_BLOCK) void scan_reduce_kernel(const uint32_t* x, int64_t n, uint32_t* part) {
    const int64_t b = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t s = 0u;
    for (int j = 0; j < SCAN_ITEMS; ++j)
        if (b + j < n) s += x[b + j];
    uint32_t total;
    (void)block_exclusive(s, &total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// one workgroup: the tile sums, scanned tile by tile with a running carry
__global__ __launch_bounds__(SCAN_BLOCK) void scan_carry_kernel(uint32_t* part, int64_t n) {
    uint32_t carry = 0u;
    for (int64_t t = 0; t < n; t += SCAN_TILE) carry += scan_tile(part, n, t, carry);
}

__global__ __launch_bounds__(SCAN_BLOCK) void scan_apply_kernel(uint32_t* x, int64_t n, const uint32_t* part) {
    (void)scan_tile(x, n, (int64_t)blockIdx.x * SCAN_TILE, part[blockIdx.x]);
}

// ---------------------------------------------------------------------------
// structure from sorted keys

// Row offsets (the first position whose key is >= r, for r in [0, n_rows]),
// degrees and degree keys of both CSRs; a CSR whose offsets are the caller's
// (key == nullptr) has them read.
template <typename P>
__global__ void rows_kernel(RowsJob A, RowsJob B, int64_t n_keys) {
    const int64_t n0 = A.n_rows + 1, all = n0 + B.n_rows + 1;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < all; i += (int64_t)gridDim.x * blockDim.x) {
        const bool second = i >= n0;
        const RowsJob& J = second ? B : A;
        const int64_t r = second ? i - n0 : i;
        P* ptr = reinterpret_cast<P*>(J.ptr);
        int64_t at, next;
        if (J.key) {
            int64_t lo = 0, hi = n_keys;
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if ((int64_t)J.key[mid] < r) lo = mid + 1;
                else hi = mid;
            }
            at = lo;
            ptr[r] = (P)at;
            if (r == J.n_rows) continue;
            // the row's end by doubling steps from its start
            int64_t step = 1;
            while (lo + step < n_keys && (int64_t)J.key[lo + step] <= r) step <<= 1;
            hi = lo + step < n_keys ? lo + step : n_keys;
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if ((int64_t)J.key[mid] <= r) lo = mid + 1;
                else hi = mid;
            }
            next = lo;
        } else {
            if (r == J.n_rows) continue;
            at = (int64_t)ptr[r];
            next = (int64_t)ptr[r + 1];
        }
        const int32_t d = (int32_t)(next - at);
        J.deg[r] = d;
        J.deg_key[r] = (uint32_t)n_keys - (uint32_t)d;
    }
}

// pos[eid of position p of the reverse CSR] = p, and the identity check of
// the in-CSR's edge ids (in_eid == nullptr: known)
// At most one atomic per wavefront that saw a difference, and none once the
// flag is seen set: all of them meet at one address (one per difference took
// about 20 ms for a shuffled list of 114.6M ids, one per wavefront 3 ms).
__global__ void edge_ids_kernel(const int32_t* out_eid, int32_t* pos, const int32_t* in_eid, int64_t n,
                                int32_t* flag, int32_t bit) {
    bool off = false;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        if (out_eid) pos[out_eid[p]] = (int32_t)p;
        if (in_eid) off |= in_eid[p] != (int32_t)p;
    }
    const uint64_t m = __ballot(off);
    if (m == 0ull || (threadIdx.x & 63) != (unsigned)__builtin_ctzll(m)) return;
    if (!(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit)) atomicOr(flag, bit);
}

__global__ void count_ids_kernel(const int32_t* eid, int64_t n, uint32_t* counts, int32_t* flag, int32_t bit) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t e = eid[p];
        if (e < 0 || e >= n) atomicOr(flag, bit);
        else atomicAdd(counts + e, 1u);
    }
}

__global__ void check_once_kernel(const uint32_t* counts, int64_t n, int32_t* flag, int32_t bit) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        if (counts[i] != 1u) atomicOr(flag, bit);
}

__global__ void fill_u32_kernel(uint32_t* x, int64_t n, uint32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        x[i] = v;
}

// endpoints of every edge id from a CSR with explicit edge ids
__global__ void edge_ends_kernel(const int32_t* idx, const int32_t* eid, const int32_t* row, int64_t n,
                                 int32_t* src_of_e, int32_t* dst_of_e) {
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t e = eid[p];
        src_of_e[e] = idx[p];
        dst_of_e[e] = row[p];
    }
}

// What the host needs to know of the sorted degrees (BuildSummary in
// internal.h).  Workgroups 0..3: hub rows and segments of the four tables;
// the next ones: how close a row's edge ids lie; the others: rows of more than
// t edges, t = 0..SUMMARY_DEG; both directions each.
__device__ __forceinline__ int64_t rows_above(const uint32_t* sorted, int64_t n_rows, int64_t E, int64_t t) {
    if (t >= E) return 0;
    const uint32_t key = (uint32_t)(E - t);  // keys are E - degree, ascending
    int64_t lo = 0, hi = n_rows;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (sorted[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

constexpr int SUMMARY_BLOCK = 256;
static_assert(SUMMARY_SAMPLES % SUMMARY_BLOCK == 0, "whole workgroups sample");

__global__ __launch_bounds__(SUMMARY_BLOCK) void summary_kernel(SummaryArgs A) {
    if (blockIdx.x < SUMMARY_TABLES) {
        const int t = blockIdx.x;
        const int d = t >> 1;  // tables 0, 1 are the in-CSR's, 2, 3 the reverse CSR's
        const int64_t S = A.seg_edges[t];
        const int64_t n_hub = rows_above(A.sorted[d], A.n_rows[d], A.n_edges, S);
        int64_t sum = 0;
        for (int64_t k = threadIdx.x; k < n_hub; k += SUMMARY_BLOCK)
            sum += (A.n_edges - (int64_t)A.sorted[d][k] + S - 1) / S;
        __shared__ int64_t part[SUMMARY_BLOCK];
        part[threadIdx.x] = sum;
        __syncthreads();
        for (int o = SUMMARY_BLOCK / 2; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            A.out->n_hub[t] = (int32_t)n_hub;
            A.out->n_seg[t] = (int32_t)part[0];
        }
        return;
    }
    int i = (int)(blockIdx.x - SUMMARY_TABLES) * SUMMARY_BLOCK + (int)threadIdx.x;
    if (i < 2 * SUMMARY_SAMPLES) {
        // evenly spaced positions whose next edge id lies on the same or the
        // next lines of an edge tensor
        const int d = i >= SUMMARY_SAMPLES;
        if (!A.eid[d] || A.n_edges < 2) return;
        const int64_t p = (int64_t)(d ? i - SUMMARY_SAMPLES : i) * (A.n_edges - 1) / SUMMARY_SAMPLES;
        const int64_t gap = (int64_t)A.eid[d][p + 1] - (int64_t)A.eid[d][p];
        const uint64_t m = __ballot(gap >= -32 && gap <= 32);
        if (m != 0ull && (threadIdx.x & 63) == 0) atomicAdd(&A.out->near_ids[d], __popcll(m));
        return;
    }
    i -= 2 * SUMMARY_SAMPLES;
    const int d = i >= SUMMARY_DEG + 1;
    const int t = d ? i - (SUMMARY_DEG + 1) : i;
    if (t > SUMMARY_DEG) return;
    A.out->above[d][t] = (int32_t)rows_above(A.sorted[d], A.n_rows[d], A.n_edges, t);
    if (t == 0) {
        A.out->above_far[d] = (int32_t)rows_above(A.sorted[d], A.n_rows[d], A.n_edges, A.far[d]);
        A.out->max_deg[d] = A.n_rows[d] > 0 ? (int32_t)(A.n_edges - (int64_t)A.sorted[d][0]) : 0;
    }
}

// first segment of every hub row of each table, one workgroup per table
__global__ __launch_bounds__(SCAN_BLOCK) void hub_offsets_kernel(HubArgs A) {
    const HubTable& T = A.table[blockIdx.x];
    uint32_t carry = 0u;
    for (int64_t k0 = 0; k0 < T.n_hub; k0 += SCAN_BLOCK) {
        const int64_t k = k0 + threadIdx.x;
        const uint32_t v = k < T.n_hub ? (uint32_t)(((int64_t)T.rowt[k].z - T.rowt[k].y + T.seg_edges - 1) / T.seg_edges) : 0u;
        uint32_t total;
        const uint32_t pre = block_exclusive(v, &total) + carry;
        if (k < T.n_hub) T.hub_off[k] = (int32_t)pre;
        carry += total;
    }
    if (threadIdx.x == 0) T.hub_off[T.n_hub] = (int32_t)carry;
}

// the table of entry i of the concatenated tables
__device__ __forceinline__ int table_of(const HubArgs& A, int64_t i) {
    int t = 0;
#pragma unroll
    for (int u = 1; u < SUMMARY_TABLES; ++u) t += i >= A.table[u].base ? 1 : 0;
    return t;
}

// The segments of every table, one thread each, and their sort keys: the
// table above the halves of the first and last neighbour id, summed (below
// the neighbour count, so it fits id_bits bits after `drop` low ones).
__global__ void hub_segments_kernel(HubArgs A, int64_t n, int id_bits, int drop, uint32_t* key) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int t = table_of(A, i);
        const HubTable& T = A.table[t];
        const int32_t o = (int32_t)(i - T.base);
        int32_t lo = 0, hi = (int32_t)T.n_hub - 1;  // the last hub row whose first segment is <= o
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (T.hub_off[mid] <= o) lo = mid;
            else hi = mid - 1;
        }
        const int4 row = T.rowt[lo];
        const int64_t b = (int64_t)row.y + (int64_t)(o - T.hub_off[lo]) * T.seg_edges;
        const int64_t e = b + T.seg_edges < row.z ? b + T.seg_edges : row.z;
        T.seg[o] = make_int4(row.x, (int32_t)b, (int32_t)e, lo);
        if (key)
            key[i] = ((uint32_t)t << id_bits) | ((((uint32_t)T.idx[b] >> 1) + ((uint32_t)T.idx[e - 1] >> 1)) >> drop);
    }
}

// the segment of each hub-segment wavefront, with its table index: the walk
// then finds its segment with one load instead of two dependent ones
// (order == nullptr: table order)
__global__ void seg_wave_kernel(HubArgs A, int64_t n, const uint32_t* order) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const HubTable& T = A.table[table_of(A, i)];
        const int32_t si = (int32_t)((order ? (int64_t)order[i] : i) - T.base);
        const int4 g = T.seg[si];
        T.seg_order[i - T.base] = si;
        T.segw[i - T.base] = make_int4(g.x, g.y, g.z, si);
    }
}

// {row, begin, end, 0} of every row of both CSRs in degree order
template <typename P>
__global__ void row_table_kernel(const P* ptr0, const int32_t* perm0, int64_t n0, int4* rowt0, const P* ptr1,
                                 const int32_t* perm1, int64_t n1, int4* rowt1) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n0 + n1;
         i += (int64_t)gridDim.x * blockDim.x) {
        const bool second = i >= n0;
        const int64_t k = second ? i - n0 : i;
        const P* ptr = second ? ptr1 : ptr0;
        const int32_t r = (second ? perm1 : perm0)[k];
        (second ? rowt1 : rowt0)[k] = make_int4(r, (int32_t)ptr[r], (int32_t)ptr[r + 1], 0);
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// host launchers

int key_bits(uint64_t max_key) { return max_key == 0 ? 0 : 64 - __builtin_clzll(max_key); }

namespace {

// passes of a sort by `bits` bits; they write out and tmp in turn, the last one out
int radix_passes(int bits) { return std::max(1, (bits + RS_BITS - 1) / RS_BITS); }

int rs_steps(int64_t n) { return n <= (int64_t)RS_DIRECT * rs_tile(4) ? 4 : 16; }

hipError_t scan_exclusive_u32(uint32_t* x, int64_t n, uint32_t* part, hipStream_t s) {
    const unsigned tiles = tiles_of(n, SCAN_TILE);
    hipLaunchKernelGGL(scan_reduce_kernel, dim3(tiles), dim3(SCAN_BLOCK), 0, s, x, n, part);
    hipLaunchKernelGGL(scan_carry_kernel, dim3(1), dim3(SCAN_BLOCK), 0, s, part, (int64_t)tiles);
    hipLaunchKernelGGL(scan_apply_kernel, dim3(tiles), dim3(SCAN_BLOCK), 0, s, x, n, part);
    return hipGetLastError();
}

}  // namespace

size_t radix_scratch_words(int64_t n0, int64_t n1) {
    // enough for any smaller sorts too (a smaller one may take smaller tiles)
    auto tiles = [](int64_t n) {
        return std::max<int64_t>(tiles_of(n, rs_tile(16)), std::min<int64_t>(tiles_of(n, rs_tile(4)), RS_DIRECT));
    };
    const int64_t hist = RS_DIGITS * (tiles(n0) + tiles(n1));
    return (size_t)(hist + tiles_of(hist, SCAN_TILE) + 64);
}

hipError_t radix_sort(const RadixSort* sorts, int n_sorts, uint32_t* scratch, hipStream_t s) {
    int64_t most = 0;
    int passes = 1;
    for (int q = 0; q < n_sorts; ++q) {
        most = std::max(most, sorts[q].n);
        if (sorts[q].n > 0) passes = std::max(passes, radix_passes(sorts[q].bits));
    }
    if (most <= 0) return hipSuccess;
    const int steps = rs_steps(most);
    RadixArrays src[2] = {};
    int shift[2] = {0, 0};
    for (int q = 0; q < n_sorts; ++q) src[q] = sorts[q].in;
    const bool two = sorts[0].in.v1 != nullptr;
    for (int pass = 0; pass < passes; ++pass) {
        RsArgs A{};
        A.hist = scratch;
        int64_t words = 0, before = 0, tiles = 0;
        A.direct = (int64_t)tiles_of(most, rs_tile(steps)) <= RS_DIRECT;
        for (int q = 0; q < n_sorts; ++q) {
            const RadixSort& R = sorts[q];
            RsJob& J = A.job[q];
            // the passes share the bits evenly; the last one lands in the
            // output.  A sort of fewer bits takes smaller digits (of 0 bits
            // too: a stable copy), so that both end in the same pass.
            const int db = (R.bits - shift[q] + passes - pass - 1) / (passes - pass);
            const RadixArrays& dst = ((passes - 1 - pass) % 2) == 0 ? R.out : R.tmp;
            J.key = src[q].key;
            J.v0 = src[q].v0;
            J.v1 = src[q].v1;
            J.key_out = dst.key;
            J.out0 = dst.v0;
            J.out1 = dst.v1;
            J.n = R.n;
            J.n_tiles = (int32_t)tiles_of(R.n, rs_tile(steps));
            J.shift = shift[q];
            J.bits = db;
            J.hist = words;
            J.before = (uint32_t)before;
            words += (int64_t)J.n_tiles << db;
            before += R.n;
            tiles += J.n_tiles;
            shift[q] += db;
            src[q] = dst;
        }
        const dim3 grid((unsigned)tiles), block(RS_BLOCK);
        if (steps == 4) hipLaunchKernelGGL(rs_count_kernel<4>, grid, block, 0, s, A);
        else hipLaunchKernelGGL(rs_count_kernel<16>, grid, block, 0, s, A);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess && !A.direct) e = scan_exclusive_u32(scratch, words, scratch + words, s);
        if (e != hipSuccess) return e;
        if (steps == 4) {
            if (two) hipLaunchKernelGGL((rs_scatter_kernel<2, 4>), grid, block, 0, s, A);
            else hipLaunchKernelGGL((rs_scatter_kernel<1, 4>), grid, block, 0, s, A);
        } else {
            if (two) hipLaunchKernelGGL((rs_scatter_kernel<2, 16>), grid, block, 0, s, A);
            else hipLaunchKernelGGL((rs_scatter_kernel<1, 16>), grid, block, 0, s, A);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_rows(const RowsJob& a, const RowsJob& b, int ptr64, int64_t n_edges, hipStream_t s) {
    dim3 grid(grid_1d(a.n_rows + b.n_rows + 2)), block(256);
    if (ptr64) hipLaunchKernelGGL(rows_kernel<int64_t>, grid, block, 0, s, a, b, n_edges);
    else hipLaunchKernelGGL(rows_kernel<int32_t>, grid, block, 0, s, a, b, n_edges);
    return hipGetLastError();
}

hipError_t launch_edge_ids(const int32_t* out_eid, int32_t* pos, const int32_t* in_eid, int64_t n, int32_t* flag,
                           int32_t bit, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(edge_ids_kernel, dim3(grid_1d(n)), dim3(256), 0, s, out_eid, pos, in_eid, n, flag, bit);
    return hipGetLastError();
}

hipError_t launch_summary(const SummaryArgs& a, hipStream_t s) {
    const unsigned n = SUMMARY_TABLES + tiles_of(2 * SUMMARY_SAMPLES + 2 * (SUMMARY_DEG + 1), SUMMARY_BLOCK);
    hipLaunchKernelGGL(summary_kernel, dim3(n), dim3(SUMMARY_BLOCK), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_check_permutation(const int32_t* eid, int64_t n, uint32_t* counts, int32_t* flag, int32_t bit,
                                    hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_1d(n)), dim3(256), 0, s, counts, n, 0u);
    hipLaunchKernelGGL(count_ids_kernel, dim3(grid_1d(n)), dim3(256), 0, s, eid, n, counts, flag, bit);
    hipLaunchKernelGGL(check_once_kernel, dim3(grid_1d(n)), dim3(256), 0, s, counts, n, flag, bit);
    return hipGetLastError();
}

hipError_t launch_edge_ends(const int32_t* idx, const int32_t* eid, const int32_t* row, int64_t n, int32_t* src_of_e,
                            int32_t* dst_of_e, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(edge_ends_kernel, dim3(grid_1d(n)), dim3(256), 0, s, idx, eid, row, n, src_of_e, dst_of_e);
    return hipGetLastError();
}

hipError_t launch_hub_tables(const HubArgs& a, int64_t n_seg, int id_bits, int drop, uint32_t* key, hipStream_t s) {
    hipLaunchKernelGGL(hub_offsets_kernel, dim3(SUMMARY_TABLES), dim3(SCAN_BLOCK), 0, s, a);
    if (n_seg > 0)
        hipLaunchKernelGGL(hub_segments_kernel, dim3(grid_1d(n_seg)), dim3(256), 0, s, a, n_seg, id_bits, drop,
                           key);
    return hipGetLastError();
}

hipError_t launch_seg_wave(const HubArgs& a, int64_t n_seg, const uint32_t* order, hipStream_t s) {
    if (n_seg <= 0) return hipSuccess;
    hipLaunchKernelGGL(seg_wave_kernel, dim3(grid_1d(n_seg)), dim3(256), 0, s, a, n_seg, order);
    return hipGetLastError();
}

hipError_t launch_row_table(const void* ptr0, const int32_t* perm0, int64_t n0, int4* rowt0, const void* ptr1,
                            const int32_t* perm1, int64_t n1, int4* rowt1, int ptr64, hipStream_t s) {
    if (n0 + n1 <= 0) return hipSuccess;
    dim3 grid(grid_1d(n0 + n1)), block(256);
    if (ptr64)
        hipLaunchKernelGGL(row_table_kernel<int64_t>, grid, block, 0, s, (const int64_t*)ptr0, perm0, n0, rowt0,
                           (const int64_t*)ptr1, perm1, n1, rowt1);
    else
        hipLaunchKernelGGL(row_table_kernel<int32_t>, grid, block, 0, s, (const int32_t*)ptr0, perm0, n0, rowt0,
                           (const int32_t*)ptr1, perm1, n1, rowt1);
    return hipGetLastError();
}

}  // namespace gnnk
