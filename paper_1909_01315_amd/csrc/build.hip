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
#include "device.h"

namespace gnnk {
namespace {

constexpr int RS_WAVES = 8;
constexpr int RS_BLOCK = RS_WAVES * 64;
constexpr int RS_STEPS = 16;                       // 64-key steps per wavefront
constexpr int RS_TILE = RS_WAVES * 64 * RS_STEPS;  // keys per workgroup
constexpr int RS_BITS = 9;                         // most bits of a digit
constexpr int RS_DIGITS = 1 << RS_BITS;
static_assert(RS_DIGITS == RS_BLOCK, "thread d of a workgroup handles digit d");
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = 256 * SCAN_ITEMS;

inline unsigned tiles_of(int64_t n, int64_t per) { return (unsigned)((n + per - 1) / per); }

inline unsigned grid_1d(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b > 65536) b = 65536;
    return (unsigned)(b > 0 ? b : 1);
}

// ---------------------------------------------------------------------------
// radix sort

__global__ __launch_bounds__(RS_BLOCK) void rs_count_kernel(const uint32_t* keys, int64_t n, int shift, int bits,
                                                            uint32_t* hist, int64_t n_tiles) {
    __shared__ uint32_t c[RS_DIGITS];
    const uint32_t mask = (1u << bits) - 1u;
    c[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
#pragma unroll
    for (int j = 0; j < RS_STEPS; ++j) {
        const int64_t i = base + j * RS_BLOCK + threadIdx.x;
        if (i < n) atomicAdd(&c[(keys[i] >> shift) & mask], 1u);
    }
    __syncthreads();
    if (threadIdx.x <= mask) hist[(int64_t)threadIdx.x * n_tiles + blockIdx.x] = c[threadIdx.x];
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

// hist holds the exclusive digit-major scan of the counts: the first output
// position of (digit, workgroup).  NV: arrays of values that move with the
// keys (v0 == nullptr stands for 0..n-1).  keys_out == nullptr drops the
// sorted keys.
template <int NV>
__global__ __launch_bounds__(RS_BLOCK) void rs_scatter_kernel(const uint32_t* keys, const uint32_t* v0,
                                                              const uint32_t* v1, int64_t n, int shift, int bits,
                                                              const uint32_t* hist, int64_t n_tiles,
                                                              uint32_t* keys_out, uint32_t* out0, uint32_t* out1) {
    __shared__ uint32_t cnt[RS_WAVES][RS_DIGITS];
    __shared__ uint32_t first[RS_DIGITS];  // output position of a digit's first key less its place in the tile
    __shared__ uint32_t wsum[RS_WAVES];
    __shared__ uint32_t stage[RS_TILE];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t mask = (1u << bits) - 1u;
    for (int i = threadIdx.x; i < RS_WAVES * RS_DIGITS; i += RS_BLOCK) (&cnt[0][0])[i] = 0u;
    __syncthreads();
    const int64_t tile = (int64_t)blockIdx.x * RS_TILE;
    const int64_t base = tile + (int64_t)w * (64 * RS_STEPS);
    const int m = (int)(n - tile < RS_TILE ? n - tile : RS_TILE);  // keys of this tile
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    uint32_t k[RS_STEPS], a[RS_STEPS], b[RS_STEPS], at[RS_STEPS];
#pragma unroll
    for (int j = 0; j < RS_STEPS; ++j) {
        const int64_t i = base + j * 64 + lane;
        const bool ok = i < n;
        k[j] = ok ? keys[i] : 0u;
        a[j] = ok ? (v0 ? v0[i] : (uint32_t)i) : 0u;
        b[j] = NV > 1 && ok ? v1[i] : 0u;
    }
#pragma unroll
    for (int j = 0; j < RS_STEPS; ++j) {
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
        uint32_t run = rs_exclusive(tot, wsum);
        first[d] = (d <= mask ? hist[(int64_t)d * n_tiles + blockIdx.x] : 0u) - run;
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
    for (int j = 0; j < RS_STEPS; ++j) {
        if (base + j * 64 + lane < n) {
            at[j] += cnt[w][(k[j] >> shift) & mask];
            stage[at[j]] = k[j];
        }
    }
    __syncthreads();
    uint32_t to[RS_STEPS];
#pragma unroll
    for (int j = 0; j < RS_STEPS; ++j) {
        const int i = j * RS_BLOCK + (int)threadIdx.x;
        to[j] = 0u;
        if (i < m) {
            const uint32_t key = stage[i];
            to[j] = first[(key >> shift) & mask] + (uint32_t)i;
            if (keys_out) keys_out[to[j]] = key;
        }
    }
    auto put = [&](const uint32_t* v, uint32_t* out) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RS_STEPS; ++j)
            if (base + j * 64 + lane < n) stage[at[j]] = v[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < RS_STEPS; ++j) {
            const int i = j * RS_BLOCK + (int)threadIdx.x;
            if (i < m) out[to[j]] = stage[i];
        }
    };
    put(a, out0);
    if constexpr (NV > 1) put(b, out1);
}

__global__ void copy_pairs_kernel(const uint32_t* keys, const uint32_t* v0, const uint32_t* v1, int64_t n,
                                  uint32_t* keys_out, uint32_t* out0, uint32_t* out1) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (keys_out) keys_out[i] = keys[i];
        out0[i] = v0 ? v0[i] : (uint32_t)i;
        if (v1) out1[i] = v1[i];
    }
}

// ---------------------------------------------------------------------------
// exclusive scan of uint32 counts (in place)

__device__ uint32_t block_exclusive(uint32_t v, uint32_t* total) {
    __shared__ uint32_t wsum[4];
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
    for (int i = 0; i < 4; ++i) {
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

__global__ __launch_bounds__(256) void scan_reduce_kernel(const uint32_t* x, int64_t n, uint32_t* part) {
    const int64_t b = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t s = 0u;
    for (int j = 0; j < SCAN_ITEMS; ++j)
        if (b + j < n) s += x[b + j];
    uint32_t total;
    (void)block_exclusive(s, &total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// one workgroup: the tile sums, scanned tile by tile with a running carry
__global__ __launch_bounds__(256) void scan_carry_kernel(uint32_t* part, int64_t n) {
    uint32_t carry = 0u;
    for (int64_t t = 0; t < n; t += SCAN_TILE) carry += scan_tile(part, n, t, carry);
}

__global__ __launch_bounds__(256) void scan_apply_kernel(uint32_t* x, int64_t n, const uint32_t* part) {
    (void)scan_tile(x, n, (int64_t)blockIdx.x * SCAN_TILE, part[blockIdx.x]);
}

// ---------------------------------------------------------------------------
// structure from sorted keys

// offsets[r] = first position whose key is >= r, for r in [0, n_rows]
template <typename P>
__global__ void ptr_from_keys_kernel(const uint32_t* keys, int64_t n_keys, int64_t n_rows, P* ptr) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r <= n_rows;
         r += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = n_keys;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)keys[mid] < r) lo = mid + 1;
            else hi = mid;
        }
        ptr[r] = (P)lo;
    }
}

template <typename P>
__global__ void degree_kernel(const P* ptr, int64_t n_rows, int32_t* deg, uint32_t* deg_key, uint32_t cap) {
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n_rows;
         r += (int64_t)gridDim.x * blockDim.x) {
        const int32_t d = (int32_t)((int64_t)ptr[r + 1] - (int64_t)ptr[r]);
        deg[r] = d;
        deg_key[r] = cap - (uint32_t)d;
    }
}

// At most one atomic per wavefront that saw a difference, and none once the
// flag is seen set: all of them meet at one address (one per difference took
// about 20 ms for a shuffled list of 114.6M ids, one per wavefront 3 ms).
__global__ void check_identity_kernel(const int32_t* eid, int64_t n, int32_t* flag, int32_t bit) {
    bool off = false;
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x)
        off |= eid[p] != (int32_t)p;
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

template <typename P>
__global__ void hub_segments_kernel(const P* ptr, const int32_t* perm, const int32_t* hub_off, int64_t n_hub,
                                    int64_t seg_edges, int4* seg) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n_hub;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = perm[k];
        const int64_t b = (int64_t)ptr[r], e = (int64_t)ptr[r + 1];
        int32_t o = hub_off[k];
        for (int64_t s = b; s < e; s += seg_edges, ++o)
            seg[o] = make_int4(r, (int32_t)s, (int32_t)(s + seg_edges < e ? s + seg_edges : e), (int32_t)k);
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// host launchers

int key_bits(uint64_t max_key) { return max_key == 0 ? 0 : 64 - __builtin_clzll(max_key); }

size_t radix_scratch_words(int64_t n) {
    const int64_t hist = RS_DIGITS * (int64_t)tiles_of(n, RS_TILE);
    return (size_t)(hist + tiles_of(hist, SCAN_TILE) + 64);
}

hipError_t scan_exclusive_u32(uint32_t* x, int64_t n, uint32_t* part, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned tiles = tiles_of(n, SCAN_TILE);
    if (tiles <= 8) {
        // few counts: one workgroup scans them (one launch instead of three)
        hipLaunchKernelGGL(scan_carry_kernel, dim3(1), dim3(256), 0, s, x, n);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(scan_reduce_kernel, dim3(tiles), dim3(256), 0, s, x, n, part);
    hipLaunchKernelGGL(scan_carry_kernel, dim3(1), dim3(256), 0, s, part, (int64_t)tiles);
    hipLaunchKernelGGL(scan_apply_kernel, dim3(tiles), dim3(256), 0, s, x, n, part);
    return hipGetLastError();
}

hipError_t radix_sort(const RadixArrays& in, const RadixArrays& out, const RadixArrays& tmp, int64_t n, int bits,
                      uint32_t* scratch, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int passes = (bits + RS_BITS - 1) / RS_BITS;
    if (passes == 0) {
        hipLaunchKernelGGL(copy_pairs_kernel, dim3(grid_1d(n)), dim3(256), 0, s, in.key, in.v0, in.v1, n, out.key,
                           out.v0, out.v1);
        return hipGetLastError();
    }
    const int64_t n_tiles = tiles_of(n, RS_TILE);
    uint32_t* hist = scratch;
    uint32_t* part = scratch + RS_DIGITS * n_tiles;
    RadixArrays src = in;
    int shift = 0;
    for (int pass = 0; pass < passes; ++pass) {
        // the passes share the bits evenly; the last one lands in the output
        const int db = (bits - shift + passes - pass - 1) / (passes - pass);
        const bool last = pass == passes - 1;
        RadixArrays dst = ((passes - 1 - pass) % 2) == 0 ? out : tmp;
        const dim3 grid((unsigned)n_tiles), block(RS_BLOCK);
        hipLaunchKernelGGL(rs_count_kernel, grid, block, 0, s, src.key, n, shift, db, hist, n_tiles);
        hipError_t e = scan_exclusive_u32(hist, ((int64_t)1 << db) * n_tiles, part, s);
        if (e != hipSuccess) return e;
        uint32_t* keys_out = last ? out.key : dst.key;
        if (in.v1)
            hipLaunchKernelGGL(rs_scatter_kernel<2>, grid, block, 0, s, src.key, src.v0, src.v1, n, shift, db, hist,
                               n_tiles, keys_out, dst.v0, dst.v1);
        else
            hipLaunchKernelGGL(rs_scatter_kernel<1>, grid, block, 0, s, src.key, src.v0, nullptr, n, shift, db, hist,
                               n_tiles, keys_out, dst.v0, nullptr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        src = dst;
        shift += db;
    }
    return hipSuccess;
}

hipError_t launch_ptr_from_keys(const uint32_t* keys, int64_t n_keys, int64_t n_rows, void* ptr, int ptr64,
                                hipStream_t s) {
    dim3 grid(grid_1d(n_rows + 1)), block(256);
    if (ptr64)
        hipLaunchKernelGGL(ptr_from_keys_kernel<int64_t>, grid, block, 0, s, keys, n_keys, n_rows, (int64_t*)ptr);
    else
        hipLaunchKernelGGL(ptr_from_keys_kernel<int32_t>, grid, block, 0, s, keys, n_keys, n_rows, (int32_t*)ptr);
    return hipGetLastError();
}

hipError_t launch_degrees(const void* ptr, int ptr64, int64_t n_rows, int32_t* deg, uint32_t* deg_key, uint32_t cap,
                          hipStream_t s) {
    if (n_rows <= 0) return hipSuccess;
    dim3 grid(grid_1d(n_rows)), block(256);
    if (ptr64)
        hipLaunchKernelGGL(degree_kernel<int64_t>, grid, block, 0, s, (const int64_t*)ptr, n_rows, deg, deg_key, cap);
    else
        hipLaunchKernelGGL(degree_kernel<int32_t>, grid, block, 0, s, (const int32_t*)ptr, n_rows, deg, deg_key, cap);
    return hipGetLastError();
}

hipError_t launch_check_identity(const int32_t* eid, int64_t n, int32_t* flag, int32_t bit, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(check_identity_kernel, dim3(grid_1d(n)), dim3(256), 0, s, eid, n, flag, bit);
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

// sort key of each hub segment: the halves of its first and last neighbour
// id, summed (below the neighbour count, so it fits the key's bits)
__global__ void seg_keys_kernel(const int4* seg, int64_t n_seg, const int32_t* idx, uint32_t* key) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n_seg; k += (int64_t)gridDim.x * blockDim.x) {
        const int4 s = seg[k];
        key[k] = ((uint32_t)idx[s.y] >> 1) + ((uint32_t)idx[s.z - 1] >> 1);
    }
}

hipError_t launch_seg_keys(const int4* seg, int64_t n_seg, const int32_t* idx, uint32_t* key, hipStream_t s) {
    if (n_seg <= 0) return hipSuccess;
    hipLaunchKernelGGL(seg_keys_kernel, dim3(grid_1d(n_seg)), dim3(256), 0, s, seg, n_seg, idx, key);
    return hipGetLastError();
}

namespace {

// the segment of each hub-segment wavefront, with its table index: the walk
// then finds its segment with one load instead of two dependent ones
__global__ void seg_wave_kernel(const int4* seg, const int32_t* order, int64_t n_seg, int4* segw) {
    for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < n_seg; w += (int64_t)gridDim.x * blockDim.x) {
        const int32_t si = order[w];
        const int4 t = seg[si];
        segw[w] = make_int4(t.x, t.y, t.z, si);
    }
}

// {row, begin, end, 0} of every row in degree order
template <typename P>
__global__ void row_table_kernel(const P* ptr, const int32_t* perm, int64_t n_rows, int4* rowt) {
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n_rows; k += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = perm[k];
        rowt[k] = make_int4(r, (int32_t)ptr[r], (int32_t)ptr[r + 1], 0);
    }
}

}  // namespace

hipError_t launch_seg_wave(const int4* seg, const int32_t* order, int64_t n_seg, int4* segw, hipStream_t s) {
    if (n_seg <= 0) return hipSuccess;
    hipLaunchKernelGGL(seg_wave_kernel, dim3(grid_1d(n_seg)), dim3(256), 0, s, seg, order, n_seg, segw);
    return hipGetLastError();
}

hipError_t launch_row_table(const void* ptr, int ptr64, const int32_t* perm, int64_t n_rows, int4* rowt,
                            hipStream_t s) {
    if (n_rows <= 0) return hipSuccess;
    dim3 grid(grid_1d(n_rows)), block(256);
    if (ptr64)
        hipLaunchKernelGGL(row_table_kernel<int64_t>, grid, block, 0, s, (const int64_t*)ptr, perm, n_rows, rowt);
    else
        hipLaunchKernelGGL(row_table_kernel<int32_t>, grid, block, 0, s, (const int32_t*)ptr, perm, n_rows, rowt);
    return hipGetLastError();
}

hipError_t launch_hub_segments(const void* ptr, int ptr64, const int32_t* perm, const int32_t* hub_off, int64_t n_hub,
                               int64_t seg_edges, int4* seg, hipStream_t s) {
    if (n_hub <= 0) return hipSuccess;
    dim3 grid(grid_1d(n_hub)), block(256);
    if (ptr64)
        hipLaunchKernelGGL(hub_segments_kernel<int64_t>, grid, block, 0, s, (const int64_t*)ptr, perm, hub_off, n_hub,
                           seg_edges, seg);
    else
        hipLaunchKernelGGL(hub_segments_kernel<int32_t>, grid, block, 0, s, (const int32_t*)ptr, perm, hub_off, n_hub,
                           seg_edges, seg);
    return hipGetLastError();
}

}  // namespace gnnk
