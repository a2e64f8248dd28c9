// Graph handles of the gnnk library: the in-CSR, the reverse graph's CSR with
// the original edge ids (Appendix B, definition of the reverse graph), the
// degree arrays, rows sorted by degree, and the segment tables of hub rows.
//
// Every structure is built on the device (build.hip: stable radix sorts, so
// the edges of a node keep ascending edge id) into the caller's workspace.
// The host reads back only a summary (a flag word, and how many rows are
// longer than each threshold a schedule can ask for), which places the role
// boundaries of the schedules and sizes the hub tables.
#include <stddef.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>

#include "host.h"

namespace gnnk {

// ---------------------------------------------------------------------------
// errors and options

static thread_local char g_err[512];
// bytes of scratch the last call on this thread that ran short asked for
static thread_local size_t g_need = 0;
static thread_local bool g_plan = false;
static thread_local size_t g_plan_peak = 0;

gnnk_status fail(gnnk_status st, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return st;
}

gnnk_status hip_fail(hipError_t e, const char* what) {
    return fail(GNNK_EHIP, "%s: %s (%d)", what, hipGetErrorString(e), (int)e);
}

void clear_error() {
    g_err[0] = 0;
    g_need = 0;
}

Options& options() {
    static Options o;
    return o;
}

int64_t seg_edges_for(int64_t E, bool reverse) {
    if (options().seg_edges > 0) return options().seg_edges;
    // in-CSR segments of 512 edges: on the 114.6M-edge graph the gathers of
    // the in-CSR passes take 0.15-0.37 ms less each than with 2048 (more of
    // every hub row runs in narrow, source-ordered pieces); the reverse
    // passes gain nothing from it (copy_e sums and the argmax scatter lose)
    const int64_t cap = reverse ? 2048 : 512, div = reverse ? 2048 : 8192;
    int64_t S = 64;
    while (S < cap && S * div < E) S <<= 1;
    return S;
}

int64_t seg_edges_fine_for(int64_t E) {
    if (options().seg_edges > 0) return options().seg_edges;
    // the reverse passes that gather node rows (dX of the sums, the fused
    // attention's source pass) run faster on 256-edge pieces of the hub rows
    // (c3 dX of u_mul_e/sum 5.53 -> 5.06 ms); the copy_e sums and the argmax
    // scatter keep the coarser table
    int64_t S = 64;
    while (S < 256 && S * 16384 < E) S <<= 1;
    return S;
}

int64_t Dir::count_above(int64_t t) const {
    if (t < 0) return n_rows;
    // every threshold a call uses is at most SUMMARY_DEG (the small-row
    // option's limit), or the table's own segment size or far_deg
    if (t > SUMMARY_DEG) return t == far_deg ? n_far : n_hub;
    return above.empty() ? 0 : above[(size_t)t];
}

void* Scratch::take(size_t n) {
    const size_t at = used;
    used += (n + 255) / 256 * 256;
    if (g_plan) {
        if (used > g_plan_peak) g_plan_peak = used;
        return base + at;
    }
    if (used > bytes) {
        g_need = used;
        return nullptr;
    }
    return base + at;
}

Scratch scratch_of(gnnk_graph* g, hipStream_t s) {
    Scratch sc;
    if (g_plan) {
        // a stand-in that no kernel sees: nothing is launched while planning
        sc.base = reinterpret_cast<char*>((uintptr_t)1 << 20);
        sc.bytes = SIZE_MAX;
        return sc;
    }
    std::lock_guard<std::mutex> lk(g->lent_mu);
    for (int k = 0; k < g->n_lent; ++k)
        if (g->lent[k].stream == s) {
            sc.base = g->lent[k].buf;
            sc.bytes = g->lent[k].bytes;
        }
    return sc;
}

bool planning() { return g_plan; }

gnnk_status planned(gnnk_graph* g, hipStream_t s, const std::function<gnnk_status()>& run) {
    if (g_plan) return run();
    g_plan = true;
    g_plan_peak = 0;
    const gnnk_status st = run();
    g_plan = false;
    if (st != GNNK_OK) return st;
    Scratch have = g ? scratch_of(g, s) : Scratch{};
    if (g_plan_peak > have.bytes) {
        g_need = g_plan_peak;
        return scratch_fail(have);
    }
    return run();
}

gnnk_status scratch_fail(const Scratch& sc) {
    return fail(GNNK_ENOMEM,
                "the call needs at least %zu bytes of scratch on its stream and has %zu: lend a larger buffer with "
                "graph_attach_scratch (graph_scratch_bytes gives a bound, gnnk_scratch_needed this call's need)",
                g_need, sc.bytes);
}

// ---------------------------------------------------------------------------
// workspace layout

namespace {

constexpr size_t ALIGN = 256;

// flag bits of the validation and build kernels
constexpr int32_t FLAG_INDEX = 1;     // an endpoint or index out of range
constexpr int32_t FLAG_PTR = 2;       // row offsets not a valid CSR
constexpr int32_t FLAG_PERM = 4;      // edge ids not a permutation
constexpr int32_t FLAG_NOT_IDENT = 8; // edge ids differ from in-CSR positions

// What a handle keeps in the caller's workspace: fixed-size regions first,
// then the hub tables whose sizes are known only once the degrees are sorted.
struct Layout {
    size_t in_ptr = 0, in_idx = 0, in_eid = 0, out_ptr = 0, out_idx = 0, out_eid = 0;
    size_t in_deg = 0, out_deg = 0, in_perm = 0, out_perm = 0, in_row = 0, out_row = 0, out_pos = 0, flag = 0;
    size_t in_hub = 0, out_hub = 0, in_seg = 0, out_seg = 0, in_sego = 0, out_sego = 0, total = 0;
    size_t fine_hub = 0, fine_seg = 0, fine_sego = 0;  // the reverse CSR's finer hub tables
    size_t in_rowt = 0, out_rowt = 0, in_segw = 0, out_segw = 0, fine_segw = 0;  // per-wavefront lookup tables
    size_t ifine_hub = 0, ifine_seg = 0, ifine_sego = 0, ifine_segw = 0;  // the in-CSR's finer hub tables
};

// Temporaries of a build, in a buffer that is the caller's again afterwards:
// within the workspace they were 20 bytes per edge on top of the 28 that a
// handle keeps, for as long as it lived.
struct TempLayout {
    size_t edge[5] = {};  // E words each: temporaries of the sorts
    size_t words = 0;     // radix-sort counts, degree sort keys
    size_t total = 0;
};

// Rows listed by neighbour id, in a buffer of their own that only graphs that
// keep such a listing ask for.
struct ListLayout {
    size_t idx[2] = {}, eid[2] = {};   // the in-CSR's and the reverse CSR's
    size_t sego[4] = {}, segw[4] = {};  // segment orders of the four hub tables
    size_t total = 0;
};

struct Bump {
    size_t off = 0;
    size_t take(size_t bytes) {
        size_t o = off;
        off += (bytes + ALIGN - 1) / ALIGN * ALIGN;
        return o;
    }
};

// segments a graph can have at most: hub rows have more than S edges, so at
// most E / S of them, and at most E / S + (hub rows) <= 2 E / S + 2 segments
int64_t max_segments(int64_t E, int64_t S) { return 2 * E / S + 2; }

size_t pad64(int64_t x) { return (size_t)((x + 63) / 64 * 64); }

// uint32 words of build temporaries beside the edge-sized ones: the counts of
// the edge sorts, or four arrays of both directions' rows and the counts of
// their degree sorts, or the counts of the segment sort (at most E / 4
// segments: 2 E / S + 2 in each of four tables, S >= 32, none below 33 edges)
size_t build_tmp_words(int64_t n_src, int64_t n_dst, int64_t E) {
    return std::max({radix_scratch_words(E, E),
                     4 * (pad64(n_src) + pad64(n_dst)) + radix_scratch_words(n_dst, n_src),
                     radix_scratch_words(E / 4 + 64, 0)});
}

Layout make_layout(int64_t n_src, int64_t n_dst, int64_t E, size_t ps, int64_t hub_in, int64_t hub_out, int64_t seg_in,
                   int64_t seg_out, int64_t hub_fine = 0, int64_t seg_fine = 0,
                   int64_t hub_ifine = 0, int64_t seg_ifine = 0) {
    Layout L;
    Bump b;
    L.in_ptr = b.take((size_t)(n_dst + 1) * ps);
    L.in_idx = b.take((size_t)E * 4);
    L.in_eid = b.take((size_t)E * 4);
    L.out_ptr = b.take((size_t)(n_src + 1) * ps);
    L.out_idx = b.take((size_t)E * 4);
    L.out_eid = b.take((size_t)E * 4);
    L.in_deg = b.take((size_t)n_dst * 4);
    L.out_deg = b.take((size_t)n_src * 4);
    L.in_perm = b.take((size_t)n_dst * 4);
    L.out_perm = b.take((size_t)n_src * 4);
    L.in_row = b.take((size_t)E * 4);
    L.out_row = b.take((size_t)E * 4);
    L.out_pos = b.take((size_t)E * 4);
    L.flag = b.take(sizeof(BuildSummary));
    L.in_rowt = b.take((size_t)n_dst * 16);
    L.out_rowt = b.take((size_t)n_src * 16);
    L.in_hub = b.take((size_t)(hub_in + 1) * 4);
    L.out_hub = b.take((size_t)(hub_out + 1) * 4);
    L.in_seg = b.take((size_t)seg_in * 16);
    L.out_seg = b.take((size_t)seg_out * 16);
    L.in_sego = b.take((size_t)seg_in * 4);
    L.out_sego = b.take((size_t)seg_out * 4);
    L.fine_hub = b.take((size_t)(hub_fine + 1) * 4);
    L.fine_seg = b.take((size_t)seg_fine * 16);
    L.fine_sego = b.take((size_t)seg_fine * 4);
    L.in_segw = b.take((size_t)seg_in * 16);
    L.out_segw = b.take((size_t)seg_out * 16);
    L.fine_segw = b.take((size_t)seg_fine * 16);
    L.ifine_hub = b.take((size_t)(hub_ifine + 1) * 4);
    L.ifine_seg = b.take((size_t)seg_ifine * 16);
    L.ifine_sego = b.take((size_t)seg_ifine * 4);
    L.ifine_segw = b.take((size_t)seg_ifine * 16);
    L.total = b.off;
    return L;
}

TempLayout make_temp(int64_t n_src, int64_t n_dst, int64_t E) {
    TempLayout T;
    Bump b;
    for (size_t& o : T.edge) o = b.take((size_t)E * 4);
    T.words = b.take(build_tmp_words(n_src, n_dst, E) * 4);
    T.total = b.off;
    return T;
}

ListLayout make_lists(int64_t E, bool in, bool out, const int64_t* segs) {
    ListLayout N;
    Bump b;
    for (int d = 0; d < 2; ++d) {
        const bool has = d ? out : in;
        N.idx[d] = b.take(has ? (size_t)E * 4 : 0);
        N.eid[d] = b.take(has ? (size_t)E * 4 : 0);
        for (int t = 2 * d; t < 2 * d + 2; ++t) {
            N.sego[t] = b.take(has ? (size_t)segs[t] * 4 : 0);
            N.segw[t] = b.take(has ? (size_t)segs[t] * 16 : 0);
        }
    }
    N.total = b.off;
    return N;
}

// Edge ids and CSR positions are int32.  The walks advance a position past a
// row's end by at most 64 lane groups x 4 slots before testing it, so edge
// counts stay 2^16 below the int32 limit and no position arithmetic wraps.
constexpr int64_t MAX_EDGES = (int64_t)INT32_MAX - 65536;

bool sizes_ok(int64_t n_src, int64_t n_dst, int64_t E) {
    return n_src >= 0 && n_dst >= 0 && E >= 0 && n_src < INT32_MAX && n_dst < INT32_MAX && E <= MAX_EDGES;
}

// edges from which the segments of hub rows are ordered by the neighbours they
// cover: below it a graph has at most 4 x 2^20 / 32 segments, few enough to be
// in flight together, and the sort's launches would be a good part of a
// mini-batch block's build
int64_t order_edges() { return options().order_edges > 0 ? options().order_edges : (int64_t)1 << 20; }

// the longest rows that the edge softmax still gives to one wavefront
int64_t far_degree(const gnnk_graph* g) { return std::max<int64_t>(g->seg_edges, 2048); }

// bits of a row id below n_rows
int row_bits(int64_t n_rows) { return key_bits(n_rows > 1 ? (uint64_t)(n_rows - 1) : 0); }

struct Builder {
    gnnk_graph* g;
    gnnk_build_memory mem;
    hipStream_t s;
    char* W = nullptr;          // the workspace
    char* T = nullptr;          // the temporaries
    char* N = nullptr;          // the rows listed by neighbour
    Layout L;
    TempLayout TL;
    ListLayout NL;
    uint32_t* scratch = nullptr;
    hipError_t err = hipSuccess;

    void chk(hipError_t x) {
        if (err == hipSuccess) err = x;
    }
    template <typename T>
    T* at(size_t off) {
        return reinterpret_cast<T*>(W + off);
    }
    int32_t read_flag() {
        int32_t h = 0;
        chk(hipMemcpyAsync(&h, g->flag, 4, hipMemcpyDeviceToHost, s));
        chk(hipStreamSynchronize(s));
        return h;
    }

    uint32_t* edge_tmp(int k) { return reinterpret_cast<uint32_t*>(T + TL.edge[k]); }
    template <typename X>
    X* list(size_t off) {
        return reinterpret_cast<X*>(N + off);
    }

    // edges sorted stably by `row_of_e`: {row, edge id, other endpoint} per position
    static RadixSort edge_sort(const int32_t* row_of_e, const int32_t* other_of_e, int64_t E, int bits,
                               const RadixArrays& out, const RadixArrays& tmp) {
        auto u = [](const int32_t* p) { return const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(p)); };
        return {{u(row_of_e), nullptr, u(other_of_e)}, out, tmp, E, bits};
    }
    RadixSort in_sort(const int32_t* src_of_e, const int32_t* dst_of_e) {
        return edge_sort(dst_of_e, src_of_e, g->n_edges, row_bits(g->n_dst),
                         {at<uint32_t>(L.in_row), at<uint32_t>(L.in_eid), at<uint32_t>(L.in_idx)},
                         {edge_tmp(2), edge_tmp(3), edge_tmp(4)});
    }
    // the reverse graph's CSR from the source and destination of every edge id
    RadixSort out_sort(const int32_t* src_of_e, const int32_t* dst_of_e) {
        Dir& d = g->out;
        d.ptr = W + L.out_ptr;
        d.idx = at<int32_t>(L.out_idx);
        d.eid = at<int32_t>(L.out_eid);
        d.row = at<int32_t>(L.out_row);
        d.pos = at<int32_t>(L.out_pos);
        return edge_sort(src_of_e, dst_of_e, g->n_edges, row_bits(g->n_src),
                         {at<uint32_t>(L.out_row), at<uint32_t>(L.out_eid), at<uint32_t>(L.out_idx)},
                         {at<uint32_t>(L.out_pos), edge_tmp(0), edge_tmp(1)});
    }

    // The common tail: row offsets, degrees and rows by descending degree
    // (ties by row id) of both CSRs, the read-back, and the tables.  coo:
    // the in-CSR's offsets are not built yet and its edge ids not checked.
    gnnk_status finish(bool coo) {
        const int64_t E = g->n_edges;
        Dir& in = g->in;
        Dir& out = g->out;
        in.n_rows = g->n_dst;
        out.n_rows = g->n_src;
        out.reverse = true;
        in.deg = at<int32_t>(L.in_deg);
        out.deg = at<int32_t>(L.out_deg);
        in.perm = at<int32_t>(L.in_perm);
        out.perm = at<int32_t>(L.out_perm);
        if (coo) chk(launch_edge_ids(nullptr, nullptr, in.eid, E, g->flag, FLAG_NOT_IDENT, s));
        const size_t pi = pad64(g->n_dst), po = pad64(g->n_src);
        uint32_t* k0 = scratch;            // degree keys: the in-CSR's arrays
        uint32_t* k1 = scratch + 4 * pi;   // and the reverse CSR's
        uint32_t* rs = k1 + 4 * po;
        // (an offset array that the caller gave is only read)
        chk(launch_rows({coo ? at<uint32_t>(L.in_row) : nullptr, const_cast<void*>(in.ptr), in.deg, k0, in.n_rows},
                        {at<uint32_t>(L.out_row), const_cast<void*>(out.ptr), out.deg, k1, out.n_rows}, g->ptr64, E,
                        s));
        auto by_degree = [&](uint32_t* k, size_t pad, Dir& d) -> RadixSort {
            return {{k, nullptr, nullptr}, {k + pad, reinterpret_cast<uint32_t*>(d.perm), nullptr},
                    {k + 2 * pad, k + 3 * pad, nullptr}, d.n_rows, key_bits((uint64_t)E)};
        };
        const RadixSort deg_sorts[2] = {by_degree(k0, pi, in), by_degree(k1, po, out)};
        chk(radix_sort(deg_sorts, 2, rs, s));
        SummaryArgs sa{};
        sa.sorted[0] = k0 + pi;
        sa.sorted[1] = k1 + po;
        sa.n_rows[0] = in.n_rows;
        sa.n_rows[1] = out.n_rows;
        sa.n_edges = E;
        sa.seg_edges[0] = g->seg_edges;
        sa.seg_edges[1] = g->seg_edges_in_fine;
        sa.seg_edges[2] = g->seg_edges_out;
        sa.seg_edges[3] = g->seg_edges_fine;
        sa.far[0] = sa.far[1] = in.far_deg = out.far_deg = far_degree(g);
        if (E >= order_edges()) {
            sa.eid[0] = in.eid;
            sa.eid[1] = out.eid;
        }
        sa.out = reinterpret_cast<BuildSummary*>(g->flag);
        chk(launch_summary(sa, s));
        BuildSummary sum;
        chk(hipMemcpyAsync(&sum, g->flag, sizeof(sum), hipMemcpyDeviceToHost, s));
        chk(hipStreamSynchronize(s));
        if (err != hipSuccess) return hip_fail(err, "graph build");
        // nothing so far indexes with an endpoint, so that an edge list is
        // refused here, in the same read-back
        if (sum.flag & FLAG_INDEX) return fail(GNNK_EINVAL, "an edge has an endpoint out of range");
        if (coo) {
            g->identity_eids = !(sum.flag & FLAG_NOT_IDENT);
            if (g->identity_eids) in.eid = nullptr;
        }
        for (int d = 0; d < 2; ++d) {
            Dir& x = d ? out : in;
            x.max_deg = sum.max_deg[d];
            x.n_far = sum.above_far[d];
            x.above.assign(sum.above[d], sum.above[d] + SUMMARY_DEG + 1);
            x.n_nz = x.above[0];
            x.n_hub = sum.n_hub[2 * d];
            x.n_seg = sum.n_seg[2 * d];
        }
        // the finer tables: the same arrays but for the hub rows and segments
        Dir& fine = g->out_fine;
        Dir& ifine = g->in_fine;
        const bool finer = g->seg_edges_fine < g->seg_edges_out, ifiner = g->seg_edges_in_fine < g->seg_edges;
        fine = out;
        ifine = in;
        if (ifiner) {
            ifine.n_hub = sum.n_hub[1];
            ifine.n_seg = sum.n_seg[1];
        }
        if (finer) {
            fine.n_hub = sum.n_hub[3];
            fine.n_seg = sum.n_seg[3];
        }
        // (the rule and its figures: list_by_neighbour)
        const bool scattered = 2 * std::max(sum.near_ids[0], sum.near_ids[1]) < SUMMARY_SAMPLES;
        auto worth = [&](const Dir& f, int64_t S) {
            return in.eid && scattered && E >= order_edges() && 4 * f.n_seg * S >= E;
        };
        bool nbr_in = worth(ifine, g->seg_edges_in_fine), nbr_out = worth(fine, g->seg_edges_fine);
        if (const int64_t o = options().neighbour_lists; o >= 0) {
            nbr_in = in.eid && (o & 1);
            nbr_out = in.eid && (o & 2);
        }
        const int64_t segs[4] = {in.n_seg, ifiner ? ifine.n_seg : 0, out.n_seg, finer ? fine.n_seg : 0};
        L = make_layout(g->n_src, g->n_dst, E, g->ptr64 ? 8 : 4, in.n_hub, out.n_hub, segs[0], segs[2],
                        finer ? fine.n_hub : 0, segs[3], ifiner ? ifine.n_hub : 0, segs[1]);
        if (mem.workspace_bytes < L.total) return short_of_memory(L.total);
        if (nbr_in || nbr_out) {
            // optional memory: a caller without it gets a graph without listings
            NL = make_lists(E, nbr_in, nbr_out, segs);
            N = mem.lists ? reinterpret_cast<char*>(mem.lists(mem.ctx, NL.total)) : nullptr;
            if ((uintptr_t)N % ALIGN) return fail(GNNK_EINVAL, "memory for neighbour lists must be 256-byte aligned");
            if (!N) nbr_in = nbr_out = false;
        }
        in.rowt = ifine.rowt = at<int4>(L.in_rowt);
        out.rowt = fine.rowt = at<int4>(L.out_rowt);
        chk(launch_row_table(in.ptr, in.perm, in.n_rows, in.rowt, out.ptr, out.perm, out.n_rows, out.rowt, g->ptr64,
                             s));
        list_by_neighbour(nbr_in, nbr_out);
        // H: the tables in the order the gathers take them; K: the same
        // segments in table order for the passes that keep the edge-id order
        HubArgs H{}, K{};
        int64_t n_seg = 0, n_keep = 0;
        auto table = [&](int t, Dir& d, Dir& by, bool nbr, bool own, size_t hub, size_t seg, size_t sego, size_t segw,
                         int64_t S) {
            const int64_t n_own = own ? d.n_seg : 0;
            d.hub_off = at<int32_t>(hub);
            d.seg = at<int4>(seg);
            d.seg_order = at<int32_t>(sego);
            d.segw = at<int4>(segw);
            const int32_t* idx = nbr ? by.idx : d.idx;
            const int32_t* eid = nbr ? by.eid : d.eid;
            K.table[t] = {d.rowt, d.idx, d.hub_off, d.seg, d.seg_order, d.segw, own ? d.n_hub : 0, S, n_keep};
            by = d;
            by.idx = idx;
            by.eid = eid;
            if (nbr) {
                by.seg_order = list<int32_t>(NL.sego[t]);
                by.segw = list<int4>(NL.segw[t]);
                n_keep += n_own;
            }
            H.table[t] = {by.rowt, by.idx, by.hub_off, by.seg, by.seg_order, by.segw, own ? by.n_hub : 0, S, n_seg};
            n_seg += n_own;
        };
        table(0, in, g->in_nbr, nbr_in, true, L.in_hub, L.in_seg, L.in_sego, L.in_segw, g->seg_edges);
        g->in_fine_nbr.idx = g->in_nbr.idx;
        g->in_fine_nbr.eid = g->in_nbr.eid;
        table(1, ifine, g->in_fine_nbr, nbr_in, ifiner, L.ifine_hub, L.ifine_seg, L.ifine_sego, L.ifine_segw,
              g->seg_edges_in_fine);
        table(2, out, g->out_nbr, nbr_out, true, L.out_hub, L.out_seg, L.out_sego, L.out_segw, g->seg_edges_out);
        g->out_fine_nbr.idx = g->out_nbr.idx;
        g->out_fine_nbr.eid = g->out_nbr.eid;
        table(3, fine, g->out_fine_nbr, nbr_out, finer, L.fine_hub, L.fine_seg, L.fine_sego, L.fine_segw,
              g->seg_edges_fine);
        if (!ifiner) {
            ifine = in;
            g->in_fine_nbr = g->in_nbr;
        }
        if (!finer) {
            fine = out;
            g->out_fine_nbr = g->out_nbr;
        }
        build_segments(H, n_seg);
        chk(launch_seg_wave(K, n_keep, nullptr, s));
        // the position of each edge id in the reverse CSR that the max/min
        // backward walks (last: its array is a temporary of the edge sort)
        chk(launch_edge_ids(g->out_nbr.eid, out.pos, nullptr, E, g->flag, FLAG_NOT_IDENT, s));
        if (err != hipSuccess) return hip_fail(err, "graph build");
        g->ws_used = L.total;
        g->listed = (nbr_in ? 1 : 0) + (nbr_out ? 2 : 0);
        g->lists_bytes = g->listed ? NL.total : 0;
        return GNNK_OK;
    }

    gnnk_status short_of_memory(size_t need) {
        return fail(GNNK_ENOMEM, "workspace of %zu bytes is smaller than the %zu bytes this graph needs",
                    mem.workspace_bytes, need);
    }

    // A second listing of each row of a CSR, by neighbour id (ties by edge
    // id or position): the other CSR, whose positions are in neighbour order
    // already, sorted stably by its neighbour.  The passes that gather node
    // rows walk it where a graph's edge ids are scattered over its rows (an
    // edge list in arrival order): their hub segments then cover narrow
    // ranges of neighbours, as those of an edge list sorted by (destination,
    // source) do, and the edge operands and outputs, reached through the
    // edge ids, are as scattered in either order.  114.6M edges in arrival
    // order, 128 columns: the fused attention forward 7.26 -> 3.95 ms and the
    // two passes of its backward 7.23 + 7.22 -> 3.83 + 5.88 ms; 61.9M edges,
    // 100 columns: the mean 4.10 -> 3.35 ms and its gradient 5.13 -> 3.98 ms.
    // The build takes 3 ms more on 60M edges and 1.4 ms on 20M.
    //
    // A graph keeps such listings where at most half of the sampled edge ids
    // of either direction's rows lie next to each other.  60M edges, listed
    // against not: a list of shuffled pairs of neighbours, half of them
    // together, 8 x 16: u_mul_e/sum 3.51 -> 2.43 ms, its backward 7.24 ->
    // 4.82, u_dot_v 3.22 -> 2.02.  A list grouped by destination, the groups
    // in another order, reads its edge tensors in sequence and loses where
    // rows are narrow: 1 x 16: u_mul_e/sum 0.62 -> 0.84, u_dot_v 0.61 -> 0.98;
    // 8 x 2: 1.29 -> 1.52 and 1.53 -> 2.47.  A list sorted by source has its
    // in-rows in neighbour order as they are (nothing gained) and its reverse
    // rows' ids together: u_mul_e/sum backward, 8 x 2: 3.38 -> 3.76.  (Rows of
    // 128 columns and passes without an edge operand gain on such lists too,
    // the mean's gradient on the last 3.34 -> 1.75 with destinations in random
    // order; they run in edge-id order all the same.)
    // And where a direction's hub segments hold a quarter of its edges: 20M
    // edges on 1M nodes with a tenth, a quarter, half and nine tenths of them
    // there, 8 x 16: the mean 1.50 -> 1.43, 1.31 -> 1.23, 1.08 -> 1.01 and
    // 0.80 -> 0.65 ms, u_dot_v 2.30 -> 2.27, 2.14 -> 2.00, 1.86 -> 1.58 and
    // 1.33 -> 1.12: at a tenth a listing pays after some 25 passes, at a
    // quarter after 10 to 18.
    void list_by_neighbour(bool nbr_in, bool nbr_out) {
        auto u = [](const int32_t* p) { return const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(p)); };
        auto list_by = [&](int d, const Dir& other, int64_t n_rows, Dir& by) {
            by.idx = list<int32_t>(NL.idx[d]);
            by.eid = list<int32_t>(NL.eid[d]);
            const RadixSort r{{u(other.idx), u(other.eid), u(other.row)}, {edge_tmp(0), u(by.eid), u(by.idx)},
                              {edge_tmp(1), edge_tmp(2), edge_tmp(3)}, g->n_edges, row_bits(n_rows)};
            chk(radix_sort(&r, 1, scratch, s));
        };
        if (nbr_in) list_by(0, g->out, g->n_dst, g->in_nbr);
        if (nbr_out) list_by(1, g->in, g->n_src, g->out_nbr);
    }

    // The segments of hub rows and the order in which wavefronts take them:
    // by the neighbour ids a segment covers (its key, the halves of its
    // first and last neighbour id, summed), a stable sort, so equal keys keep
    // table order.  Where rows list their neighbours in ascending order, the
    // segments that run at the same time then gather from one slice of the
    // neighbour table; elsewhere the order changes nothing.  Results do not
    // depend on it (partials are combined in table order).  Graphs of few
    // edges keep table order: all their segments are in flight at once.
    void build_segments(const HubArgs& H, int64_t n_seg) {
        const bool ordered = n_seg > 0 && g->n_edges >= order_edges();
        // 32-bit keys: ids of more than 30 bits lose their lowest ones
        const int bits = row_bits(std::max(g->n_src, g->n_dst)), id_bits = std::min(bits, 30);
        // (fewer segments than edges: an edge-sized temporary holds an array)
        uint32_t* key = ordered ? edge_tmp(0) : nullptr;
        chk(launch_hub_tables(H, n_seg, id_bits, bits - id_bits, key, s));
        if (!ordered) {
            chk(launch_seg_wave(H, n_seg, nullptr, s));
            return;
        }
        // one sort of all tables, the table number above the neighbour ids
        const RadixSort r{{key, nullptr, nullptr}, {edge_tmp(1), edge_tmp(2), nullptr},
                          {edge_tmp(3), edge_tmp(4), nullptr}, n_seg, id_bits + 2};
        chk(radix_sort(&r, 1, scratch, s));
        chk(launch_seg_wave(H, n_seg, edge_tmp(2), s));
    }
};

// The handle owns no device memory (its arrays live in the caller's
// workspace, its scratch is lent by the caller), so destroying it is a host
// operation; kernels still in flight keep reading the caller's buffers.
void free_graph(gnnk_graph* g) { delete g; }

gnnk_graph* new_graph(int64_t num_src, int64_t num_dst, int64_t num_edges, gnnk_itype ptr_t) {
    gnnk_graph* g = new gnnk_graph();
    g->n_src = num_src;
    g->n_dst = num_dst;
    g->n_edges = num_edges;
    g->ptr64 = ptr_t == GNNK_I64;
    g->seg_edges = seg_edges_for(num_edges, false);
    g->seg_edges_out = seg_edges_for(num_edges, true);
    g->seg_edges_fine = seg_edges_fine_for(num_edges);
    g->seg_edges_in_fine = seg_edges_fine_for(num_edges);
    return g;
}

// memory checks shared by both constructors; fills b.W, b.T, b.L, g->flag
gnnk_status begin_build(Builder& b) {
    gnnk_graph* g = b.g;
    b.L = make_layout(g->n_src, g->n_dst, g->n_edges, g->ptr64 ? 8 : 4, 0, 0, 0, 0);
    b.TL = make_temp(g->n_src, g->n_dst, g->n_edges);
    if (!b.mem.workspace || b.mem.workspace_bytes < b.L.total) return b.short_of_memory(b.L.total);
    if (!b.mem.temp || b.mem.temp_bytes < b.TL.total)
        return fail(GNNK_ENOMEM, "temporaries of %zu bytes are smaller than the %zu bytes this build needs",
                    b.mem.temp_bytes, b.TL.total);
    b.W = reinterpret_cast<char*>(b.mem.workspace);
    b.T = reinterpret_cast<char*>(b.mem.temp);
    if ((uintptr_t)b.W % ALIGN) return fail(GNNK_EINVAL, "workspace must be 256-byte aligned");
    if ((uintptr_t)b.T % ALIGN) return fail(GNNK_EINVAL, "temporaries must be 256-byte aligned");
    b.scratch = reinterpret_cast<uint32_t*>(b.T + b.TL.words);
    g->flag = b.at<int32_t>(b.L.flag);
    b.chk(hipMemsetAsync(g->flag, 0, offsetof(BuildSummary, n_hub), b.s));  // the flag word and near_ids
    return GNNK_OK;
}

gnnk_status create_coo(Builder& b, const int32_t* src, const int32_t* dst) {
    gnnk_graph* g = b.g;
    const int64_t E = g->n_edges;
    gnnk_status st = begin_build(b);
    if (st != GNNK_OK) return st;
    b.chk(launch_validate(src, g->n_src, dst, g->n_dst, E, g->flag, b.s));
    const Layout& L = b.L;
    Dir& in = g->in;
    in.ptr = b.W + L.in_ptr;
    in.idx = b.at<int32_t>(L.in_idx);
    in.eid = b.at<int32_t>(L.in_eid);
    in.row = b.at<int32_t>(L.in_row);
    // both CSRs in the same launches: edges sorted by destination and by
    // source, ties in edge-id order
    const RadixSort sorts[2] = {b.in_sort(src, dst), b.out_sort(src, dst)};
    b.chk(radix_sort(sorts, 2, b.scratch, b.s));
    return b.finish(true);
}

gnnk_status create_csr(Builder& b, const void* indptr, const int32_t* indices, const int32_t* eids) {
    gnnk_graph* g = b.g;
    const int64_t E = g->n_edges;
    gnnk_status st = begin_build(b);
    if (st != GNNK_OK) return st;
    const Layout& L = b.L;
    b.chk(launch_validate_ptr(indptr, g->ptr64, g->n_dst, E, g->flag, b.s));
    b.chk(launch_validate(indices, g->n_src, nullptr, 0, E, g->flag, b.s));
    if (eids) {
        b.chk(launch_check_permutation(eids, E, b.at<uint32_t>(L.out_pos), g->flag, FLAG_PERM, b.s));
        b.chk(launch_edge_ids(nullptr, nullptr, eids, E, g->flag, FLAG_NOT_IDENT, b.s));
    }
    const int32_t h = b.read_flag();
    if (b.err != hipSuccess) return hip_fail(b.err, "checking the CSR");
    if (h & FLAG_PTR)
        return fail(GNNK_EINVAL, "indptr must start at 0, end at num_edges and never decrease");
    if (h & FLAG_INDEX) return fail(GNNK_EINVAL, "an index is out of range");
    if (h & FLAG_PERM) return fail(GNNK_EINVAL, "eids is not a permutation of 0..num_edges-1");
    const bool identity = !eids || !(h & FLAG_NOT_IDENT);
    g->identity_eids = identity;
    Dir& in = g->in;
    in.ptr = indptr;
    in.idx = indices;
    in.eid = identity ? nullptr : eids;
    in.row = b.at<int32_t>(L.in_row);
    b.chk(launch_fill_rows(indptr, g->ptr64, g->n_dst, E, in.row, b.s));
    const int32_t* src_of_e = indices;
    const int32_t* dst_of_e = in.row;
    if (!identity) {
        b.chk(launch_edge_ends(indices, eids, in.row, E, b.at<int32_t>(L.in_idx), b.at<int32_t>(L.in_eid), b.s));
        src_of_e = b.at<int32_t>(L.in_idx);
        dst_of_e = b.at<int32_t>(L.in_eid);
    }
    const RadixSort sort = b.out_sort(src_of_e, dst_of_e);
    b.chk(radix_sort(&sort, 1, b.scratch, b.s));
    return b.finish(false);
}

// the most that a handle of these sizes keeps, whatever its degrees
size_t kept_bound(int64_t num_src, int64_t num_dst, int64_t num_edges, gnnk_itype ptr_t) {
    // hub rows have more than S edges: at most E / S of them, and at most
    // E / S + (hub rows) <= 2 E / S segments
    const int64_t Si = seg_edges_for(num_edges, false), So = seg_edges_for(num_edges, true);
    const int64_t Sf = seg_edges_fine_for(num_edges);  // both CSRs' finer tables
    return make_layout(num_src, num_dst, num_edges, ptr_t == GNNK_I64 ? 8 : 4, num_edges / Si + 1,
                       num_edges / So + 1, max_segments(num_edges, Si), max_segments(num_edges, So),
                       Sf < So ? num_edges / Sf + 1 : 0, Sf < So ? max_segments(num_edges, Sf) : 0,
                       Sf < Si ? num_edges / Sf + 1 : 0, Sf < Si ? max_segments(num_edges, Sf) : 0)
        .total;
}

gnnk_status check_sizes(int64_t num_src, int64_t num_dst, int64_t num_edges, gnnk_itype ptr_t) {
    if (!sizes_ok(num_src, num_dst, num_edges))
        return fail(GNNK_EINVAL, "sizes out of range (node counts < 2^31 - 1, edges <= 2^31 - 2^16 - 1)");
    if (ptr_t != GNNK_I32 && ptr_t != GNNK_I64) return fail(GNNK_EINVAL, "bad ptr type");
    return GNNK_OK;
}

// one buffer for everything: the temporaries at its end
gnnk_build_memory one_buffer(int64_t num_src, int64_t num_dst, int64_t num_edges, void* workspace, size_t ws_bytes) {
    const size_t temp = make_temp(num_src, num_dst, num_edges).total;
    if (!workspace || ws_bytes < temp) return {workspace, ws_bytes, nullptr, 0, nullptr, nullptr};
    const size_t at = (ws_bytes - temp) / ALIGN * ALIGN;
    return {workspace, at, reinterpret_cast<char*>(workspace) + at, ws_bytes - at, nullptr, nullptr};
}

gnnk_status build_coo(int64_t num_src, int64_t num_dst, int64_t num_edges, const int32_t* src, const int32_t* dst,
                      gnnk_itype ptr_t, const gnnk_build_memory& mem, hipStream_t stream, gnnk_graph_t* out) {
    if (num_edges > 0 && (!src || !dst)) return fail(GNNK_EINVAL, "src/dst is NULL");
    Builder b{new_graph(num_src, num_dst, num_edges, ptr_t), mem, stream};
    const gnnk_status st = create_coo(b, src, dst);
    if (st != GNNK_OK) free_graph(b.g);
    else *out = b.g;
    return st;
}

gnnk_status build_csr(int64_t num_src, int64_t num_dst, int64_t num_edges, const void* indptr, gnnk_itype ptr_t,
                      const int32_t* indices, const int32_t* eids, const gnnk_build_memory& mem, hipStream_t stream,
                      gnnk_graph_t* out) {
    if (!indptr || (num_edges > 0 && !indices)) return fail(GNNK_EINVAL, "indptr/indices is NULL");
    Builder b{new_graph(num_src, num_dst, num_edges, ptr_t), mem, stream};
    const gnnk_status st = create_csr(b, indptr, indices, eids);
    if (st != GNNK_OK) free_graph(b.g);
    else *out = b.g;
    return st;
}

}  // namespace
}  // namespace gnnk

using namespace gnnk;

extern "C" {

gnnk_status graph_build_bytes(int64_t num_src, int64_t num_dst, int64_t num_edges, gnnk_itype ptr_t,
                              size_t* workspace, size_t* temp) {
    clear_error();
    if (!workspace || !temp) return fail(GNNK_EINVAL, "workspace or temp is NULL");
    const gnnk_status st = check_sizes(num_src, num_dst, num_edges, ptr_t);
    if (st != GNNK_OK) return st;
    *workspace = kept_bound(num_src, num_dst, num_edges, ptr_t);
    *temp = make_temp(num_src, num_dst, num_edges).total;
    return GNNK_OK;
}

gnnk_status graph_workspace_bytes(int64_t num_src, int64_t num_dst, int64_t num_edges, gnnk_itype ptr_t,
                                  size_t* bytes) {
    clear_error();
    if (!bytes) return fail(GNNK_EINVAL, "bytes is NULL");
    const gnnk_status st = check_sizes(num_src, num_dst, num_edges, ptr_t);
    if (st != GNNK_OK) return st;
    *bytes = kept_bound(num_src, num_dst, num_edges, ptr_t) + make_temp(num_src, num_dst, num_edges).total;
    return GNNK_OK;
}

gnnk_status graph_build_coo(int64_t num_src, int64_t num_dst, int64_t num_edges, const int32_t* src,
                            const int32_t* dst, gnnk_itype ptr_t, const gnnk_build_memory* mem, hipStream_t stream,
                            gnnk_graph_t* out) {
    clear_error();
    if (!mem || !out) return fail(GNNK_EINVAL, "mem or out is NULL");
    *out = nullptr;
    const gnnk_status st = check_sizes(num_src, num_dst, num_edges, ptr_t);
    return st == GNNK_OK ? build_coo(num_src, num_dst, num_edges, src, dst, ptr_t, *mem, stream, out) : st;
}

gnnk_status graph_build_csr(int64_t num_src, int64_t num_dst, int64_t num_edges, const void* indptr,
                            gnnk_itype ptr_t, const int32_t* indices, const int32_t* eids,
                            const gnnk_build_memory* mem, hipStream_t stream, gnnk_graph_t* out) {
    clear_error();
    if (!mem || !out) return fail(GNNK_EINVAL, "mem or out is NULL");
    *out = nullptr;
    const gnnk_status st = check_sizes(num_src, num_dst, num_edges, ptr_t);
    return st == GNNK_OK ? build_csr(num_src, num_dst, num_edges, indptr, ptr_t, indices, eids, *mem, stream, out)
                         : st;
}

gnnk_status graph_create_coo(int64_t num_src, int64_t num_dst, int64_t num_edges, const int32_t* src,
                             const int32_t* dst, gnnk_itype ptr_t, void* workspace, size_t ws_bytes,
                             hipStream_t stream, gnnk_graph_t* out) {
    clear_error();
    if (!out) return fail(GNNK_EINVAL, "out is NULL");
    *out = nullptr;
    gnnk_status st = check_sizes(num_src, num_dst, num_edges, ptr_t);
    if (st != GNNK_OK) return st;
    const gnnk_build_memory mem = one_buffer(num_src, num_dst, num_edges, workspace, ws_bytes);
    st = build_coo(num_src, num_dst, num_edges, src, dst, ptr_t, mem, stream, out);
    if (st == GNNK_OK) (*out)->one_buffer = true;
    return st;
}

gnnk_status graph_create_csr(int64_t num_src, int64_t num_dst, int64_t num_edges, const void* indptr,
                             gnnk_itype ptr_t, const int32_t* indices, const int32_t* eids, void* workspace,
                             size_t ws_bytes, hipStream_t stream, gnnk_graph_t* out) {
    clear_error();
    if (!out) return fail(GNNK_EINVAL, "out is NULL");
    *out = nullptr;
    gnnk_status st = check_sizes(num_src, num_dst, num_edges, ptr_t);
    if (st != GNNK_OK) return st;
    const gnnk_build_memory mem = one_buffer(num_src, num_dst, num_edges, workspace, ws_bytes);
    st = build_csr(num_src, num_dst, num_edges, indptr, ptr_t, indices, eids, mem, stream, out);
    if (st == GNNK_OK) (*out)->one_buffer = true;
    return st;
}

gnnk_status graph_info(gnnk_graph_t g, gnnk_graph_info* info) {
    clear_error();
    if (!g || !info) return fail(GNNK_EINVAL, "NULL argument");
    info->num_src = g->n_src;
    info->num_dst = g->n_dst;
    info->num_edges = g->n_edges;
    info->ptr_type = g->ptr64 ? GNNK_I64 : GNNK_I32;
    info->identity_eids = g->identity_eids;
    info->max_in_degree = g->in.max_deg;
    info->max_out_degree = g->out.max_deg;
    info->empty_dst_rows = g->n_dst - g->in.n_nz;
    info->empty_src_rows = g->n_src - g->out.n_nz;
    info->seg_edges = g->seg_edges;
    info->seg_edges_out = g->seg_edges_out;
    info->seg_edges_gather = g->seg_edges_fine;
    info->segments_gather = g->out_fine.n_seg;
    info->seg_edges_in_gather = g->seg_edges_in_fine;
    info->segments_in_gather = g->in_fine.n_seg;
    info->hub_dst_rows = g->in.n_hub;
    info->hub_src_rows = g->out.n_hub;
    info->segments_in = g->in.n_seg;
    info->segments_out = g->out.n_seg;
    info->workspace_bytes =
        g->ws_used + (g->one_buffer ? make_temp(g->n_src, g->n_dst, g->n_edges).total : 0);
    info->kept_bytes = g->ws_used;
    info->lists_bytes = g->lists_bytes;
    info->neighbour_lists = g->listed;
    info->reserved = 0;
    return GNNK_OK;
}

gnnk_status graph_in_degrees(gnnk_graph_t g, int32_t* out, hipStream_t stream) {
    clear_error();
    if (!g || (!out && g->n_dst > 0)) return fail(GNNK_EINVAL, "NULL argument");
    if (g->n_dst == 0) return GNNK_OK;
    hipError_t e = hipMemcpyAsync(out, g->in.deg, (size_t)g->n_dst * 4, hipMemcpyDeviceToDevice, stream);
    return e == hipSuccess ? GNNK_OK : hip_fail(e, "graph_in_degrees");
}

gnnk_status graph_out_degrees(gnnk_graph_t g, int32_t* out, hipStream_t stream) {
    clear_error();
    if (!g || (!out && g->n_src > 0)) return fail(GNNK_EINVAL, "NULL argument");
    if (g->n_src == 0) return GNNK_OK;
    hipError_t e = hipMemcpyAsync(out, g->out.deg, (size_t)g->n_src * 4, hipMemcpyDeviceToDevice, stream);
    return e == hipSuccess ? GNNK_OK : hip_fail(e, "graph_out_degrees");
}

gnnk_status graph_csr_export(gnnk_graph_t g, int reverse, void* indptr, int32_t* indices, int32_t* eids,
                             hipStream_t stream) {
    clear_error();
    if (!g) return fail(GNNK_EINVAL, "NULL graph");
    const Dir& d = reverse ? g->out : g->in;
    const int64_t E = g->n_edges;
    hipError_t e = hipSuccess;
    if (indptr) e = launch_copy_ptr(d.ptr, g->ptr64, indptr, g->ptr64, d.n_rows + 1, stream);
    if (e == hipSuccess && indices && E > 0)
        e = hipMemcpyAsync(indices, d.idx, (size_t)E * 4, hipMemcpyDeviceToDevice, stream);
    if (e == hipSuccess && eids && E > 0) {
        if (d.eid) e = hipMemcpyAsync(eids, d.eid, (size_t)E * 4, hipMemcpyDeviceToDevice, stream);
        else e = launch_iota(eids, E, stream);
    }
    return e == hipSuccess ? GNNK_OK : hip_fail(e, "graph_csr_export");
}

gnnk_status graph_validate(gnnk_graph_t g, hipStream_t stream) {
    clear_error();
    if (!g) return fail(GNNK_EINVAL, "NULL graph");
    hipError_t e = hipMemsetAsync(g->flag, 0, 4, stream);
    const int64_t E = g->n_edges;
    if (e == hipSuccess) e = launch_validate_ptr(g->in.ptr, g->ptr64, g->n_dst, E, g->flag, stream);
    if (e == hipSuccess) e = launch_validate_ptr(g->out.ptr, g->ptr64, g->n_src, E, g->flag, stream);
    if (e == hipSuccess) e = launch_validate(g->in.idx, g->n_src, g->out.idx, g->n_dst, E, g->flag, stream);
    if (e == hipSuccess) e = launch_validate(g->out.eid, E, g->in.eid, E, E, g->flag, stream);
    if (e == hipSuccess && g->listed)
        e = launch_validate(g->in_nbr.idx, g->n_src, g->out_nbr.idx, g->n_dst, E, g->flag, stream);
    if (e == hipSuccess && g->listed) e = launch_validate(g->out_nbr.eid, E, g->in_nbr.eid, E, E, g->flag, stream);
    int32_t h = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&h, g->flag, 4, hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return hip_fail(e, "graph_validate");
    if (h) return fail(GNNK_ERANGE, "graph has out-of-range entries (flags %d)", h);
    return GNNK_OK;
}

gnnk_status graph_destroy(gnnk_graph_t g) {
    clear_error();
    if (!g) return fail(GNNK_EINVAL, "NULL graph");
    free_graph(g);
    return GNNK_OK;
}

gnnk_status graph_attach_scratch(gnnk_graph_t g, hipStream_t stream, void* buf, size_t bytes) {
    clear_error();
    if (!g) return fail(GNNK_EINVAL, "NULL graph");
    if (bytes > 0 && !buf) return fail(GNNK_EINVAL, "buf is NULL");
    if ((uintptr_t)buf % ALIGN) return fail(GNNK_EINVAL, "scratch must be 256-byte aligned");
    std::lock_guard<std::mutex> lk(g->lent_mu);
    int k = 0;
    while (k < g->n_lent && g->lent[k].stream != stream) ++k;
    if (!buf || bytes == 0) {
        if (k < g->n_lent) g->lent[k] = g->lent[--g->n_lent];
        return GNNK_OK;
    }
    if (k == g->n_lent) {
        if (g->n_lent == gnnk_graph::MAX_STREAMS)
            return fail(GNNK_EINVAL, "a handle takes scratch for at most %d streams", gnnk_graph::MAX_STREAMS);
        ++g->n_lent;
    }
    g->lent[k] = {stream, reinterpret_cast<char*>(buf), bytes};
    return GNNK_OK;
}

gnnk_status gnnk_scratch_needed(size_t* bytes) {
    // not clear_error(): this reports on the previous call
    if (!bytes) return GNNK_EINVAL;
    *bytes = g_need;
    return GNNK_OK;
}

gnnk_status gnnk_set_option(const char* key, int64_t value) {
    clear_error();
    if (!key) return fail(GNNK_EINVAL, "NULL key");
    std::string k(key);
    if (k == "seg_edges") {
        if (value != 0 && (value < 32 || value > (1 << 30)))
            return fail(GNNK_EINVAL, "seg_edges is 0 (per graph, from its edge count) or in [32, 2^30]");
        options().seg_edges = value;
    } else if (k == "no_split") {
        if (value != 0 && value != 1) return fail(GNNK_EINVAL, "no_split is 0 or 1");
        options().no_split = value;
    } else if (k == "small_deg") {
        if (value < -1 || value > 4096) return fail(GNNK_EINVAL, "small_deg must be in [-1, 4096]");
        options().small_deg = value;
    } else if (k == "schedule") {
        if (value < 0 || value > 3) return fail(GNNK_EINVAL, "schedule is 0 (auto), 1 (row), 2 (edge) or 3 (edge, atomic)");
        options().schedule = value;
    } else if (k == "edge_chunk") {
        if (value != 0 && (value < 4 || value > (1 << 20) || value % 4))
            return fail(GNNK_EINVAL, "edge_chunk is 0 (auto) or a multiple of 4 in [4, 2^20]");
        options().edge_chunk = value;
    } else if (k == "fused_dw") {
        if (value < -1 || value > 1) return fail(GNNK_EINVAL, "fused_dw is -1 (auto), 0 or 1");
        options().fused_dw = value;
    } else if (k == "sddmm_split") {
        if (value < 0 || value > 8) return fail(GNNK_EINVAL, "sddmm_split is 0 (auto) or in [1, 8]");
        options().sddmm_split = value;
    } else if (k == "order_edges") {
        if (value < 0 || value > MAX_EDGES) return fail(GNNK_EINVAL, "order_edges is 0 (auto) or in [1, 2^31 - 2^16 - 1]");
        options().order_edges = value;
    } else if (k == "neighbour_lists") {
        if (value < -1 || value > 3) return fail(GNNK_EINVAL, "neighbour_lists is -1 (auto) or in [0, 3]");
        options().neighbour_lists = value;
    } else if (k == "no_fast") {
        if (value != 0 && value != 1) return fail(GNNK_EINVAL, "no_fast is 0 or 1");
        options().no_fast = value;
    } else {
        return fail(GNNK_EINVAL, "unknown option '%s'", key);
    }
    return GNNK_OK;
}

const char* gnnk_last_error(void) { return g_err; }

}  // extern "C"
