// Fused graph attention: the u_add_v -> leaky ReLU -> edge softmax ->
// u_mul_e/sum chain (the multi-head attention layer of Appendix E, written
// there as a g-SDDMM followed by a g-SpMM) in one pass over each
// destination's in-edges:
//
//   s_e = leaky(el[u, h] + er[v, h])            (two single fp32 operations)
//   out[v, h, :] = sum_e exp(s_e - m) feat[u, h, :] / sum_e exp(s_e - m)
//
// with m the running maximum of s over the edges seen so far: when m grows,
// the fp64 sums so far are rescaled by exp(m_old - m_new) (online softmax),
// so no edge tensor is read or written between the steps.  Optionally the
// attention a_e = exp(s_e - m) / sum is written (the softmax output the
// backward pass needs), by a second walk over the row once m and the sum
// are final.  Rows use the degree-sorted roles of the row engine; hub rows
// leave per-segment (m, sum, acc) partials merged in segment order.
#include "walk.h"

namespace gnnk {

struct GatArgs {
    const void* er;       // (N_dst, H) per-head destination score
    int64_t er_stride;
    void* attn;           // (E, H) attention out, nullable
    int64_t attn_stride;
    float slope;
    int32_t pad;
    void* row_ml;         // hub rows: final (m, sum) per column, 2 x D doubles per hub row
    float* stats;         // (N_dst, H, 2) fp32: max score and 1 / sum per head, nullable
    int64_t stats_stride;
};

// the per-head statistics of a destination row: the max score and the
// reciprocal of the sum of exp(score - max), rounded to fp32 as the
// attention written by this kernel uses it
__device__ __forceinline__ void gat_write_stats(const GatArgs& G, int64_t row, int h, float m, double l) {
    if (!G.stats) return;
    float* p = G.stats + row * G.stats_stride + 2 * h;
    p[0] = l > 0.0 ? m : 0.0f;
    p[1] = l > 0.0 ? (float)(1.0 / l) : 0.0f;
}

// online state of one lane for its VEC columns
template <int VEC>
struct Online {
    float m;
    double l;
    double acc[VEC];
    __device__ __forceinline__ void init() {
        m = -INFINITY;
        l = 0.0;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = 0.0;
    }
    // add U edges with scores s and source rows x: the state is rescaled once
    // to the new maximum, and only where it grew for some lane of the
    // wavefront (seldom after a row's first batches), then the terms are
    // added; edge by edge every term paid the comparison, the selects and
    // the rescaling (114.6M edges, H = 8, F = 16: 3.95 -> 3.48 ms).  A score
    // of -inf weighs nothing; while the maximum is still -inf the terms are
    // taken against 0 (-inf - (-inf) would be NaN).  One of +inf leaves NaN
    // sums.
    template <int U, class X>
    __device__ __forceinline__ void add(const float* s, const X& x) {
        float mb = s[0];
#pragma unroll
        for (int u = 1; u < U; ++u) mb = fmaxf(mb, s[u]);
        const float mn = fmaxf(m, mb);
        const float at = mn == -INFINITY ? 0.0f : mn;
        if (__ballot(mn > m) != 0ull) {
            const double f = (double)exp_le0(m - at);
            l *= f;
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] *= f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double p = (double)exp_le0(s[u] - at);
            l += p;
#pragma unroll
            for (int i = 0; i < VEC; ++i) acc[i] = fma(p, (double)x(u)[i], acc[i]);
        }
        m = mn;
    }
    // add one edge, +inf included: it takes the whole weight, and a second one
    // or a NaN makes the state NaN
    __device__ __forceinline__ void add_any(float s, const float* x) {
        const float mn = fmaxf(m, s);
        const double f = mn == -INFINITY ? 0.0 : (double)exp_le0((m < s ? m : s) - mn);
        const bool up = s > m;
        const double c_old = up ? f : 1.0;
        const double c_new = up ? 1.0 : f;
        l = l * c_old + c_new;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = acc[i] * c_old + c_new * (double)x[i];
        m = mn;
    }
    // no sum is infinite or NaN
    __device__ __forceinline__ bool finite() const {
        double t = acc[0];
#pragma unroll
        for (int i = 1; i < VEC; ++i) t += acc[i];
        return fabs(t) < INFINITY;
    }
    // merge another state (in segment or lane-group order)
    __device__ __forceinline__ void merge(float om, double ol, const double* oacc) {
        const float mn = fmaxf(m, om);
        // (the larger one by a comparison: +inf - (+inf) would be NaN)
        const double f1 = m == -INFINITY ? 0.0 : (m > om ? 1.0 : (double)exp_le0(m - mn));
        const double f2 = om == -INFINITY ? 0.0 : (om > m ? 1.0 : (double)exp_le0(om - mn));
        l = l * f1 + ol * f2;
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = acc[i] * f1 + oacc[i] * f2;
        m = mn;
    }
};

template <typename T>
__device__ __forceinline__ float gat_score(float el, float er, float slope) {
    const float s = el + er;
    return s > 0.0f ? s : slope * s;
}

// consumer of a row's edges: a full batch at once, others one by one.
// BATCHED = false: the runtime layouts of one or two columns a lane, which have
// no full batches.  Edge by edge the state of some lane of a wavefront nearly
// always grows, and add() then takes two exponentials an edge where add_any()
// takes one: bf16, 8 heads of 5 columns, 1M and 8.4M edges, 73 -> 67 and
// 528 -> 501 us.  Those of four or more columns, a whole row in a lane each,
// keep add(): 8.4M edges, fp32, 4 columns, 100 us with it, 107 without.
template <int VEC, class S>
constexpr bool gat_batched = S::FAST || VEC >= 4;

template <typename T, int VEC, bool BATCHED>
struct GatSink {
    Online<VEC>& st;
    float er_h, slope;
    static constexpr bool kBatch = true;
    __device__ __forceinline__ void batch(const Raw<VEC>* rw, const int32_t*) {
        float s[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) s[u] = gat_score<T>(rw[u].b[0], er_h, slope);
        st.template add<UNR>(s, [&](int u) { return rw[u].a; });
    }
    __device__ __forceinline__ void operator()(const Raw<VEC>& rw, int32_t, int32_t, bool ok) {
        if constexpr (!BATCHED) {
            if (ok) st.add_any(gat_score<T>(rw.b[0], er_h, slope), rw.a);
        } else {
            // a slot outside the row holds another edge's values and scores
            // -inf: it weighs nothing (0 times an infinite value: see gat_again)
            const float s = ok ? gat_score<T>(rw.b[0], er_h, slope) : -INFINITY;
            st.template add<1>(&s, [&](int) { return rw.a; });
        }
    }
};

template <typename T, int VEC>
__device__ __forceinline__ float load_er(const GatArgs& G, int32_t v, int h) {
    return IO<T, VEC>::load1(reinterpret_cast<const T*>(G.er) + (uint64_t)(uint32_t)v * (uint32_t)G.er_stride + h);
}

// A lane whose sums are infinite or NaN adds its edges b + start, b + start +
// stride, ... < e once more, one by one: there the slots outside the row are
// left out (0 times an infinite feature is NaN) and a score of +inf has its
// weight.  Tests of both among the additions took the forward on 20,000 rows
// of 5 edges from 13.8 to 14.7 us; this look at the sums takes it to 14.0.
template <typename T, int VEC>
__device__ __forceinline__ void gat_again(const EngineArgs& A, int32_t b, int32_t e, int start, int stride, int col0,
                                     int h, float er_h, float slope, Online<VEC>& st) {
    if (st.finite()) return;
    st.init();
    for (int32_t p = b + start; p < e; p += stride) {
        const uint64_t u = (uint32_t)A.csr.idx[p];
        float x[VEC];
        IO<T, VEC>::load(reinterpret_cast<const T*>(A.a.data) + u * (uint32_t)A.a.stride + col0, x);
        const float el = IO<T, 1>::load1(reinterpret_cast<const T*>(A.b.data) + u * (uint32_t)A.b.stride + h);
        st.add_any(gat_score<T>(el, er_h, slope), x);
    }
}

// write a_e for the edges b + start, b + start + stride, ... < e of a row,
// given the final (m, sum) of the lane's head (one writer lane per head)
template <typename T, int VEC>
__device__ __forceinline__ void gat_write_attn(const EngineArgs& A, const GatArgs& G, int64_t b64, int64_t e64,
                                               int64_t start, int stride, int lig, int h, bool active, float er_h,
                                               float m, double l) {
    const int per_head = A.geo.FV;  // lanes of one head
    const bool writer = active & (lig % per_head == 0);
    const int32_t b = (int32_t)b64, e = (int32_t)e64;
    const T* el = reinterpret_cast<const T*>(A.b.data);
    T* out = reinterpret_cast<T*>(G.attn);
    const float inv = (float)(1.0 / l);
    for (int32_t p0 = b + (int32_t)start; p0 < e; p0 += stride * UNR) {
        int32_t nb[UNR], ed[UNR], ps[UNR];
        bool ok[UNR];
        batch_ids(A.csr, b, e, p0, stride, ok, nb, ed, ps);
        float x[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u)
            x[u] = IO<T, 1>::load1(el + (uint64_t)(uint32_t)nb[u] * (uint32_t)A.b.stride + h);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const float s = gat_score<T>(x[u], er_h, G.slope);
            if (ok[u] & writer)
                IO<T, 1>::store1(out + (uint64_t)(uint32_t)ed[u] * (uint32_t)G.attn_stride + h,
                                 exp_le0(s - m) * inv);
        }
    }
}

template <typename T, int VEC, class S, bool ATTN>
__global__ __launch_bounds__(256) void gat_kernel(EngineArgs A, GatArgs G) {
    const int w = wave_id();
    if (w >= A.sch.w_total) return;
    const GeomDev& geo = A.geo;
    const Lanes ln = lanes_of<S::GC>(geo);
    const int Gn = S::GC > 0 ? S::GC : geo.G;
    const int L = WAVE / Gn;
    const int64_t D = (int64_t)geo.D;

    if (w < A.sch.w_big_end) {
        int64_t r, b, e;
        int slot = -1;
        if (w < A.sch.n_seg) {
            const int4 s = A.csr.segw[w];
            r = s.x; b = s.y; e = s.z; slot = s.w;
        } else {
            const int4 t = A.csr.rowt[A.sch.n_hub + (w - A.sch.n_seg)];
            r = t.x; b = t.y; e = t.z;
        }
        r = uniform64(r);
        b = uniform64(b);
        e = uniform64(e);
        for (int ch = 0; ch < geo.nchunk; ++ch) {
            const int j = ch * L + ln.lig;
            const bool active = j < geo.NV;
            const Cols cc = cols_of<VEC, S::OV>(geo, active, j);
            const int col0 = cc.col0, h = cc.h;
            const float er_h = load_er<T, VEC>(G, (int32_t)r, h);
            Online<VEC> st;
            st.init();
            Pre<VEC> pre;
            GatSink<T, VEC, gat_batched<VEC, S>> sink{st, er_h, G.slope};
            walk_row<T, VEC, 1, EXT_NONE, S>(A, (int32_t)r, b, e, ln.g, Gn, col0, h, pre, sink);
            if constexpr (gat_batched<VEC, S>)
                gat_again<T, VEC>(A, (int32_t)b, (int32_t)e, ln.g, Gn, col0, h, er_h, G.slope, st);
            for (int s = L; s < WAVE; s <<= 1) {
                double oacc[VEC];
#pragma unroll
                for (int i = 0; i < VEC; ++i) oacc[i] = shfl_xor_d(st.acc[i], s);
                st.merge(__shfl_xor(st.m, s, WAVE), shfl_xor_d(st.l, s), oacc);
            }
            if (slot >= 0) {
                if (ln.g == 0 && active) {
                    // the weighted row, then (max, sum) of each head
                    double* P = reinterpret_cast<double*>(A.partial) + (int64_t)slot * A.partial_stride;
#pragma unroll
                    for (int i = 0; i < VEC; ++i) P[col0 + i] = st.acc[i];
                    if (col0 % geo.F == 0) {
                        P[D + 2 * h] = (double)st.m;
                        P[D + 2 * h + 1] = st.l;
                    }
                }
            } else {
                if (ln.g == 0 && active) {
                    float v[VEC];
#pragma unroll
                    for (int i = 0; i < VEC; ++i) v[i] = (float)(st.acc[i] / st.l);
                    IO<T, VEC>::store(reinterpret_cast<T*>(A.out.data) + r * A.out.stride + col0, v);
                    if (col0 % geo.F == 0) gat_write_stats(G, r, h, st.m, st.l);
                }
                if constexpr (ATTN) gat_write_attn<T, VEC>(A, G, b, e, ln.g, Gn, ln.lig, h, active, er_h, st.m, st.l);
            }
        }
    } else if (w < A.sch.w_small_end) {
        const int64_t k = A.sch.n_big + (int64_t)(w - A.sch.w_big_end) * Gn + ln.g;
        int64_t r = -1, b = 0, e = 0;
        if (k < A.sch.n_nz) {
            const int4 t = A.csr.rowt[k];
            r = t.x; b = t.y; e = t.z;
        }
        const int32_t self = r >= 0 ? (int32_t)r : 0;
        for (int ch = 0; ch < geo.nchunk; ++ch) {
            const int j = ch * L + ln.lig;
            const bool active = j < geo.NV;
            const Cols cc = cols_of<VEC, S::OV>(geo, active, j);
            const int col0 = cc.col0, h = cc.h;
            const float er_h = r >= 0 ? load_er<T, VEC>(G, self, h) : 0.0f;
            Online<VEC> st;
            st.init();
            Pre<VEC> pre;
            GatSink<T, VEC, gat_batched<VEC, S>> sink{st, er_h, G.slope};
            walk_lane<T, VEC, 1, EXT_NONE, S>(A, self, b, e, col0, h, pre, sink);
            if constexpr (gat_batched<VEC, S>)
                gat_again<T, VEC>(A, (int32_t)b, (int32_t)e, 0, 1, col0, h, er_h, G.slope, st);
            if (r >= 0 && active) {
                float v[VEC];
#pragma unroll
                for (int i = 0; i < VEC; ++i) v[i] = (float)(st.acc[i] / st.l);
                IO<T, VEC>::store(reinterpret_cast<T*>(A.out.data) + r * A.out.stride + col0, v);
                if (col0 % geo.F == 0) gat_write_stats(G, r, h, st.m, st.l);
            }
            if constexpr (ATTN)
                if (r >= 0) gat_write_attn<T, VEC>(A, G, b, e, 0, 1, ln.lig, h, active, er_h, st.m, st.l);
        }
    } else {
        // empty rows: no edge, output 0
        const int64_t k0 = A.sch.n_nz +
                           ((int64_t)(w - A.sch.w_small_end) * Gn + ln.g) * A.sch.fill_rows_per_group;
        for (int q = 0; q < A.sch.fill_rows_per_group; ++q) {
            const int64_t k = k0 + q;
            const int64_t r = k < A.sch.n_rows ? A.csr.perm[k] : -1;
            for (int ch = 0; ch < geo.nchunk; ++ch) {
                const int j = ch * L + ln.lig;
                if (j < geo.NV && r >= 0) {
                    const Cols cc = cols_of<VEC, S::OV>(geo, true, j);
                    float v[VEC];
#pragma unroll
                    for (int i = 0; i < VEC; ++i) v[i] = 0.0f;
                    IO<T, VEC>::store(reinterpret_cast<T*>(A.out.data) + r * A.out.stride + cc.col0, v);
                    if (j % geo.FV == 0) gat_write_stats(G, r, cc.h, 0.0f, 0.0);
                }
            }
        }
    }
}

// hub rows: merge the segment partials in order and write the row; keep the
// row's final (m, sum) for the attention writes
constexpr int GC_UNR = 4;

template <typename T, int VEC, bool OV>
__global__ __launch_bounds__(256) void gat_combine_kernel(EngineArgs A, GatArgs G) {
    const int w = wave_id();
    const GeomDev& geo = A.geo;
    const Lanes ln = lanes_of(geo);
    if ((int64_t)w * geo.G >= A.sch.n_hub) return;
    const int64_t k = (int64_t)w * geo.G + ln.g;
    const bool row_ok = k < A.sch.n_hub;
    const int64_t r = row_ok ? A.csr.perm[k] : -1;
    const int s0 = row_ok ? A.csr.hub_off[k] : 0;
    const int s1 = row_ok ? A.csr.hub_off[k + 1] : 0;
    const int64_t D = (int64_t)geo.D;
    const double* P = reinterpret_cast<const double*>(A.partial);
    for (int ch = 0; ch < geo.nchunk; ++ch) {
        const int j = ch * geo.L + ln.lig;
        const bool active = j < geo.NV && row_ok;
        const Cols cc = cols_of<VEC, OV>(geo, active, j);
        const int col0 = cc.col0, h = cc.h;
        if (!active) continue;
        // the row's maximum first, then its segments' sums against it, in
        // segment order; GC_UNR segments' loads in flight at once
        Online<VEC> st;
        st.init();
        const double* Q = P + (int64_t)s0 * A.partial_stride;
        const int n = s1 - s0;
        for (int s = 0; s < n; s += GC_UNR) {
#pragma unroll
            for (int u = 0; u < GC_UNR; ++u)
                st.m = fmaxf(st.m, (float)Q[(int64_t)(s + u < n ? s + u : s) * A.partial_stride + D + 2 * h]);
        }
        const float at = st.m == -INFINITY ? 0.0f : st.m;
        for (int s = 0; s < n; s += GC_UNR) {
            double pm[GC_UNR], pl[GC_UNR], pa[GC_UNR][VEC];
#pragma unroll
            for (int u = 0; u < GC_UNR; ++u) {
                const double* q = Q + (int64_t)(s + u < n ? s + u : s) * A.partial_stride;
                pm[u] = q[D + 2 * h];
                pl[u] = q[D + 2 * h + 1];
#pragma unroll
                for (int i = 0; i < VEC; ++i) pa[u][i] = q[col0 + i];
            }
#pragma unroll
            for (int u = 0; u < GC_UNR; ++u) {
                const double f = s + u < n ? (double)exp_le0((float)pm[u] - at) : 0.0;
                st.l = fma(f, pl[u], st.l);
#pragma unroll
                for (int i = 0; i < VEC; ++i) st.acc[i] = fma(f, pa[u][i], st.acc[i]);
            }
        }
        if (!st.finite()) {
            // one by one, without the slots past the last segment
            st.init();
            for (int s = 0; s < n; ++s) {
                const double* q = Q + (int64_t)s * A.partial_stride;
                double pa[VEC];
#pragma unroll
                for (int i = 0; i < VEC; ++i) pa[i] = q[col0 + i];
                st.merge((float)q[D + 2 * h], q[D + 2 * h + 1], pa);
            }
        }
        float v[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = (float)(st.acc[i] / st.l);
        IO<T, VEC>::store(reinterpret_cast<T*>(A.out.data) + r * A.out.stride + col0, v);
        if (col0 % geo.F == 0) gat_write_stats(G, r, h, st.m, st.l);
        if (G.attn) {
            double* ML = reinterpret_cast<double*>(G.row_ml) + k * 2 * D;
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                ML[col0 + i] = (double)st.m;
                ML[D + col0 + i] = st.l;
            }
        }
    }
}

// hub rows with attention out: each segment writes its edges' a_e
template <typename T, int VEC, bool OV>
__global__ __launch_bounds__(256) void gat_attn_segments_kernel(EngineArgs A, GatArgs G) {
    const int w = wave_id();
    if (w >= A.sch.n_seg) return;
    const GeomDev& geo = A.geo;
    const Lanes ln = lanes_of(geo);
    const int64_t D = (int64_t)geo.D;
    const int4 sg = A.csr.seg[A.csr.seg_order[w]];
    const double* ML = reinterpret_cast<const double*>(G.row_ml) + (int64_t)sg.w * 2 * D;
    for (int ch = 0; ch < geo.nchunk; ++ch) {
        const int j = ch * geo.L + ln.lig;
        const bool active = j < geo.NV;
        const Cols cc = cols_of<VEC, OV>(geo, active, j);
        const int col0 = cc.col0, h = cc.h;
        const float er_h = load_er<T, VEC>(G, sg.x, h);
        gat_write_attn<T, VEC>(A, G, sg.y, sg.z, ln.g, geo.G, ln.lig, h, active, er_h, (float)ML[col0],
                               ML[D + col0]);
    }
}

// ---------------------------------------------------------------------------
// backward of the fused attention
//
// With s_e = leaky(el[u] + er[v]) per head, a_e = softmax over the in-edges
// of v of s_e, and out[v] = sum over in-edges of a_e feat[u] (per head):
//   da_e      = dZ[v] . feat[u]                        (per head)
//   ds_e      = a_e (da_e - S_v) lk_e                  lk_e = leaky'(el[u] + er[v])
//   S_v       = sum_in a_e da_e
//   d_er[v]   = sum_in ds_e = P_v - S_v Q_v           P_v = sum_in a_e da_e lk_e, Q_v = sum_in a_e lk_e
//   d_el[u]   = sum_out ds_e
//   d_feat[u] = sum_out a_e dZ[v]
// (the chain rule through the four steps, Theorem 1's gradients of g-SpMM
// and g-SDDMM).  a_e is recomputed from the forward's per-row max and
// 1 / sum, so no tensor of E x H elements is read or written.  Pass A walks
// the in-CSR: S, P, Q per destination and head in fp64, d_er, and a record
// {er, max, 1 / sum, S} per (destination, head) for pass B.  Pass B walks the
// reverse graph's CSR and gathers dZ[v] and that record per edge.
//
// Every sum that da enters is linear in it, and da is a sum over the lanes of
// a head, so each lane sums with its own share of da and the lanes of a head
// are added once per row: no lane moves per edge (they were about a quarter
// of the passes' vector instructions, and for heads of other than 2, 4, 8 or
// 16 lanes most of them).

// sum of a per-lane value over the `red` lanes of one head (aligned runs in
// the lane group); the total is exact in the head's first lane
__device__ __forceinline__ double head_sum(double v, int lig, int red) {
    return (red & (red - 1)) == 0 ? run_sum(v, red) : seg_sum(v, lig, red);
}

// a lane's share of a head's dot product without the first `skip` columns
template <int VEC>
__device__ __forceinline__ double last_share(const float (&x)[VEC], const double (&y)[VEC], int skip) {
    double dp = 0.0;
#pragma unroll
    for (int i = 0; i < VEC; ++i) dp += i < skip ? 0.0 : (double)x[i] * y[i];
    return dp;
}

// the attention of one edge, recomputed as the forward computes it
__device__ __forceinline__ float gat_attention(float el, float er, float slope, float m, float il, bool& pos) {
    const float s = el + er;
    pos = s > 0.0f;
    return exp_le0((pos ? s : slope * s) - m) * il;
}

template <typename T>
__device__ __forceinline__ void gat_finish_dst(const GatBwdArgs& B, int64_t v, int h, float er_h, float m, float il,
                                               double S, double P, double Q) {
    if (B.chunk) {
        // S and P of this column chunk: stored by the first, added by the
        // others in chunk order; Q does not depend on the columns
        double* ac = B.acc_dst + (v * B.H + h) * 2;
        if (B.chunk > 1) {
            S += ac[0];
            P += ac[1];
        }
        if (B.chunk < 3) {
            ac[0] = S;
            ac[1] = P;
            return;
        }
    }
    if (B.d_er) IO<T, 1>::store1(reinterpret_cast<T*>(B.d_er) + v * B.d_er_stride + h, (float)(P - S * Q));
    B.rec[v * B.H + h] = make_float4(er_h, m, il, (float)S);
}

// pass A: one destination row (a hub segment, a row by the wavefront, or a
// row by this lane group)
template <typename T, int VEC, class S, bool WAVE_ROW>
__device__ __forceinline__ void gat_bwd_dst_row(const EngineArgs& A, const GatBwdArgs& B, const Lanes& ln, int Gn,
                                                int64_t r, int64_t b, int64_t e, int slot) {
    const GeomDev& geo = A.geo;
    const int L = WAVE / Gn;
    const int red = geo.FV;  // lanes of a head
    const bool active = ln.lig < geo.NV;
    const Cols cc = cols_of<VEC, S::OV>(geo, active, ln.lig);
    const int col0 = cc.col0, h = cc.h;
    const bool head_lane = active && (col0 % geo.F) == 0;
    const int32_t self = r >= 0 ? (int32_t)r : 0;
    float dz[VEC];
    IO<T, VEC>::load(reinterpret_cast<const T*>(B.dz) + (int64_t)self * B.dz_stride + col0, dz);
    double dzd[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) dzd[i] = dz[i];
    const float er_h = IO<T, 1>::load1(reinterpret_cast<const T*>(B.er) + (int64_t)self * B.er_stride + h);
    const float m = B.stats[(int64_t)self * B.stats_stride + 2 * h];
    const float il = B.stats[(int64_t)self * B.stats_stride + 2 * h + 1];
    double sS = 0.0, sP = 0.0, sQ = 0.0;
    Pre<VEC> pre;
    auto sink = [&](const Raw<VEC>& rw, int32_t, int32_t, bool ok) {
        // a slot outside the row holds another edge's values: a weight of 0
        // times an infinite one would be NaN.  (A branch: with selects the
        // backward of 20,000 rows of 5 edges took 31.4 us, now 30.7.)
        if (!ok) return;
        bool pos;
        const double a = (double)gat_attention(rw.b[0], er_h, B.slope, m, il, pos);
        const double al = pos ? a : a * (double)B.slope;
        double dp = 0.0;
#pragma unroll
        for (int i = 0; i < VEC; ++i) dp = fma((double)rw.a[i], dzd[i], dp);
        if constexpr (S::OV) dp = last_share(rw.a, dzd, cc.skip);
        sS = fma(a, dp, sS);   // this lane's share of S and P
        sP = fma(al, dp, sP);
        sQ += al;              // the same in every lane of a head
    };
    if constexpr (WAVE_ROW) {
        walk_row<T, VEC, 1, EXT_NONE, S>(A, self, b, e, ln.g, Gn, col0, h, pre, sink);
        for (int s = L; s < WAVE; s <<= 1) {
            sS += shfl_xor_d(sS, s);
            sP += shfl_xor_d(sP, s);
            sQ += shfl_xor_d(sQ, s);
        }
        sS = head_sum(sS, ln.lig, red);
        sP = head_sum(sP, ln.lig, red);
        if (ln.g != 0 || !head_lane) return;
        if (slot >= 0) {
            double* p = B.part + (int64_t)slot * 3 * B.H;
            p[h] = sS;
            p[B.H + h] = sP;
            p[2 * B.H + h] = sQ;
        } else {
            gat_finish_dst<T>(B, r, h, er_h, m, il, sS, sP, sQ);
        }
    } else {
        walk_lane<T, VEC, 1, EXT_NONE, S>(A, self, b, e, col0, h, pre, sink);
        sS = head_sum(sS, ln.lig, red);
        sP = head_sum(sP, ln.lig, red);
        if (r >= 0 && head_lane) gat_finish_dst<T>(B, r, h, er_h, m, il, sS, sP, sQ);
    }
}

template <typename T, int VEC, class S>
__global__ __launch_bounds__(256) void gat_bwd_dst_kernel(EngineArgs A, GatBwdArgs B) {
    const int w = wave_id();
    if (w >= A.sch.w_total) return;
    const GeomDev& geo = A.geo;
    const Lanes ln = lanes_of<S::GC>(geo);
    const int Gn = S::GC > 0 ? S::GC : geo.G;
    if (w < A.sch.w_big_end) {
        int64_t r, b, e;
        int slot = -1;
        if (w < A.sch.n_seg) {
            const int4 sg = A.csr.segw[w];
            r = sg.x; b = sg.y; e = sg.z; slot = sg.w;
        } else {
            const int4 t = A.csr.rowt[A.sch.n_hub + (w - A.sch.n_seg)];
            r = t.x; b = t.y; e = t.z;
        }
        gat_bwd_dst_row<T, VEC, S, true>(A, B, ln, Gn, uniform64(r), uniform64(b), uniform64(e), slot);
    } else if (w < A.sch.w_small_end) {
        const int64_t k = A.sch.n_big + (int64_t)(w - A.sch.w_big_end) * Gn + ln.g;
        int64_t r = -1, b = 0, e = 0;
        if (k < A.sch.n_nz) {
            const int4 t = A.csr.rowt[k];
            r = t.x; b = t.y; e = t.z;
        }
        gat_bwd_dst_row<T, VEC, S, false>(A, B, ln, Gn, r, b, e, -1);
    } else if (B.d_er) {
        // rows without in-edges: d_er = 0 (no edge reads their record)
        const int64_t k0 = A.sch.n_nz + ((int64_t)(w - A.sch.w_small_end) * Gn + ln.g) * A.sch.fill_rows_per_group;
        if (ln.lig < geo.NV && ln.lig % geo.FV == 0) {
            for (int q = 0; q < A.sch.fill_rows_per_group; ++q) {
                const int64_t k = k0 + q;
                if (k < A.sch.n_rows)
                    IO<T, 1>::store1(reinterpret_cast<T*>(B.d_er) + (int64_t)A.csr.perm[k] * B.d_er_stride +
                                         ln.lig / geo.FV, 0.0f);
            }
        }
    }
}

// pass A, hub rows: one thread per (hub row, head), segments in order
template <typename T>
__global__ __launch_bounds__(256) void gat_bwd_dst_combine_kernel(EngineArgs A, GatBwdArgs B) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t k = t / B.H;
    const int h = (int)(t % B.H);
    if (k >= A.sch.n_hub) return;
    const int64_t r = A.csr.perm[k];
    const int s0 = A.csr.hub_off[k], s1 = A.csr.hub_off[k + 1];
    double sS = 0.0, sP = 0.0, sQ = 0.0;
    for (int s = s0; s < s1; s += GC_UNR) {
        double v[GC_UNR][3];
#pragma unroll
        for (int u = 0; u < GC_UNR; ++u) {
            const double* p = B.part + (int64_t)(s + u < s1 ? s + u : s) * 3 * B.H + h;
#pragma unroll
            for (int c = 0; c < 3; ++c) v[u][c] = p[c * B.H];
        }
#pragma unroll
        for (int u = 0; u < GC_UNR; ++u) {
            const bool ok = s + u < s1;
            sS += ok ? v[u][0] : 0.0;
            sP += ok ? v[u][1] : 0.0;
            sQ += ok ? v[u][2] : 0.0;
        }
    }
    const float er_h = IO<T, 1>::load1(reinterpret_cast<const T*>(B.er) + r * B.er_stride + h);
    const float m = B.stats[r * B.stats_stride + 2 * h];
    const float il = B.stats[r * B.stats_stride + 2 * h + 1];
    gat_finish_dst<T>(B, r, h, er_h, m, il, sS, sP, sQ);
}

template <typename T, int VEC>
__device__ __forceinline__ void gat_write_src(const GatBwdArgs& B, int64_t u, int col0, int h, bool active,
                                              bool head_lane, const double* df, double dl) {
    if (B.d_feat && active) {
        float v[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = (float)df[i];
        IO<T, VEC>::store(reinterpret_cast<T*>(B.d_feat) + u * B.d_feat_stride + col0, v);
    }
    if (B.d_el && head_lane) {
        if (B.chunk) {
            // this column chunk's share of d_el, added in chunk order
            double* ac = B.acc_src + u * B.H + h;
            if (B.chunk > 1) dl += *ac;
            if (B.chunk < 3) {
                *ac = dl;
                return;
            }
        }
        IO<T, 1>::store1(reinterpret_cast<T*>(B.d_el) + u * B.d_el_stride + h, (float)dl);
    }
}

// pass B: one source row (a hub segment, a row by the wavefront, or a row by
// this lane group)
template <typename T, int VEC, class S, bool WAVE_ROW>
__device__ __forceinline__ void gat_bwd_src_row(const EngineArgs& A, const GatBwdArgs& B, const Lanes& ln, int Gn,
                                                int64_t r, int64_t b, int64_t e, int slot) {
    const GeomDev& geo = A.geo;
    const int L = WAVE / Gn;
    const int red = geo.FV;  // lanes of a head
    const bool active = ln.lig < geo.NV;
    const Cols cc = cols_of<VEC, S::OV>(geo, active, ln.lig);
    const int col0 = cc.col0, h = cc.h;
    const bool head_lane = active && (col0 % geo.F) == 0;
    const int64_t self = r >= 0 ? r : 0;
    float x[VEC];
    IO<T, VEC>::load(reinterpret_cast<const T*>(B.feat) + self * B.feat_stride + col0, x);
    double xd[VEC], df[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        xd[i] = x[i];
        df[i] = 0.0;
    }
    const float el_h = IO<T, 1>::load1(reinterpret_cast<const T*>(B.el) + self * B.el_stride + h);
    double dl = 0.0, ds = 0.0;
    // d_el = sum of a (da - S) lk: dl this lane's share of the da part, ds the
    // S part, the same in every lane of a head; a head in column chunks takes
    // the S part with its first chunk only (da is summed chunk by chunk)
    const bool with_s = B.chunk <= 1;
    Pre<VEC> pre;
    auto sink = [&](const Raw<VEC>& rw, int32_t, int32_t, bool ok) {
        // (as in pass A; 20M edges, 4 x 16 bf16, both passes: with selects
        // 647 us, now 628)
        if (!ok) return;
        bool pos;
        const double a = (double)gat_attention(el_h, rw.rec.x, B.slope, rw.rec.y, rw.rec.z, pos);
        const double al = pos ? a : a * (double)B.slope;
        double dp = 0.0;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const double z = (double)rw.a[i];
            dp = fma(z, xd[i], dp);
            df[i] = fma(a, z, df[i]);
        }
        if constexpr (S::OV) dp = last_share(rw.a, xd, cc.skip);
        dl = fma(al, dp, dl);
        ds = fma(al, (double)rw.rec.w, ds);
    };
    auto d_el = [&]() { return head_sum(dl, ln.lig, red) - (with_s ? ds : 0.0); };
    if constexpr (WAVE_ROW) {
        walk_row<T, VEC, 0, EXT_REC, S>(A, (int32_t)self, b, e, ln.g, Gn, col0, h, pre, sink);
        for (int s = L; s < WAVE; s <<= 1) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) df[i] += shfl_xor_d(df[i], s);
            dl += shfl_xor_d(dl, s);
            ds += shfl_xor_d(ds, s);
        }
        dl = d_el();
        if (ln.g != 0) return;
        if (slot >= 0) {
            const int64_t D = (int64_t)geo.D;
            double* p = B.part + (int64_t)slot * (D + B.H);
            if (active) {
#pragma unroll
                for (int i = 0; i < VEC; ++i) p[col0 + i] = df[i];
            }
            if (head_lane) p[D + h] = dl;
        } else {
            gat_write_src<T, VEC>(B, r, col0, h, active, head_lane, df, dl);
        }
    } else {
        walk_lane<T, VEC, 0, EXT_REC, S>(A, (int32_t)self, b, e, col0, h, pre, sink);
        dl = d_el();
        if (r >= 0) gat_write_src<T, VEC>(B, r, col0, h, active, head_lane, df, dl);
    }
}

// The ids of a batch come as in the other walks (scalar loads one batch ahead
// for 1-4 lane groups) and the node rows and records through 32-bit offsets:
// with ids loaded per lane and 64-bit addresses this pass took 5.88 ms on the
// 114.6M-edge graph at H = 8, F = 16 where pass A, which gathers as much, took
// 3.83; now 4.22 and 3.52 (with the lane sums taken once per row).
template <typename T, int VEC, class S>
__global__ __launch_bounds__(256) void gat_bwd_src_kernel(EngineArgs A, GatBwdArgs B) {
    const int w = wave_id();
    if (w >= A.sch.w_total) return;
    const GeomDev& geo = A.geo;
    const Lanes ln = lanes_of<S::GC>(geo);
    const int Gn = S::GC > 0 ? S::GC : geo.G;
    if (w < A.sch.w_big_end) {
        int64_t r, b, e;
        int slot = -1;
        if (w < A.sch.n_seg) {
            const int4 sg = A.csr.segw[w];
            r = sg.x; b = sg.y; e = sg.z; slot = sg.w;
        } else {
            const int4 t = A.csr.rowt[A.sch.n_hub + (w - A.sch.n_seg)];
            r = t.x; b = t.y; e = t.z;
        }
        gat_bwd_src_row<T, VEC, S, true>(A, B, ln, Gn, uniform64(r), uniform64(b), uniform64(e), slot);
    } else if (w < A.sch.w_small_end) {
        const int64_t k = A.sch.n_big + (int64_t)(w - A.sch.w_big_end) * Gn + ln.g;
        int64_t r = -1, b = 0, e = 0;
        if (k < A.sch.n_nz) {
            const int4 t = A.csr.rowt[k];
            r = t.x; b = t.y; e = t.z;
        }
        gat_bwd_src_row<T, VEC, S, false>(A, B, ln, Gn, r, b, e, -1);
    } else {
        // sources without out-edges: zero gradients
        const int64_t k0 = A.sch.n_nz + ((int64_t)(w - A.sch.w_small_end) * Gn + ln.g) * A.sch.fill_rows_per_group;
        const bool active = ln.lig < geo.NV;
        const Cols cc = cols_of<VEC, S::OV>(geo, active, ln.lig);
        const double zero[VEC] = {};
        for (int q = 0; q < A.sch.fill_rows_per_group; ++q) {
            const int64_t k = k0 + q;
            if (k < A.sch.n_rows)
                gat_write_src<T, VEC>(B, A.csr.perm[k], cc.col0, cc.h, active, active && cc.col0 % geo.F == 0,
                                      zero, 0.0);
        }
    }
}

// pass B, hub rows: partials of the row's segments summed in order
template <typename T, int VEC, bool OV>
__global__ __launch_bounds__(256) void gat_bwd_src_combine_kernel(EngineArgs A, GatBwdArgs B) {
    const int w = wave_id();
    const GeomDev& geo = A.geo;
    const Lanes ln = lanes_of(geo);
    if ((int64_t)w * geo.G >= A.sch.n_hub) return;
    const int64_t k = (int64_t)w * geo.G + ln.g;
    if (k >= A.sch.n_hub) return;
    const int64_t r = A.csr.perm[k];
    const int s0 = A.csr.hub_off[k], s1 = A.csr.hub_off[k + 1];
    const int64_t D = (int64_t)geo.D;
    const bool active = ln.lig < geo.NV;
    const Cols cc = cols_of<VEC, OV>(geo, active, ln.lig);
    const int col0 = cc.col0, h = cc.h;
    const bool head_lane = active && (col0 % geo.F) == 0;
    double df[VEC], dl = 0.0;
#pragma unroll
    for (int i = 0; i < VEC; ++i) df[i] = 0.0;
    for (int s = s0; s < s1; s += GC_UNR) {
        double v[GC_UNR][VEC], vl[GC_UNR];
#pragma unroll
        for (int u = 0; u < GC_UNR; ++u) {
            const double* p = B.part + (int64_t)(s + u < s1 ? s + u : s) * (D + B.H);
#pragma unroll
            for (int i = 0; i < VEC; ++i) v[u][i] = p[col0 + i];
            vl[u] = p[D + h];
        }
#pragma unroll
        for (int u = 0; u < GC_UNR; ++u) {
            const bool ok = s + u < s1;
#pragma unroll
            for (int i = 0; i < VEC; ++i) df[i] += ok ? v[u][i] : 0.0;
            dl += ok ? vl[u] : 0.0;
        }
    }
    gat_write_src<T, VEC>(B, r, col0, h, active, head_lane, df, dl);
}

namespace {

// the walks of the forward and of the backward's destination pass (feat and
// the head's el at the neighbour), and of its source pass (dZ at the neighbour)
template <int C, bool OV>
using SpGat = Spec<T_NBR, OK_FULL, T_NBR, OK_HEAD, C, false, true, OV>;
template <int C, bool OV>
using SpGatOut = Spec<T_NBR, OK_FULL, DYN, DYN, C, false, true, OV>;

template <typename T, int V>
constexpr bool gat_fast = (sizeof(T) == 4 && V == 4) || (sizeof(T) == 2 && (V == 4 || V == 8));

template <typename T, int V, bool ATTN, bool OV>
void gat_launch_t(const EngineArgs& a, const GatArgs& g, int gc, hipStream_t s) {
    const dim3 grid(blocks_for_waves(a.sch.w_total)), block(WAVE * WPB);
    if constexpr (gat_fast<T, V>) {
        if (gc > 0) {
            GNNK_GC_DISPATCH(gc, {
                hipLaunchKernelGGL((gat_kernel<T, V, SpGat<C, OV>, ATTN>), grid, block, 0, s, a, g);
            })
            return;
        }
    }
    hipLaunchKernelGGL((gat_kernel<T, V, SpGat<0, OV>, ATTN>), grid, block, 0, s, a, g);
}

template <typename T, int V, bool OV>
void gat_ov(const EngineArgs& a, const GatArgs& g, int gc, hipStream_t s) {
    if (g.attn) gat_launch_t<T, V, true, OV>(a, g, gc, s);
    else gat_launch_t<T, V, false, OV>(a, g, gc, s);
    if (a.sch.n_hub > 0) {
        const dim3 block(WAVE * WPB);
        const dim3 cgrid(blocks_for_waves((a.sch.n_hub + a.geo.G - 1) / a.geo.G));
        hipLaunchKernelGGL((gat_combine_kernel<T, V, OV>), cgrid, block, 0, s, a, g);
        if (g.attn)
            hipLaunchKernelGGL((gat_attn_segments_kernel<T, V, OV>), dim3(blocks_for_waves(a.sch.n_seg)), block, 0, s,
                               a, g);
    }
}

template <typename T, int V>
void gat_all(const EngineArgs& a, const GatArgs& g, int gc, hipStream_t s) {
    if constexpr ((sizeof(T) == 4 && V == 4) || (sizeof(T) == 2 && V == 8)) {
        if (a.geo.ov) {
            gat_ov<T, V, true>(a, g, gc, s);
            return;
        }
    }
    gat_ov<T, V, false>(a, g, gc, s);
}

template <typename T, int V, bool OV>
void gat_bwd_ov(const EngineArgs& ain, const EngineArgs& aout, const GatBwdArgs& B, int gc, hipStream_t s) {
    const dim3 block(WAVE * WPB);
    if ((B.passes & 1) && ain.sch.w_total > 0) {
        const dim3 grid(blocks_for_waves(ain.sch.w_total));
        bool done = false;
        if constexpr (gat_fast<T, V>) {
            if (gc > 0) {
                GNNK_GC_DISPATCH(gc, {
                    hipLaunchKernelGGL((gat_bwd_dst_kernel<T, V, SpGat<C, OV>>), grid, block, 0, s, ain, B);
                })
                done = true;
            }
        }
        if (!done) hipLaunchKernelGGL((gat_bwd_dst_kernel<T, V, SpGat<0, OV>>), grid, block, 0, s, ain, B);
        if (ain.sch.n_hub > 0) {
            const int64_t n = (int64_t)ain.sch.n_hub * B.H;
            hipLaunchKernelGGL((gat_bwd_dst_combine_kernel<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                               ain, B);
        }
    }
    if ((B.passes & 2) && aout.sch.w_total > 0 && (B.d_feat || B.d_el)) {
        const dim3 grid(blocks_for_waves(aout.sch.w_total));
        bool done = false;
        if constexpr (gat_fast<T, V>) {
            if (gc > 0) {
                GNNK_GC_DISPATCH(gc, {
                    hipLaunchKernelGGL((gat_bwd_src_kernel<T, V, SpGatOut<C, OV>>), grid, block, 0, s, aout, B);
                })
                done = true;
            }
        }
        if (!done) hipLaunchKernelGGL((gat_bwd_src_kernel<T, V, SpGatOut<0, OV>>), grid, block, 0, s, aout, B);
        if (aout.sch.n_hub > 0)
            hipLaunchKernelGGL((gat_bwd_src_combine_kernel<T, V, OV>),
                               dim3(blocks_for_waves((aout.sch.n_hub + aout.geo.G - 1) / aout.geo.G)), block, 0, s,
                               aout, B);
    }
}

template <typename T, int V>
void gat_bwd_all(const EngineArgs& ain, const EngineArgs& aout, const GatBwdArgs& B, int gc, hipStream_t s) {
    if constexpr ((sizeof(T) == 4 && V == 4) || (sizeof(T) == 2 && V == 8)) {
        if (ain.geo.ov) {
            gat_bwd_ov<T, V, true>(ain, aout, B, gc, s);
            return;
        }
    }
    gat_bwd_ov<T, V, false>(ain, aout, B, gc, s);
}

}  // namespace

hipError_t launch_gat(const EngineArgs& a, const void* er, int64_t er_stride, void* attn, int64_t attn_stride,
                      float slope, void* row_ml, float* stats, int64_t stats_stride, int dtype, int vec, int gc,
                      hipStream_t s) {
    if (a.sch.w_total <= 0) return hipSuccess;
    GatArgs g{er, er_stride, attn, attn_stride, slope, 0, row_ml, stats, stats_stride};
    if (dtype == 0) {
        GNNK_VEC_DISPATCH_F32(vec, gat_all<float, V>(a, g, gc, s))
    } else {
        GNNK_VEC_DISPATCH_BF16(vec, gat_all<bf16_t, V>(a, g, gc, s))
    }
    return hipGetLastError();
}

hipError_t launch_gat_backward(const EngineArgs& ain, const EngineArgs& aout, const GatBwdArgs& b, int dtype, int vec,
                               int gc, hipStream_t s) {
    if (dtype == 0) {
        GNNK_VEC_DISPATCH_F32(vec, gat_bwd_all<float, V>(ain, aout, b, gc, s))
    } else {
        GNNK_VEC_DISPATCH_BF16(vec, gat_bwd_all<bf16_t, V>(ain, aout, b, gc, s))
    }
    return hipGetLastError();
}

}  // namespace gnnk
