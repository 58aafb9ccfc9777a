// hgt.hip -- HGT edge traversal for d = heads x d_k in {32, 64, 128}.
//
// Keys and values of every node come from node-typed GEMMs (K|V stored side
// by side, 512 bytes per node at d = 64) and are gathered once per edge.
// Both per-relation head matrices are moved to the destination side by linear
// operator reordering (Section "Linear Operator Reordering"):
//   a_e,i = (K_s,i Watt[r,i]) . Q_t,i  =  K_s,i . (Q_t,i Watt[r,i]^T)
//   sum_e alpha_e,i (V_s,i Wmsg[r,i])  =  (sum_e alpha_e,i V_s,i) Wmsg[r,i]
// The reordered query of every (destination, relation) segment, with the
// prior mu[r] and the attention scale folded in, is one typed GEMM over the
// segments (weights built by hgt_qp_weights_kernel); the traversal then only
// dots each key row with its segment's query row.  Wmsg is applied once per
// segment to the attention-weighted value sum, from LDS (shared by a
// 1024-thread workgroup) when it fits.
//
// Work items are those of the RGAT traversal (at most kChunkEdges edges: a
// bundle of small destinations or a piece of a large one), one per group of
// d / 4 lanes; lane l holds features 4l..4l+3, so head i is lanes
// [i*LH, (i+1)*LH) with LH = d_k / 4.  Each item first stages its edge
// sources and segment / destination boundaries in LDS, then streams the
// K|V rows of its edges, kU at a time with the next kU in flight; each
// segment's query row is loaded once, while the segment before it runs.
#include "hgt_weights.h"
#include "rgnn_internal.h"
#include "wave_ops.h"

namespace rgnn {

namespace {

__device__ __forceinline__ float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ void st4(float *p, float4 v) { *reinterpret_cast<float4 *>(p) = v; }
__device__ __forceinline__ float dot4(float4 a, float4 b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }
__device__ __forceinline__ float4 scale4(float4 a, float s) { return make_float4(a.x * s, a.y * s, a.z * s, a.w * s); }
__device__ __forceinline__ float4 lin4(float4 a, float s, float4 b, float t)
{
    return make_float4(a.x * s + b.x * t, a.y * s + b.y * t, a.z * s + b.z * t, a.w * s + b.w * t);
}
__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }
__device__ __forceinline__ float4 zero4() { return make_float4(0.f, 0.f, 0.f, 0.f); }

constexpr int kE = kChunkEdges, kDst = kMaxDstPerItem;
constexpr int kU = 2;                    // gathered K|V rows per batch

template <bool FQ>
struct HStage {
    int eidx[kE];          // source node of each edge
    int vptr[kE + 1];      // item-local edge offset of each virtual segment
    int vrel[kE];
    int dptr[kDst + 1];    // item-local edge offset of each destination
    int vdst[FQ ? kE : 1]; // destination of each virtual segment (queries formed in the kernel)
};

struct HK {
    int64_t n_items;
    const Item *items;
    const int32_t *item_slot, *dst_vsegptr, *vseg_ptr, *vseg_rel, *vseg_dst, *in_src;
    const float *KV, *QP, *Wmsg;
    const float *Q, *Watt, *mu;   // queries formed in the kernel: Q [N, d], Watt, mu, scale
    float scale;
    int R, ldq;            // ldq: row stride of QP
    float *agg, *partial;
    float *saved;          // [N, H, 2] per destination and head (max, sum), or NULL
};

// Value of lane jj of this lane's head (LH aligned lanes).  A DPP quad
// broadcast would serve LH = 4 without the LDS crossbar, but it lets the LDS
// matrix rows of several steps be hoisted ahead of their FMAs and the 1024-lane
// launch bound then spills; ds_bpermute keeps one step live at a time.
template <int G>
__device__ __forceinline__ float head_bcast(float v, int jj, int base)
{
    return __shfl(v, base + jj, G);
}

// y[4 values of this lane] = x_head (1 x dk) . Mat (dk x dk), Mat row-major,
// with x_head distributed over the head's LH lanes (4 values each).
// ROLLED: a loop instead of LH unrolled steps (one code copy where several
// call sites are inlined into the unrolled edge loop).
template <int LH, int G, bool ROLLED = false>
__device__ __forceinline__ float4 head_vecmat(float4 x, const float *Mt, int gl)
{
    constexpr int DK = LH * 4;
    const int base = (gl / LH) * LH;     // first lane of this head within the group
    const int c0 = 4 * (gl % LH);
    float4 y = zero4();
#pragma unroll(ROLLED ? 1 : LH)
    for (int jj = 0; jj < LH; ++jj) {
        const float x0 = head_bcast<G>(x.x, jj, base), x1 = head_bcast<G>(x.y, jj, base);
        const float x2 = head_bcast<G>(x.z, jj, base), x3 = head_bcast<G>(x.w, jj, base);
        y = lin4(y, 1.f, ld4(Mt + (4 * jj + 0) * DK + c0), x0);
        y = lin4(y, 1.f, ld4(Mt + (4 * jj + 1) * DK + c0), x1);
        y = lin4(y, 1.f, ld4(Mt + (4 * jj + 2) * DK + c0), x2);
        y = lin4(y, 1.f, ld4(Mt + (4 * jj + 3) * DK + c0), x3);
        __builtin_amdgcn_sched_barrier(0);   // bound the live LDS rows to one step
    }
    return y;
}

// FQ: the reordered query of each segment, Q_t,i (mu[r] scale Watt[r, i]^T),
// is formed in the kernel at the segment's first edge from LDS-resident
// blocks (requires LDSW), with the next segment's Q row already in flight,
// instead of being read from a materialized [V, d] array.
template <int D, int H, bool LDSW, bool FQ, int kBlock>
__global__ __launch_bounds__(kBlock) void hgt_kernel(HK k)
{
    static_assert(!FQ || LDSW, "kernel-formed queries keep both weight sets in LDS");
    constexpr int G = D / 4, GPB = kBlock / G;
    constexpr int DK = D / H, LH = DK / 4;
    constexpr int MAT = H * DK * DK;            // floats per relation per matrix
    extern __shared__ float4 smem4[];
    float *smem = reinterpret_cast<float *>(smem4);
    const int nW = LDSW ? k.R * MAT : 0;
    const int nQ = FQ ? k.R * MAT : 0;
    HStage<FQ> *stages = reinterpret_cast<HStage<FQ> *>(smem + nW + nQ);
    const float *Wmsg = k.Wmsg;
    if (LDSW) {
        const int n4 = k.R * MAT / 4;
        for (int i = threadIdx.x; i < n4; i += kBlock) smem4[i] = reinterpret_cast<const float4 *>(k.Wmsg)[i];
        Wmsg = smem;
    }
    float *Wq = smem + nW;   // [R][H][j][n] = mu[r] scale Watt[r, i][n][j]
    if (FQ) {
        for (int idx = threadIdx.x; idx < nQ; idx += kBlock) {
            const int r = idx / MAT, rem = idx % MAT;
            const int i = rem / (DK * DK), j = rem / DK % DK, n = rem % DK;
            Wq[idx] = k.mu[r] * k.scale * k.Watt[(((size_t)r * H + i) * DK + n) * DK + j];
        }
    }
    const int gl = threadIdx.x % G, gi = threadIdx.x / G;
    HStage<FQ> &st = stages[gi];
    const int64_t item = (int64_t)blockIdx.x * GPB + gi;
    const bool valid = item < k.n_items;
    int dst0 = 0, nd = 0, vs0 = 0, nv = 0, e0 = 0, ne = 0, slot = -1;
    if (valid) {
        const Item x = k.items[item];
        dst0 = x.dst0; nd = x.dst1 - x.dst0; vs0 = x.vs0; nv = x.vs1 - x.vs0;
        e0 = k.vseg_ptr[x.vs0]; ne = k.vseg_ptr[x.vs1] - e0;
        slot = k.item_slot[item];
        for (int j = gl; j < nv; j += G) {
            const int a = k.vseg_ptr[vs0 + j] - e0;
            st.vptr[j] = a;
            st.vrel[j] = k.vseg_rel[vs0 + j];
            if (FQ) st.vdst[j] = k.vseg_dst[vs0 + j];
        }
        if (gl == 0) st.vptr[nv] = ne;
        auto dst_edge = [&](int jj) {
            int vs = k.dst_vsegptr[dst0 + jj];
            vs = vs < vs0 ? vs0 : (vs > vs0 + nv ? vs0 + nv : vs);
            return k.vseg_ptr[vs] - e0;
        };
        for (int j = gl; j < nd; j += G) st.dptr[j] = dst_edge(j);
        if (gl == 0) st.dptr[nd] = ne;
        for (int e = gl; e < ne; e += G) st.eidx[e] = k.in_src[e0 + e];
    }
    __syncthreads();
    if (!valid) return;

    const int head = gl / LH;
    float m = -INFINITY, s = 0.f;
    float4 agg = zero4(), vacc = zero4();
    auto flush = [&](int jj) {
        if (slot < 0) {
            st4(k.agg + (size_t)(dst0 + jj) * D + gl * 4, scale4(agg, s > 0.f ? 1.f / s : 0.f));
            if (k.saved && gl % LH == 0)
                *reinterpret_cast<float2 *>(k.saved + ((size_t)(dst0 + jj) * H + head) * 2) =
                    make_float2(s > 0.f ? m : 0.f, s);
        } else {
            float *pr = k.partial + (size_t)slot * (2 * H + D);
            if (gl % LH == 0) { pr[head * 2] = m; pr[head * 2 + 1] = s; }
            st4(pr + 2 * H + gl * 4, agg);
        }
        m = -INFINITY; s = 0.f; agg = zero4();
    };
    int j = 0, jv = 0;
    while (j < nd && st.dptr[j + 1] == st.dptr[j]) { flush(j); ++j; }
    // qcur: FQ, the Q row of segment jv's destination; otherwise segment jv's
    // reordered query row, loaded one segment ahead.  qp: segment jv's query.
    float4 qcur = zero4(), qp = zero4();
    if (ne > 0) qcur = FQ ? ld4(k.Q + (size_t)st.vdst[0] * D + gl * 4) : ld4(k.QP + (size_t)vs0 * k.ldq + gl * 4);
    if (ne > 0) {
        // Ping-pong batches: batch A is consumed while batch B is in flight.
        // Each edge brings its K|V row; each segment's query row is read once,
        // at the segment before it.
        float4 Ak[kU], Av[kU], Bk[kU], Bv[kU];
        auto load = [&](float4 (&Xk)[kU], float4 (&Xv)[kU], int base) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int e = base + u < ne ? base + u : ne - 1;
                const size_t row = (size_t)st.eidx[e] * (2 * D);
                Xk[u] = ld4(k.KV + row + gl * 4);
                Xv[u] = ld4(k.KV + row + D + gl * 4);
            }
        };
        auto consume = [&](const float4 (&Xk)[kU], const float4 (&Xv)[kU], int base) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int e = base + u;
                if (e < ne) {
                    if (e == st.vptr[jv]) {   // first edge of segment jv: its query
                        if (FQ) {
                            qp = head_vecmat<LH, G, true>(qcur, Wq + (size_t)st.vrel[jv] * MAT + (size_t)head * DK * DK, gl);
                            if (jv + 1 < nv && st.vdst[jv + 1] != st.vdst[jv])
                                qcur = ld4(k.Q + (size_t)st.vdst[jv + 1] * D + gl * 4);
                        } else {
                            qp = qcur;
                            if (jv + 1 < nv) qcur = ld4(k.QP + (size_t)(vs0 + jv + 1) * k.ldq + gl * 4);
                        }
                    }
                    const float a = gsum<LH>(dot4(Xk[u], qp));
                    const float mn = fmaxf(m, a);
                    const float c1 = __expf(m - mn), c2 = __expf(a - mn);
                    s = s * c1 + c2;
                    vacc = lin4(vacc, c1, Xv[u], c2);
                    agg = scale4(agg, c1);
                    m = mn;
                    if (e + 1 == st.vptr[jv + 1]) {
                        const size_t off = (size_t)st.vrel[jv] * MAT + (size_t)head * DK * DK;
                        agg = add4(agg, head_vecmat<LH, G>(vacc, Wmsg + off, gl));
                        vacc = zero4();
                        ++jv;
                        if (e + 1 == st.dptr[j + 1]) {
                            flush(j);
                            ++j;
                            while (j < nd && st.dptr[j + 1] == st.dptr[j]) { flush(j); ++j; }
                        }
                    }
                }
            }
        };
        load(Ak, Av, 0);
        __builtin_amdgcn_sched_barrier(0);
        for (int eb = 0; eb < ne; eb += 2 * kU) {
            load(Bk, Bv, eb + kU);
            __builtin_amdgcn_sched_barrier(0);
            consume(Ak, Av, eb);
            load(Ak, Av, eb + 2 * kU);
            __builtin_amdgcn_sched_barrier(0);
            consume(Bk, Bv, eb + kU);
        }
    }
    while (j < nd) { flush(j); ++j; }
}

// ---------------------------------------------------------------- wide heads
// Wmsg is applied by a typed GEMM over the segments instead of in the traversal,
// whose per-segment product of a dk-vector with a dk x dk matrix from LDS (or,
// beyond 160 KB of matrices, from L2) takes longer than the segment's gathers when
// dk is large: on 200 000 nodes and 1.5M edges the traversal took 0.685 ms at d =
// 64 with one head of 64 against 0.173 ms with four of 16, and 2.41 ms at d = 128
// with one head (hgt_seg_values has the rule and both sides).  Each segment keeps an
// online softmax of its own, (max, sum) per head and the value sum relative to that
// max; the destination's softmax is finished when the transformed rows are summed.
// No destination boundaries, weights or queries in LDS: 256-thread workgroups at
// the occupancy that the registers allow.
struct HSegK {
    int64_t n_items;
    const Item *items;
    const int32_t *vseg_ptr, *vseg_pos, *in_src;
    const float *KV, *QP;
    int ldq;
    float *Sv;      // [V, D] by-relation order: sum exp(a - m) V
    float *stat;    // [V, H, 2] vseg order: (m, sum exp(a - m))
};

struct HSegStage {
    int eidx[kE];          // source node of each edge
    int vptr[kE + 1];      // item-local edge offset of each virtual segment
    int vpos[kE];          // by-relation position of each virtual segment
};

template <int D, int H>
__global__ __launch_bounds__(256) void hgt_seg_kernel(HSegK k)
{
    constexpr int G = D / 4, GPB = 256 / G, LH = G / H;
    __shared__ HSegStage stage[GPB];
    const int gl = threadIdx.x % G, gi = threadIdx.x / G;
    HSegStage &st = stage[gi];
    const int64_t item = (int64_t)blockIdx.x * GPB + gi;
    int vs0 = 0, nv = 0, ne = 0;
    if (item < k.n_items) {
        const Item x = k.items[item];
        vs0 = x.vs0; nv = x.vs1 - x.vs0;
        const int e0 = k.vseg_ptr[x.vs0];
        ne = k.vseg_ptr[x.vs1] - e0;
        for (int j = gl; j < nv; j += G) {
            st.vptr[j] = k.vseg_ptr[vs0 + j] - e0;
            st.vpos[j] = k.vseg_pos[vs0 + j];
        }
        if (gl == 0) st.vptr[nv] = ne;
        for (int e = gl; e < ne; e += G) st.eidx[e] = k.in_src[e0 + e];
    }
    __syncthreads();
    if (ne == 0) return;
    const int head = gl / LH;
    float m = -INFINITY, s = 0.f;
    float4 vacc = zero4();
    int jv = 0;
    // ping-pong batches of K|V rows; each segment's query row one segment ahead
    const float *qp = k.QP + (size_t)vs0 * k.ldq + gl * 4;
    float4 qn = ld4(qp), q = zero4();
    float4 Ak[kU], Av[kU], Bk[kU], Bv[kU];
    auto load = [&](float4 (&Xk)[kU], float4 (&Xv)[kU], int base) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = base + u < ne ? base + u : ne - 1;
            const size_t row = (size_t)st.eidx[e] * (2 * D);
            Xk[u] = ld4(k.KV + row + gl * 4);
            Xv[u] = ld4(k.KV + row + D + gl * 4);
        }
    };
    auto consume = [&](const float4 (&Xk)[kU], const float4 (&Xv)[kU], int base) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = base + u;
            if (e < ne) {
                if (e == st.vptr[jv]) {
                    q = qn;
                    if (jv + 1 < nv) qn = ld4(qp + (size_t)(jv + 1) * k.ldq);
                }
                const float a = gsum<LH>(dot4(Xk[u], q));
                const float mn = fmaxf(m, a);
                const float c1 = __expf(m - mn), c2 = __expf(a - mn);
                s = s * c1 + c2;
                vacc = lin4(vacc, c1, Xv[u], c2);
                m = mn;
                if (e + 1 == st.vptr[jv + 1]) {
                    st4(k.Sv + (size_t)st.vpos[jv] * D + gl * 4, vacc);
                    if (gl % LH == 0)
                        *reinterpret_cast<float2 *>(k.stat + ((size_t)(vs0 + jv) * H + head) * 2) = make_float2(m, s);
                    m = -INFINITY; s = 0.f; vacc = zero4();
                    ++jv;
                }
            }
        }
    };
    load(Ak, Av, 0);
    __builtin_amdgcn_sched_barrier(0);
    for (int eb = 0; eb < ne; eb += 2 * kU) {
        load(Bk, Bv, eb + kU);
        __builtin_amdgcn_sched_barrier(0);
        consume(Ak, Av, eb);
        load(Ak, Av, eb + 2 * kU);
        __builtin_amdgcn_sched_barrier(0);
        consume(Bk, Bv, eb + kU);
    }
}

// out_t = sum_i exp(m_i - M) T_i / Z per head over t's segments i (+ residual), with
// M = max m_i and Z = sum s_i exp(m_i - M), (M, Z) to saved: a group of D / 4 lanes per
// destination merges its segments' states online, four rows in flight.  Blocks [0,
// nbig) take the destinations of big_vdst, the groups of a workgroup each a
// strided share, the groups' states merged in group order.
template <int D, int H>
__global__ __launch_bounds__(256) void hgt_seg_reduce_kernel(int64_t N, int64_t nbig, const int32_t *big_vdst,
                                                             const int32_t *dst_vsegptr, const float *T,
                                                             const float *stat, const float *residual, float *out,
                                                             float *saved)
{
    constexpr int G = D / 4, NG = 256 / G, LH = G / H, U = 4;
    __shared__ float4 pacc[NG * G];
    __shared__ float2 pms[NG * H];
    const int gl = threadIdx.x % G, gi = threadIdx.x / G, head = gl / LH;
    const bool big = (int64_t)blockIdx.x < nbig;
    int64_t v;
    if (big) v = big_vdst[blockIdx.x];
    else v = ((int64_t)blockIdx.x - nbig) * NG + gi;
    if (v >= N) return;   // never in a big workgroup
    const int b = dst_vsegptr[v], e = dst_vsegptr[v + 1];
    if (!big && e - b > kBigRange) return;
    float m = -INFINITY, s = 0.f;
    float4 acc = zero4();
    auto merge = [&](float mi, float si, float4 t) {
        const float mn = fmaxf(m, mi);
        const float c1 = __expf(m - mn), c2 = __expf(mi - mn);
        s = s * c1 + si * c2;
        acc = lin4(acc, c1, t, c2);
        m = mn;
    };
    const int step = big ? NG : 1;
    for (int i0 = b + (big ? gi : 0); i0 < e; i0 += U * step) {
        float4 t[U];
        float2 ms[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * step < e ? i0 + u * step : i0;
            t[u] = ld4(T + (size_t)i * D + gl * 4);
            ms[u] = *reinterpret_cast<const float2 *>(stat + ((size_t)i * H + head) * 2);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * step < e) merge(ms[u].x, ms[u].y, t[u]);
    }
    if (big) {
        pacc[gi * G + gl] = acc;
        if (gl % LH == 0) pms[gi * H + head] = make_float2(m, s);
        __syncthreads();
        if (gi != 0) return;
        for (int j = 1; j < NG; ++j)   // groups without segments skipped; a NaN sum is merged
            if (!(pms[j * H + head].y == 0.f)) merge(pms[j * H + head].x, pms[j * H + head].y, pacc[j * G + gl]);
    }
    float4 o = scale4(acc, s > 0.f ? 1.f / s : 0.f);
    if (residual) o = add4(o, ld4(residual + (size_t)v * D + gl * 4));
    st4(out + (size_t)v * D + gl * 4, o);
    if (saved && gl % LH == 0)
        *reinterpret_cast<float2 *>(saved + ((size_t)v * H + head) * 2) = make_float2(s > 0.f ? m : 0.f, s);
}

// Wf[r][a][g] = sum_b Wmsg[r][a][b] Wa[t(r)][b][g] (one head): the output linear
// folded into the message weights.
__global__ __launch_bounds__(256) void hgt_out_fold_kernel(const float *Wmsg, const float *Wa,
                                                           const int32_t *rel_dsttype, int R, int D, float *Wf)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)R * D * D) return;
    const int r = (int)(idx / (D * D)), a = (int)(idx / D % D), g = (int)(idx % D);
    const float *wm = Wmsg + ((size_t)r * D + a) * D;
    const float *wa = Wa + (size_t)rel_dsttype[r] * D * D + g;
    float acc = 0.f;
#pragma unroll 16
    for (int b = 0; b < D; ++b) acc = fmaf(wm[b], wa[(size_t)b * D], acc);
    Wf[idx] = acc;
}

__global__ __launch_bounds__(256) void hgt_msgT_weights_kernel(const float *Wmsg, int R, int D, int heads, float *Wmt)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx < (int64_t)R * D * D) Wmt[idx] = hgt_msgT_entry(idx, Wmsg, D, heads);
}

constexpr size_t kLds = 160 * 1024;   // of a CU

constexpr size_t weight_bytes(int D, int R, int heads)
{
    return (size_t)R * heads * (D / heads) * (D / heads) * sizeof(float);
}

template <int D, bool FQ>
constexpr size_t stage_bytes(int threads) { return (size_t)(threads / (D / 4)) * sizeof(HStage<FQ>); }

// Threads per workgroup of the traversal, which stages the weights once per
// workgroup.  1024 where the matrices take most of the LDS (d = 64, 2 heads of 32:
// 2.43 ms against 3.41 with 512), 512 at d = 32, whose 128 item stages of 1024
// threads would not fit.  With d = 64 and heads of 16 two workgroups of 512 are a
// finer grid than one of 1024 at the same occupancy (7 relations, 1.9M nodes: 1.96
// -> 1.91 ms, 85 000 nodes 0.132 -> 0.118; 256 threads 2.12 and 0.116) as long as
// both keep their matrices in LDS, up to 12 relations; from 13 on one of 512 would
// leave the CU half empty where one of 1024 fits, up to 25; one of 512 with its
// matrices in LDS beats reading them from L2, up to 32; beyond that the stages are
// all the LDS it takes.  Forward on 200 000 nodes, 1.5M edges, us, 1024 / 512
// threads: 12 relations 437 / 428, 13 443 / 478, 20 475 / 507, 25 493 / 523, 26
// (1024: matrices from L2) 657 / 526, 32 676 / 541, 40 700 / 693.
template <int D, int H>
constexpr int traverse_threads(int R)
{
    if (D == 32) return 512;
    if (D / H > 16 || D == 128) return 1024;
    const size_t wb = weight_bytes(D, R, H);
    const bool two = 2 * (stage_bytes<D, false>(512) + wb) <= kLds;
    return !two && stage_bytes<D, false>(1024) + wb <= kLds ? 1024 : 512;
}
static_assert(traverse_threads<64, 4>(12) == 512 && traverse_threads<64, 4>(13) == 1024 &&
                  traverse_threads<64, 4>(25) == 1024 && traverse_threads<64, 4>(26) == 512,
              "the comment above has the relation counts");

__global__ void hgt_qp_weights_kernel(const float *Watt, const float *mu, float scale, int R, int D,
                                      int heads, float *Wqp)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)R * D * D) return;
    const int r = (int)(idx / (D * D)), j = (int)(idx / D % D), n = (int)(idx % D);
    const int dk = D / heads, i = j / dk;
    float v = 0.f;
    if (n / dk == i)
        v = mu[r] * scale * Watt[(((size_t)r * heads + i) * dk + (n - i * dk)) * dk + (j - i * dk)];
    Wqp[idx] = v;
}

__global__ __launch_bounds__(256) void hgt_qp_fold_kernel(const float *Wq, const float *Watt, const float *mu,
                                                          float scale, const int32_t *rel_dsttype, int R, int D,
                                                          int heads, float *Wc)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx < (int64_t)R * D * D) Wc[idx] = hgt_qp_fold_entry(idx, Wq, Watt, mu, scale, rel_dsttype, D, heads);
}

// whether the traversal's workgroups hold every relation's Wmsg
template <int D, int H>
bool wmsg_in_lds(int R) { return weight_bytes(D, R, H) + stage_bytes<D, false>(traverse_threads<D, H>(R)) <= kLds; }

template <int D, int H, int NTH>
hipError_t launch_hgt_threads(const HK &k, int64_t n_items, int R, hipStream_t s)
{
    const size_t wb = weight_bytes(D, R, H);
    constexpr int GPB = NTH / (D / 4);
    const unsigned nb = (unsigned)((n_items + GPB - 1) / GPB);
    hipError_t e;
#define HGT_LAUNCH(LDSW, FQ, LDS)                                                                          \
    do {                                                                                                   \
        e = hipFuncSetAttribute((const void *)hgt_kernel<D, H, LDSW, FQ, NTH>,                             \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)(LDS));                   \
        if (e == hipSuccess)                                                                               \
            hipLaunchKernelGGL((hgt_kernel<D, H, LDSW, FQ, NTH>), dim3(nb), dim3(NTH), (LDS), s, k);       \
    } while (0)
    if (!k.QP) {   // queries formed in the kernel (the caller checked that both weight sets fit)
        if constexpr (D == 128) HGT_LAUNCH(true, true, (stage_bytes<D, true>(NTH) + 2 * wb));
        else e = hipErrorInvalidValue;
    } else if (wmsg_in_lds<D, H>(R)) {
        HGT_LAUNCH(true, false, (stage_bytes<D, false>(NTH) + wb));
    } else if constexpr (D / H < 32 && NTH == traverse_threads<D, H>(1 << 16)) {
        HGT_LAUNCH(false, false, (stage_bytes<D, false>(NTH)));   // (wide heads with more matrices take the segment GEMM)
    } else {
        e = hipErrorInvalidValue;
    }
#undef HGT_LAUNCH
    return e;
}

template <int D, int H>
hipError_t launch_hgt_shape(const HK &k, int64_t n_items, int R, hipStream_t s)
{
    if constexpr (D == 64 && D / H == 16)
        return traverse_threads<D, H>(R) == 512 ? launch_hgt_threads<D, H, 512>(k, n_items, R, s)
                                                : launch_hgt_threads<D, H, 1024>(k, n_items, R, s);
    else
        return launch_hgt_threads<D, H, traverse_threads<D, H>(1)>(k, n_items, R, s);
}

}  // namespace

// Whether Wmsg leaves the traversal for a GEMM over the segments (see "wide
// heads"): always for dk >= 64, for dk = 32 at d = 32 and where the matrices do
// not fit in LDS, never for dk = 16.  ms per forward, traversal -> GEMM, 200 000
// nodes and 1.5M edges, typed graph of 7 relations / one type and 40 relations (both
// sides with the query GEMM's tiles by destination range; with 40 relations it takes
// them by relation since, 0.02 ms less at d = 64 and 0.16 at d = 128):
//   d = 64,  1 head of 64   0.80 -> 0.32 / 1.46 -> 0.69
//   d = 128, 1 head of 128  2.72 -> 0.71,  2 heads of 64  1.30 -> 0.75
//   d = 32,  1 head of 32   0.25 -> 0.16 / 0.47 -> 0.36
//   d = 64,  2 heads of 32  0.36 -> 0.34 / 0.98 -> 0.73 (12 relations, in LDS: 0.53 -> 0.61)
//   d = 128, 4 heads of 32  0.65 -> 0.73 / 2.11 -> 1.69
//   d = 64,  4 heads of 16  0.29 -> 0.35 / 0.70 -> 0.74
bool hgt_seg_values(int R, int d, int heads)
{
    const int dk = d / heads;
    if (dk >= 64) return true;
    if (dk < 32) return false;
    return d == 32 || !(d == 64 ? wmsg_in_lds<64, 2>(R) : wmsg_in_lds<128, 4>(R));
}

rgnn_status launch_hgt_msgT_weights(const float *Wmsg, int R, int d, int heads, float *Wmt, hipStream_t s)
{
    const int64_t n = (int64_t)R * d * d;
    if (n == 0) return RGNN_OK;
    LaunchScope ls("hgt_msgT_weights", s);
    hipLaunchKernelGGL(hgt_msgT_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Wmsg, R, d, heads,
                       Wmt);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? RGNN_OK : hip_fail(e, "hgt_msgT_weights launch");
}

namespace {

// The traversal, message GEMM and reduction of wide heads.  With fold_out (one
// head, typed relations) the output linear is part of the GEMM's weight.
rgnn_status launch_hgt_seg(const HgtArgs &a, hipStream_t s)
{
    const rgnn_graph *g = a.g;
    const int d = a.d, H = a.heads;
    rgnn_status st;
    hipError_t e;
    if (a.fold_out && H != 1) return fail(RGNN_EINVAL, "the output linear folds into one head's messages only");
    if (g->V > 0) {
        HSegK k{};
        k.n_items = g->n_items; k.items = g->dev.items; k.vseg_ptr = g->dev.vseg_ptr; k.vseg_pos = g->dev.vseg_pos;
        k.in_src = g->dev.in_src; k.KV = a.KV; k.QP = a.QP; k.ldq = a.ldq ? a.ldq : d; k.Sv = a.Sv; k.stat = a.stat;
        const unsigned nb = (unsigned)((g->n_items + 1024 / d - 1) / (1024 / d));
        bool ok = true;
        {
            LaunchScope ls("hgt_traverse", s);
#define HSEG(D, H) hipLaunchKernelGGL((hgt_seg_kernel<D, H>), dim3(nb), dim3(256), 0, s, k)
            if (d == 32 && H == 1) HSEG(32, 1);
            else if (d == 64 && H == 1) HSEG(64, 1);
            else if (d == 64 && H == 2) HSEG(64, 2);
            else if (d == 128 && H == 1) HSEG(128, 1);
            else if (d == 128 && H == 2) HSEG(128, 2);
            else if (d == 128 && H == 4) HSEG(128, 4);
            else ok = false;
#undef HSEG
        }
        if (!ok) return fail(RGNN_EUNSUPPORTED, "HGT segment traversal: unsupported (d, heads)");
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt segment traversal launch");
        GemmArgs gm;
        gm.split_bf16 = 1;
        gm.X = a.Sv; gm.ldx = d; gm.W[0] = a.Wt; gm.K = d; gm.Nc = d;
        gm.tiles = g->gemm_tiles(kRowsVsegs);
        gm.Y = a.T; gm.ldy = d; gm.scatter = g->dev.vseg_byrel;
        if (a.fold_out) {
            const int64_t n = (int64_t)g->R * d * d;
            {
                LaunchScope ls("hgt_msgT_weights", s);
                hipLaunchKernelGGL(hgt_out_fold_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a.Wmsg,
                                   a.Wa, g->dev.rel_dsttype, g->R, d, a.Wt);
            }
            if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_out_fold launch");
        } else {
            if ((st = launch_hgt_msgT_weights(a.Wmsg, g->R, d, H, a.Wt, s)) != RGNN_OK) return st;
            gm.trans_b = 1; gm.ep.diag_blocks = H;
        }
        if ((st = launch_typed_gemm(gm, s)) != RGNN_OK) return st;
    }
    if (g->N == 0) return RGNN_OK;
    const int64_t nbig = g->n_big_vdst;
    const unsigned nr = (unsigned)(nbig + (g->N + 1024 / d - 1) / (1024 / d));
    {
        LaunchScope ls("hgt_seg_reduce", s);
#define HRED(D, H) hipLaunchKernelGGL((hgt_seg_reduce_kernel<D, H>), dim3(nr), dim3(256), 0, s, g->N, nbig, \
                                      g->dev.big_vdst, g->dev.dst_vsegptr, a.T, a.stat, a.residual, a.agg, a.saved)
        if (d == 32) HRED(32, 1);
        else if (d == 64 && H == 1) HRED(64, 1);
        else if (d == 64) HRED(64, 2);
        else if (H == 1) HRED(128, 1);
        else if (H == 2) HRED(128, 2);
        else HRED(128, 4);
#undef HRED
    }
    e = hipGetLastError();
    return e == hipSuccess ? RGNN_OK : hip_fail(e, "hgt_seg_reduce launch");
}

}  // namespace

rgnn_status launch_hgt_traverse(const HgtArgs &a, hipStream_t s)
{
    const rgnn_graph *g = a.g;
    if (hgt_seg_values(g->R, a.d, a.heads)) return launch_hgt_seg(a, s);
    if (g->n_items == 0) return RGNN_OK;
    HK k{};
    k.n_items = g->n_items; k.items = g->dev.items; k.item_slot = g->dev.item_slot;
    k.dst_vsegptr = g->dev.dst_vsegptr; k.vseg_ptr = g->dev.vseg_ptr;
    k.vseg_rel = g->dev.vseg_rel; k.vseg_dst = g->dev.vseg_dst; k.in_src = g->dev.in_src;
    k.KV = a.KV; k.QP = a.QP; k.Wmsg = a.Wmsg;
    k.Q = a.Q; k.Watt = a.Watt; k.mu = a.mu; k.scale = a.scale;
    if (!a.QP && !(a.Q && a.Watt && a.mu && hgt_fused_query_fits(g->R, a.d, a.heads)))
        return fail(RGNN_EINVAL, "HGT traversal without segment queries needs Q, Watt, mu and LDS room");
    k.R = g->R; k.ldq = a.ldq ? a.ldq : a.d; k.agg = a.agg; k.partial = a.partial; k.saved = a.saved;
    LaunchScope ls("hgt_traverse", s);
    hipError_t e;
    const int64_t n = g->n_items;
    const int R = g->R;
    if (a.d == 32 && a.heads == 2) e = launch_hgt_shape<32, 2>(k, n, R, s);
    else if (a.d == 64 && a.heads == 2) e = launch_hgt_shape<64, 2>(k, n, R, s);
    else if (a.d == 64 && a.heads == 4) e = launch_hgt_shape<64, 4>(k, n, R, s);
    else if (a.d == 128 && a.heads == 4) e = launch_hgt_shape<128, 4>(k, n, R, s);
    else if (a.d == 128 && a.heads == 8) e = launch_hgt_shape<128, 8>(k, n, R, s);
    else return fail(RGNN_EUNSUPPORTED, "HGT traversal: unsupported (d, heads)");
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute (HGT LDS)");
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "hgt traversal launch");
    return launch_merge_partials(g, a.d, a.heads, 1, a.partial, a.agg, a.saved, 0, s);
}

bool hgt_fused_query_fits(int R, int d, int heads)
{
    // instantiated at d = 128 only, the width where it beats the segment-query
    // GEMM, and not for wide heads, whose traversal has no weights in LDS
    if (d != 128 || hgt_seg_values(R, d, heads)) return false;
    return stage_bytes<128, true>(1024) + 2 * weight_bytes(d, R, heads) <= kLds;
}

rgnn_status launch_hgt_qp_weights(const float *Watt, const float *mu, float scale, int R, int d,
                                  int heads, float *Wqp, hipStream_t s)
{
    if (d != 32 && d != 64 && d != 128) return fail(RGNN_EUNSUPPORTED, "HGT supports d = 32, 64, 128");
    const int64_t n = (int64_t)R * d * d;
    if (n == 0) return RGNN_OK;
    LaunchScope ls("hgt_qp_weights", s);
    hipLaunchKernelGGL(hgt_qp_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Watt, mu, scale,
                       R, d, heads, Wqp);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? RGNN_OK : hip_fail(e, "hgt_qp_weights launch");
}

rgnn_status launch_hgt_qp_fold(const float *Wq, const float *Watt, const float *mu, float scale,
                               const int32_t *rel_dsttype, int R, int d, int heads, float *Wc, hipStream_t s)
{
    if (d != 32 && d != 64 && d != 128) return fail(RGNN_EUNSUPPORTED, "HGT supports d = 32, 64, 128");
    const int64_t n = (int64_t)R * d * d;
    if (n == 0) return RGNN_OK;
    LaunchScope ls("hgt_qp_weights", s);
    hipLaunchKernelGGL(hgt_qp_fold_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Wq, Watt, mu, scale,
                       rel_dsttype, R, d, heads, Wc);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? RGNN_OK : hip_fail(e, "hgt_qp_fold launch");
}

}  // namespace rgnn
