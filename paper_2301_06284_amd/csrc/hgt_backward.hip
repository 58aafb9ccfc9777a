// hgt_backward.hip -- HGT backward pass for the loss L = sum(out * G), the
// chain rule of the HGT layer (Section "Backward Propagation" derives the
// backward from the forward; here it is written out), for d in {32, 64, 128}
// and d / heads >= 16.  With the forward's reordered segment queries QP_vs = c_r Q_t
// Watt[r]^T per head (c_r = mu[r] * scale), the per-edge score a_e = K_s . QP_vs,
// alpha_e its softmax over the destination's in-edges (saved max M_t and sum
// Z_t), and dagg = G Wa^T (or G):
//   dP_vs   = dagg_t Wmsg[r]^T                (per head; so dalpha_e = V_s . dP_vs)
//   s_t     = sum_e alpha_e dalpha_e,   da_e = alpha_e (dalpha_e - s_t)
//   dK_s    = sum over s's out-edges of da_e QP_vs
//   dV_s    = sum over s's out-edges of alpha_e dP_vs
//   dQP_vs  = sum_{e in vs} da_e K_s = A_vs - s_t B_vs,
//             A_vs = sum alpha dalpha K_s,  B_vs = sum alpha K_s
//   dQ_t    = sum over t's segments of dQP_vs Wqp[r]^T
//   dWatt[r] = c_r (sum_vs dQP_vs^T Q_t)[head blocks],  dmu[r] = scale <., Watt[r]>
//   dWmsg[r] = (sum_vs Salpha_vs^T dagg_t)[head blocks],  Salpha_vs = sum alpha V_s
//   dWa = sum_t agg_t^T G_t,  dh = dK Wk^T + dV Wv^T + dQ Wq^T (+ G with the residual)
//   dWk = sum_n h_n^T dK_n (per node type), likewise dWv, dWq.
//
// Kernel sequence: the forward (K|V|Q GEMM, segment queries, traversal with
// its softmax statistics) is recomputed; dagg and dWa; the block-diagonal
// W_msg^T and the segment rows dP (typed GEMM), kept beside the segment queries
// (one 2d-float row QP | dP per segment, so that the source-major pass gathers
// 512 contiguous bytes per out-edge at d = 64); a destination-major pass over
// the forward's work items (per edge alpha and dalpha from the K|V row and the
// segment's QP and dP rows; per segment Salpha, A, B; per destination s); the
// split destinations' s merged in slot order; dQP; dQ by the typed GEMM and
// the segment reduction; the per-relation outer products (MFMA chunks);
// a source-major pass over the out-edge index that recomputes alpha and da per
// out-edge and writes dK|dV once per source (float atomics only for pieces of
// sources with more than kChunkEdges out-edges); dh and the per-type weight
// gradients by typed GEMMs and outer-product chunks.
//
// With typed relations (every relation's destinations of one node type, the
// case of heterogeneous graphs) and not too many of them for the graph's size
// (fold_types) the node-type weights Wq and Wa are folded into
// the per-relation ones instead (see "typed relations" below): no Q, dagg,
// rebuilt aggregate or dQ, and two outer products over all nodes fewer.
// 950 000 nodes, 10.5M edges, d = 64, 4 heads: 5.11 -> 4.28 ms.
#include "hgt_weights.h"
#include "rgnn_internal.h"
#include "wave_ops.h"

namespace rgnn {

namespace {

constexpr int kE = kChunkEdges, kDst = kMaxDstPerItem;
constexpr int kU = 2;             // edges per prefetch batch

__device__ __forceinline__ float4 ld4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ void st4(float *p, float4 v) { *reinterpret_cast<float4 *>(p) = v; }
__device__ __forceinline__ float dot4(float4 a, float4 b) { return a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w; }
__device__ __forceinline__ float4 zero4() { return make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ __forceinline__ float4 axpy4(float4 y, float a, float4 x)
{
    return make_float4(y.x + a * x.x, y.y + a * x.y, y.z + a * x.z, y.w + a * x.w);
}
__device__ __forceinline__ void atomic_add4(float *p, float4 v)
{
    atomicAdd(p + 0, v.x); atomicAdd(p + 1, v.y); atomicAdd(p + 2, v.z); atomicAdd(p + 3, v.w);
}

// ---------------------------------------------------------------- destination-major pass
// dQP = A - s_t B needs s_t, which is known at the destination's last edge only.
// A destination of this pass with at most kHeldSegs segments (and no more edges
// than one item) keeps A and B of all but its last one in LDS until then, each
// lane its own four features, and writes dQP itself; the others leave A in dQP's
// place and B beside it for hgt_bwd_dqp_kernel.  Three segments cover the
// destinations of graphs with a few relations per node type.  The registers (106 to
// 112) allow four waves per SIMD; with two held segments the workgroup's LDS is 24
// KB at d = 128, 31 KB at d = 64 (a third would be 39 KB and leave four) and 46 KB at
// d = 32, where it leaves three.  Writing A and B and combining all of them in a pass
// of its own took 1.10 + 0.25 ms on the 950 000-node graph at d = 64, 4 heads.
constexpr int kHeldSegs = 3;
__device__ __forceinline__ bool dqp_in_pass(int segs, int edges) { return segs <= kHeldSegs && edges <= kE; }

template <int D>
struct DStage {
    int eidx[kE];                  // source node of each edge
    int vptr[kE + 1];              // item-local first edge of each virtual segment
    int vpos[kE];                  // by-relation position of each virtual segment
    int dvs[kDst + 1];             // item-local first virtual segment of each destination
    float4 held[kHeldSegs - 1][2][D / 4];   // A and B of a destination's earlier segments
};

struct DKArgs {
    int64_t n_items;
    const Item *items;
    const int32_t *item_slot, *dst_vsegptr, *vseg_ptr, *in_src, *vseg_pos;
    const float *KV, *QD, *saved;   // QD [V, 2D]: QP | dP of each virtual segment
    float *Sal, *dQP, *Bac, *spart;
    float4 *rec;   // [N, H] (max, 1 / sum, s, 0) per destination and head, for the source-major pass
};

template <int D, int H>
__global__ __launch_bounds__(256) void hgt_bwd_dst_kernel(DKArgs k)
{
    constexpr int G = D / 4, GPB = 256 / G;
    constexpr int DKH = D / H, LH = DKH / 4;
    __shared__ DStage<D> stage[GPB];
    const int gl = threadIdx.x % G, gi = threadIdx.x / G;
    DStage<D> &st = stage[gi];
    const int64_t item = (int64_t)blockIdx.x * GPB + gi;
    const bool valid = item < k.n_items;
    int dst0 = 0, nd = 0, vs0 = 0, nv = 0, e0 = 0, ne = 0, slot = -1;
    if (valid) {
        const Item x = k.items[item];
        dst0 = x.dst0; nd = x.dst1 - x.dst0; vs0 = x.vs0; nv = x.vs1 - x.vs0;
        e0 = k.vseg_ptr[x.vs0]; ne = k.vseg_ptr[x.vs1] - e0;
        slot = k.item_slot[item];
        for (int j = gl; j < nv; j += G) {
            st.vptr[j] = k.vseg_ptr[vs0 + j] - e0;
            st.vpos[j] = k.vseg_pos[vs0 + j];
        }
        if (gl == 0) st.vptr[nv] = ne;
        for (int j = gl; j < nd; j += G) {
            const int vs = k.dst_vsegptr[dst0 + j] - vs0;
            st.dvs[j] = vs < 0 ? 0 : (vs > nv ? nv : vs);
        }
        if (gl == 0) st.dvs[nd] = nv;
        for (int e = gl; e < ne; e += G) st.eidx[e] = k.in_src[e0 + e];
    }
    __syncthreads();
    if (!valid) return;

    const int head = gl / LH;
    float4 sal = zero4(), aac = zero4(), bac = zero4();
    float sacc = 0.f;
    int j = 0, jv = 0;
    // (max, 1 / sum) of destination j for this lane's head, read one destination ahead
    float dm = 0.f, dzi = 0.f;
    float2 next = make_float2(0.f, 0.f);
    auto load_next = [&](int jj) {
        if (jj < nd) next = *reinterpret_cast<const float2 *>(k.saved + ((size_t)(dst0 + jj) * H + head) * 2);
    };
    auto enter_dst = [&]() {   // destination j's statistics; those of j + 1 on their way
        dm = next.x;
        dzi = next.y > 0.f ? 1.f / next.y : 0.f;
        load_next(j + 1);
    };
    auto flush_dst = [&](int jj) {
        if (gl % LH == 0) {
            if (slot < 0) k.rec[(size_t)(dst0 + jj) * H + head] = make_float4(dm, dzi, sacc, 0.f);
            else k.spart[(size_t)slot * H + head] = sacc;
        }
        sacc = 0.f;
    };
    while (j < nd && st.dvs[j + 1] == st.dvs[j]) { flush_dst(j); ++j; }
    load_next(j);
    if (j < nd) enter_dst();
    if (ne > 0) {
        // ping-pong batches of (K row, V row); each segment's QP and dP rows
        // are read once, while the segment before it runs
        const float *qd = k.QD + (size_t)vs0 * (2 * D) + gl * 4;
        float4 qn = ld4(qd), pn = ld4(qd + D);
        float4 qs = zero4(), ps = zero4();
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
                    if (e == st.vptr[jv]) {   // first edge of segment jv
                        qs = qn; ps = pn;
                        if (jv + 1 < nv) {
                            qn = ld4(qd + (size_t)(jv + 1) * (2 * D));
                            pn = ld4(qd + (size_t)(jv + 1) * (2 * D) + D);
                        }
                    }
                    const float a = gsum<LH>(dot4(Xk[u], qs));
                    const float da = gsum<LH>(dot4(Xv[u], ps));
                    const float al = __expf(a - dm) * dzi;
                    sal = axpy4(sal, al, Xv[u]);
                    bac = axpy4(bac, al, Xk[u]);
                    aac = axpy4(aac, al * da, Xk[u]);
                    sacc += al * da;
                    if (e + 1 == st.vptr[jv + 1]) {
                        const int v0 = st.dvs[j], v1 = st.dvs[j + 1];
                        const size_t o = (size_t)st.vpos[jv] * D + gl * 4;
                        st4(k.Sal + o, sal);
                        if (slot < 0 && dqp_in_pass(v1 - v0, st.vptr[v1] - st.vptr[v0])) {
                            if (jv + 1 < v1) {
                                st.held[jv - v0][0][gl] = aac;
                                st.held[jv - v0][1][gl] = bac;
                            } else {
                                st4(k.dQP + o, axpy4(aac, -sacc, bac));
#pragma unroll 1
                                for (int h = 0; h < jv - v0; ++h)
                                    st4(k.dQP + (size_t)st.vpos[v0 + h] * D + gl * 4,
                                        axpy4(st.held[h][0][gl], -sacc, st.held[h][1][gl]));
                            }
                        } else {
                            st4(k.dQP + o, aac);
                            st4(k.Bac + o, bac);
                        }
                        sal = zero4(); aac = zero4(); bac = zero4();
                        ++jv;
                        if (jv == v1) {
                            flush_dst(j);
                            ++j;
                            while (j < nd && st.dvs[j + 1] == st.dvs[j]) { flush_dst(j); ++j; load_next(j); }
                            if (j < nd) enter_dst();
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
    while (j < nd) { flush_dst(j); ++j; }
}

// The record of destinations split over several items: their s from their slots
// in order.
__global__ __launch_bounds__(256) void hgt_bwd_merge_s_kernel(int64_t n_split, int heads,
                                                              const int32_t *split_dst,
                                                              const int32_t *split_slotptr,
                                                              const float *spart, const float *saved, float4 *rec)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n_split * heads) return;
    const int64_t i = idx / heads;
    const int hh = (int)(idx % heads);
    float s = 0.f;
    for (int sl = split_slotptr[i]; sl < split_slotptr[i + 1]; ++sl) s += spart[(size_t)sl * heads + hh];
    const size_t o = (size_t)split_dst[i] * heads + hh;
    const float2 mz = *reinterpret_cast<const float2 *>(saved + o * 2);
    rec[o] = make_float4(mz.x, mz.y > 0.f ? 1.f / mz.y : 0.f, s, 0.f);
}

// dQP = A - s_t B (A in dQP on entry) for the by-relation segment rows of the
// destinations that the destination-major pass left to this kernel: a group of
// D / 4 lanes per kDqpRows rows, head blocks of D / heads features.
constexpr int kDqpRows = 4;
__global__ __launch_bounds__(256) void hgt_bwd_dqp_kernel(int64_t V, int D, int heads, const int32_t *vsegdst_byrel,
                                                          const int32_t *dst_vsegptr, const int32_t *rowptr,
                                                          const float *B, const float4 *rec, float *dQP)
{
    const int g = D / 4, gl = (int)threadIdx.x % g;
    const int64_t row0 = ((int64_t)blockIdx.x * (256 / g) + threadIdx.x / g) * kDqpRows;
    if (row0 >= V) return;
    int v[kDqpRows];
    bool todo[kDqpRows];
#pragma unroll
    for (int i = 0; i < kDqpRows; ++i) v[i] = vsegdst_byrel[row0 + i < V ? row0 + i : V - 1];
#pragma unroll
    for (int i = 0; i < kDqpRows; ++i)
        todo[i] = row0 + i < V &&
                  !dqp_in_pass(dst_vsegptr[v[i] + 1] - dst_vsegptr[v[i]], rowptr[v[i] + 1] - rowptr[v[i]]);
#pragma unroll
    for (int i = 0; i < kDqpRows; ++i) {
        if (!todo[i]) continue;
        const size_t o = (size_t)(row0 + i) * D + gl * 4;
        st4(dQP + o, axpy4(ld4(dQP + o), -rec[(size_t)v[i] * heads + (gl * 4) / (D / heads)].z, ld4(B + o)));
    }
}

// ---------------------------------------------------------------- source-major pass
struct SStageH {
    int ev[kE];          // virtual segment (QP | dP row) of each out-edge
    int et[kE];          // its destination
    int enode[kE];       // item-local source of each out-edge
    int optr[kDst + 1];  // item-local first out-edge of each source
};

struct SKArgs {
    int64_t n_items;
    const Item *items;
    const int32_t *out_ptr;
    const int32_t *out_vs, *out_dst;   // per out-edge: vseg (QP | dP row) and destination, read in order
    const float *KV, *QD;
    const float4 *rec;   // [N, H] (max, 1 / sum, s, 0) per destination and head
    float *dKV;          // [N, ldk] dK | dV first in each row: of split sources zero on entry,
                         // of every other source written here
    int ldk;
};

template <int D, int H>
__global__ __launch_bounds__(256) void hgt_bwd_src_kernel(SKArgs k)
{
    constexpr int G = D / 4, GPB = 256 / G;
    constexpr int DKH = D / H, LH = DKH / 4;
    __shared__ SStageH stage[GPB];
    const int gl = threadIdx.x % G, gi = threadIdx.x / G;
    SStageH &st = stage[gi];
    const int64_t item = (int64_t)blockIdx.x * GPB + gi;
    const bool valid = item < k.n_items;
    int n0 = 0, nn = 0, q0 = 0, nq = 0;
    bool split = false;   // a piece of a source whose out-edges span several items
    if (valid) {
        const Item x = k.items[item];
        n0 = x.dst0; nn = x.dst1 - x.dst0; q0 = x.vs0; nq = x.vs1 - x.vs0;
        split = nn == 1 && k.out_ptr[n0 + 1] - k.out_ptr[n0] > nq;
        for (int e = gl; e < nq; e += G) {
            st.ev[e] = k.out_vs[q0 + e];
            st.et[e] = k.out_dst[q0 + e];
        }
        auto opos = [&](int jj) {
            const int q = k.out_ptr[n0 + jj];
            return (q < q0 ? q0 : (q > q0 + nq ? q0 + nq : q)) - q0;
        };
        for (int j = gl; j < nn; j += G) {
            const int a = opos(j), b = opos(j + 1);
            st.optr[j] = a;
            for (int e = a; e < b; ++e) st.enode[e] = j;
        }
        if (gl == 0) st.optr[nn] = nq;
    }
    __syncthreads();
    if (!valid) return;
    // sources of a bundle without out-edges get zero rows
    for (int jj = 0; jj < nn; ++jj)
        if (st.optr[jj + 1] == st.optr[jj]) {
            float *p = k.dKV + (size_t)(n0 + jj) * k.ldk + gl * 4;
            st4(p, zero4());
            st4(p + D, zero4());
        }
    if (nq == 0) return;
    const int head = gl / LH;
    int j = 0;
    while (st.optr[j + 1] == st.optr[j]) ++j;   // first source with out-edges
    float4 dk = zero4(), dv = zero4();
    // ping-pong batches of (K row, V row of the source, QP and dP rows of the
    // segment, the destination's max, sum and s for this head)
    float4 Ak[kU], Av[kU], Aq[kU], Ap[kU], Bk[kU], Bv[kU], Bq[kU], Bp[kU];
    float4 Am[kU], Bm[kU];
    auto load = [&](float4 (&Xk)[kU], float4 (&Xv)[kU], float4 (&Xq)[kU], float4 (&Xp)[kU],
                    float4 (&Xm)[kU], int b0) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = b0 + u < nq ? b0 + u : nq - 1;
            const size_t row = (size_t)(n0 + st.enode[e]) * (2 * D);
            const size_t vrow = (size_t)st.ev[e] * (2 * D);
            const size_t th = (size_t)st.et[e] * H + head;
            Xk[u] = ld4(k.KV + row + gl * 4);
            Xv[u] = ld4(k.KV + row + D + gl * 4);
            Xq[u] = ld4(k.QD + vrow + gl * 4);
            Xp[u] = ld4(k.QD + vrow + D + gl * 4);
            Xm[u] = k.rec[th];
        }
    };
    auto consume = [&](const float4 (&Xk)[kU], const float4 (&Xv)[kU], const float4 (&Xq)[kU],
                       const float4 (&Xp)[kU], const float4 (&Xm)[kU], int b0) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = b0 + u;
            if (e < nq) {
                const float a = gsum<LH>(dot4(Xk[u], Xq[u]));
                const float dal = gsum<LH>(dot4(Xv[u], Xp[u]));
                const float al = __expf(a - Xm[u].x) * Xm[u].y;
                dk = axpy4(dk, al * (dal - Xm[u].z), Xq[u]);
                dv = axpy4(dv, al, Xp[u]);
                if (e + 1 == st.optr[j + 1]) {   // the source's last out-edge in this item
                    float *p = k.dKV + (size_t)(n0 + j) * k.ldk + gl * 4;
                    if (split) {
                        atomic_add4(p, dk);
                        atomic_add4(p + D, dv);
                    } else {
                        st4(p, dk);
                        st4(p + D, dv);
                    }
                    dk = zero4(); dv = zero4();
                    ++j;
                    while (j < nn && st.optr[j + 1] == st.optr[j]) ++j;
                }
            }
        }
    };
    load(Ak, Av, Aq, Ap, Am, 0);
    __builtin_amdgcn_sched_barrier(0);
    for (int eb = 0; eb < nq; eb += 2 * kU) {
        load(Bk, Bv, Bq, Bp, Bm, eb + kU);
        __builtin_amdgcn_sched_barrier(0);
        consume(Ak, Av, Aq, Ap, Am, eb);
        load(Ak, Av, Aq, Ap, Am, eb + 2 * kU);
        __builtin_amdgcn_sched_barrier(0);
        consume(Bk, Bv, Bq, Bp, Bm, eb + kU);
    }
}

// Per relation: dWatt, dWmsg from the head blocks of OT = sum dQP^T Q and
// M2 = sum Salpha^T dagg, and dmu = scale * <OT head blocks, Watt> (fixed order).
__global__ __launch_bounds__(256) void hgt_bwd_rel_kernel(const float *OT, const float *M2, const float *Watt,
                                                          const float *mu, float scale, int D, int heads,
                                                          float *dWatt, float *dWmsg, float *dmu)
{
    __shared__ float red[256];
    const int r = blockIdx.x, tid = threadIdx.x;
    const int dk = D / heads, n = heads * dk * dk;
    float part = 0.f;
    for (int idx = tid; idx < n; idx += 256) {
        const int i = idx / (dk * dk), p = idx / dk % dk, q = idx % dk;
        const size_t src = ((size_t)r * D + i * dk + p) * D + i * dk + q;
        const float ot = OT[src];
        dWatt[(size_t)r * n + idx] = mu[r] * scale * ot;
        dWmsg[(size_t)r * n + idx] = M2[src];
        part += ot * Watt[(size_t)r * n + idx];
    }
    red[tid] = part;
    __syncthreads();
    if (tid == 0) {
        float s = 0.f;
        for (int t = 0; t < 256; ++t) s += red[t];
        dmu[r] = scale * s;
    }
}

// ---------------------------------------------------------------- typed relations
// When all destinations of a relation share one node type t(r), Q = h Wq[t] and
// dagg = G Wa[t]^T enter the per-segment terms only through products with
// per-relation weights, so neither is formed:
//   QP_vs = h_t Wf[r],   Wf[r] = Wq[t(r)] Wqp[r]       (as in the forward)
//   dP_vs = G_t Wg[r],   Wg[r] = Wa[t(r)]^T Wmsg[r]^T  (without the output linear: Wmsg[r]^T)
// and every weight gradient on the destination side follows from two outer
// products per relation, P1[r] = sum_vs dQP_vs^T h_t and P2[r] = sum_vs
// Salpha_vs^T G_t, by products of d x d matrices:
//   sum_vs dQP^T Q = P1 Wq[t],      sum_vs Salpha^T dagg = P2 Wa[t]^T
//   dWq[t] = sum_{r of t} P1[r]^T Wqp[r]^T,   dWa[t] = sum_{r of t} Wmsg[r]^T P2[r]
// and dh's query part is sum_vs dQP_vs Wf[r]^T.  Against the general path this
// drops the Q and dagg projections, the rebuilt aggregate (a GEMM over the
// segments and a reduction), dQ and two outer products over all nodes.

// Every per-relation and per-type weight of the typed path in one launch: blocks
// [0, nr) Wf, [nr, 2 nr) Wg (Wa NULL: the block-diagonal Wmsg^T), then Wc[t][n][j D +
// k] = (Wk, Wv)[j][t][n][k], for dh = [dK | dV] Wc^T.
__global__ __launch_bounds__(256) void hgt_bwd_weights_kernel(const float *Wk, const float *Wv, const float *Wq,
                                                              const float *Wa, const float *Watt, const float *Wmsg,
                                                              const float *mu, const int32_t *rel_dsttype, float scale,
                                                              int R, int T, int D, int heads, int nr, float *Wf,
                                                              float *Wg, float *Wc)
{
    const int b = (int)blockIdx.x, part = b < nr ? 0 : (b < 2 * nr ? 1 : 2);
    const int64_t idx = (int64_t)(b - part * nr) * 256 + threadIdx.x;
    if (part < 2) {
        if (idx >= (int64_t)R * D * D) return;
        if (part == 0) Wf[idx] = hgt_qp_fold_entry(idx, Wq, Watt, mu, scale, rel_dsttype, D, heads);
        else if (Wa) Wg[idx] = hgt_msg_fold_entry(idx, Wa, Wmsg, rel_dsttype, D, heads);
        else Wg[idx] = hgt_msgT_entry(idx, Wmsg, D, heads);
    } else if (idx < (int64_t)T * D * 2 * D) {
        const int64_t row = idx / (2 * D);
        const int c = (int)(idx % (2 * D));
        Wc[idx] = (c < D ? Wk : Wv)[row * D + (c < D ? c : c - D)];
    }
}

// Per relation (blockIdx.x) and 256 entries of its head blocks (blockIdx.y):
// dWatt = c_r (P1 Wq[t])[blocks], dWmsg = (P2 Wa[t]^T)[blocks] (Wa NULL: P2's
// blocks), and the block's share of <P1 Wq[t], Watt> for dmu.  A relation without
// segments (rel_ptr) has zero products whatever the weights of the node type that
// stands in for its own hold.
__global__ __launch_bounds__(256) void hgt_bwd_rel_typed_kernel(const float *P1, const float *P2, const float *Wq,
                                                                const float *Wa, const float *Watt, const float *mu,
                                                                const int32_t *rel_dsttype, const int32_t *rel_ptr,
                                                                float scale, int D, int heads, float *dWatt,
                                                                float *dWmsg, float *mupart)
{
    __shared__ float red[4];
    const int r = blockIdx.x, tid = threadIdx.x;
    const int dk = D / heads, n = heads * dk * dk;
    const int idx = blockIdx.y * 256 + tid;
    float part = 0.f;
    if (idx < n) {
        const int i = idx / (dk * dk), p = idx / dk % dk, q = idx % dk;
        const size_t t = (size_t)rel_dsttype[r] * D;
        const float *p1 = P1 + ((size_t)r * D + i * dk + p) * D;
        const float *p2 = P2 + ((size_t)r * D + i * dk + p) * D;
        const float *wq = Wq + t * D + i * dk + q;
        float ot = 0.f, m2 = 0.f;
        if (rel_ptr[r + 1] > rel_ptr[r]) {
#pragma unroll 16
            for (int k = 0; k < D; ++k) ot = fmaf(p1[k], wq[(size_t)k * D], ot);
            if (Wa) {
                const float *wa = Wa + (t + i * dk + q) * D;
#pragma unroll 16
                for (int k = 0; k < D; ++k) m2 = fmaf(p2[k], wa[k], m2);
            } else {
                m2 = p2[i * dk + q];
            }
        }
        dWatt[(size_t)r * n + idx] = mu[r] * scale * ot;
        dWmsg[(size_t)r * n + idx] = m2;
        part = ot * Watt[(size_t)r * n + idx];
    }
    part = gsum<32>(part);
    part += __shfl_xor(part, 32);
    if ((tid & 63) == 0) red[tid >> 6] = part;
    __syncthreads();
    if (tid == 0) mupart[(size_t)r * gridDim.y + blockIdx.y] = red[0] + red[1] + red[2] + red[3];
}

// Blocks [0, nb): 64 entries of dWq[t], nb = T D^2 / 64; then, with Wmsg, nb
// blocks for dWa[t]; the last ones dmu.  Sixteen slices of threads take every
// sixteenth relation, their sums are added in slice order.  Relations without
// segments are left out: their weights have no part in the layer and may hold
// anything.
__global__ __launch_bounds__(1024) void hgt_bwd_type_kernel(const float *P1, const float *P2, const float *Watt,
                                                            const float *Wmsg, const float *mu,
                                                            const int32_t *rel_dsttype, const int32_t *rel_ptr,
                                                            float scale, int R, int D, int heads, int nb, int want_wa,
                                                            const float *mupart, int nmu, float *dWq, float *dWa,
                                                            float *dmu)
{
    __shared__ float red[16][64];
    const int tid = threadIdx.x, li = tid & 63, sl = tid >> 6;
    int b = (int)blockIdx.x;
    const int which = b < nb ? 0 : (want_wa && b < 2 * nb ? 1 : 2);
    if (which == 2) {   // dmu[r] = scale * the ordered sum of its shares
        const int r = (b - (want_wa ? 2 : 1) * nb) * 1024 + tid;
        if (r < R) {
            float s = 0.f;
            for (int j = 0; j < nmu; ++j) s += mupart[(size_t)r * nmu + j];
            dmu[r] = scale * s;
        }
        return;
    }
    if (which == 1) b -= nb;
    const int dk = D / heads;
    const int64_t idx = (int64_t)b * 64 + li;   // (t, row, col)
    const int t = (int)(idx / (D * D)), row = (int)(idx / D % D), col = (int)(idx % D);
    float acc = 0.f;
    for (int r = sl; r < R; r += 16) {
        if (rel_dsttype[r] != t || rel_ptr[r + 1] == rel_ptr[r]) continue;
        if (which == 0) {   // dWq[j][i dk + q] += c_r sum_p P1[i dk + p][j] Watt[i][p][q]
            const int i = col / dk;
            const float *p1 = P1 + ((size_t)r * D + i * dk) * D + row;
            const float *wa = Watt + ((size_t)r * heads + i) * dk * dk + (col - i * dk);
            float x = 0.f;
#pragma unroll 8
            for (int p = 0; p < dk; ++p) x = fmaf(p1[(size_t)p * D], wa[(size_t)p * dk], x);
            acc = fmaf(mu[r] * scale, x, acc);
        } else {            // dWa[i dk + b][g] += sum_a Wmsg[i][a][b] P2[i dk + a][g]
            const int i = row / dk;
            const float *p2 = P2 + ((size_t)r * D + i * dk) * D + col;
            const float *wm = Wmsg + ((size_t)r * heads + i) * dk * dk + (row - i * dk);
#pragma unroll 8
            for (int a = 0; a < dk; ++a) acc = fmaf(p2[(size_t)a * D], wm[(size_t)a * dk], acc);
        }
    }
    red[sl][li] = acc;
    __syncthreads();
    if (sl == 0) {
        float s = red[0][li];
        for (int j = 1; j < 16; ++j) s += red[j][li];
        (which == 0 ? dWq : dWa)[idx] = s;
    }
}

// zero the first w floats (w a multiple of 4) of the rows (stride ld) listed in rows
__global__ __launch_bounds__(256) void zero_rows_kernel(const int32_t *rows, int64_t n, int w, int ld, float *p)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, q = w / 4;
    if (i < n * q) st4(p + (size_t)rows[i / q] * ld + (i % q) * 4, zero4());
}

// Wc[t][n][j D + k] = W_j[t][n][k] for (W_0, W_1, W_2) = (Wk, Wv, Wq): the three
// transposed weights side by side, so that dh = [dK | dV | dQ] Wc^T is one GEMM.
__global__ __launch_bounds__(256) void hgt_cat_weights_kernel(const float *Wk, const float *Wv, const float *Wq,
                                                              int T, int D, float *Wc)
{
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)T * D * 3 * D) return;
    const int64_t row = idx / (3 * D);
    const int c = (int)(idx % (3 * D)), j = c / D, k = c % D;
    const float *W = j == 0 ? Wk : (j == 1 ? Wv : Wq);
    Wc[idx] = W[row * D + k];
}

inline unsigned blocks_for(int64_t n, int per_block) { return (unsigned)((n + per_block - 1) / per_block); }
inline size_t pad256(size_t b) { return (b + 255) & ~size_t(255); }

struct HgtBwdWs {
    float *KV, *Q, *Wqp, *QD, *agg, *partial, *saved, *dagg, *Wmt, *Sal, *Bac,
        *spart, *dQP, *Tq, *dKV, *chunks, *OT, *M2, *rec, *Wc, *Wf, *Wg, *mupart, *stat, *chunks2;
};

// the forward forms its segment queries from Q inside the traversal
bool forward_queries_in_kernel(const rgnn_graph *g, int D, int H)
{
    return D == 128 && hgt_fused_query_fits(g->R, D, H);
}
// Whether the node-type weights are folded into the per-relation ones (typed
// relations only).  The folded weights and the weight gradients that follow from
// P1 and P2 are products of about R D^2 dk terms each on the vector units, against
// the general path's passes over the nodes (N D^2 on the matrix cores and N D
// values written and read several times), so the line lies at R dk against N, with
// the constant that the general path's seven more launches are worth.  Backward of
// one-type graphs with 6.5 N edges, us, folded / general:
//   N = 3 000    R dk = 2 400 (d = 64, dk = 16)  146 / 163,   4 800 (128, 32)   393 / 343
//   N = 12 000   R dk = 5 120 (128, 128)         502 / 533,   8 560 (128, 16)   852 / 754
//   N = 50 000   R dk = 9 600 (64, 64)           598 / 642,   17 120 (128, 32) 1960 / 1775
//   N = 200 000  R dk = 34 240 (64, 64)         2166 / 2209,  68 480 (128, 128) 6619 / 5484
bool fold_types(const rgnn_graph *g, int D, int H)
{
    return g->rel_dst_typed && (int64_t)g->R * (D / H) <= 4000 + g->N * 3 / 16;
}
// 256-entry blocks of a relation's head blocks
constexpr int rel_blocks(int D, int H) { return (H * (D / H) * (D / H) + 255) / 256; }

size_t hgt_bwd_layout(const rgnn_graph *g, int D, int H, void *base, HgtBwdWs *w)
{
    char *b = (char *)base;
    size_t off = 0;
    auto take = [&](size_t n) {
        float *p = b ? (float *)(b + off) : nullptr;
        off += pad256(std::max<size_t>(n, 1) * sizeof(float));
        return p;
    };
    const size_t N = (size_t)g->N, V = (size_t)g->V, R = (size_t)g->R;
    const size_t slots = (size_t)g->n_slots;
    const size_t nchunks = (size_t)std::max<int64_t>(std::max(g->n_tiles_outer, g->n_tiles_types_outer), 1);
    HgtBwdWs x{};
    const bool typed = fold_types(g, D, H);   // as hgt_backward_d
    x.KV = take(N * 2 * D); x.Q = take(typed && !forward_queries_in_kernel(g, D, H) ? 0 : N * D);
    x.Wqp = take(typed && !forward_queries_in_kernel(g, D, H) ? 0 : R * D * D); x.QD = take(V * 2 * D);
    x.agg = take(N * D); x.partial = take(slots * (2 * H + D)); x.saved = take(N * H * 2);
    x.dagg = take(typed ? 0 : N * D); x.Wmt = take(R * D * D);
    x.Sal = take(V * D); x.Bac = take(V * D);
    x.spart = take(slots * H);
    x.dQP = take(V * D); x.Tq = take(V * D);
    x.dKV = take(N * (typed ? 2 : 3) * D);   // dK | dV (| dQ) side by side per node
    x.Wc = take(D <= 64 ? (size_t)g->T * D * 3 * D : 0);
    x.chunks = take(nchunks * D * D); x.chunks2 = take(nchunks * D * D); x.OT = take(R * D * D); x.M2 = take(R * D * D);
    x.rec = take(N * H * 4);
    x.Wf = take(R * D * D); x.Wg = take(typed ? R * D * D : 0);
    x.mupart = take(R * rel_blocks(D, H));
    x.stat = take(hgt_seg_values(g->R, D, H) ? V * H * 2 : 0);   // traversal recomputed, wide heads
    if (w) *w = x;
    return off;
}

// Y = X W[type]^T over the nodes grouped by type (typed GEMM, B = W^T).
rgnn_status node_gemm_t(const rgnn_graph *g, int D, const float *X, int64_t ldx, const float *W, float *Y,
                        const float *residual, int accumulate, hipStream_t s)
{
    GemmArgs ga;
    ga.split_bf16 = 1;
    ga.X = X; ga.ldx = ldx; ga.gather = g->dev.ntype_perm; ga.scatter = g->dev.ntype_perm;
    ga.W[0] = W; ga.trans_b = 1; ga.K = D; ga.Nc = D;
    ga.tiles = g->gemm_tiles(kRowsNodes);
    ga.Y = Y; ga.ldy = D;
    if (residual) { ga.ep.residual = residual; ga.ep.ld_res = D; }
    ga.ep.accumulate = accumulate;
    return launch_typed_gemm(ga, s);
}

// dW[type] = sum over the nodes n of the type of X[n]^T Y[n].
rgnn_status type_outer(const rgnn_graph *g, int D, const float *X, int ldx, const float *Y, int ldy, float *chunks,
                       float *dW, hipStream_t s)
{
    rgnn_status st = launch_outer_chunks(g->dev.tiles_types_outer, g->n_tiles_types_outer, g->dev.ntype_perm, 1,
                                         X, ldx, Y, ldy, chunks, D, s);
    if (st != RGNN_OK) return st;
    return launch_chunk_sum(chunks, g->dev.types_chunkptr, g->T, dW, D, s);
}

template <int D>
rgnn_status hgt_backward_d(const rgnn_graph *g, const float *h, const float *Wk, const float *Wq,
                           const float *Wv, const float *Wa, const float *Watt, const float *Wmsg,
                           const float *mu, int H, float att_scale, int flags, const float *Gm,
                           const float *saved, float *dh, float *dWk, float *dWq, float *dWv, float *dWa,
                           float *dWatt, float *dWmsg, float *dmu, void *ws, hipStream_t s)
{
    constexpr int G = D / 4, GPB = 256 / G;
    const bool a_linear = (flags & RGNN_FLAG_A_LINEAR) != 0;
    const bool typed = fold_types(g, D, H);
    HgtBwdWs w;
    hgt_bwd_layout(g, D, H, ws, &w);
    rgnn_status st;
    hipError_t e;
    // ---- forward recomputation: K | V (| Q), the segment queries and, without the
    //      forward's statistics, the traversal that yields them and agg
    const float *stats = saved ? saved : w.saved;
    // the segment queries exactly as the forward forms them (with the query
    // projection folded into the per-relation weight when the relations are
    // typed, whether or not the rest is), so that the recomputed scores match its
    // statistics
    const bool fold_q = g->rel_dst_typed && !forward_queries_in_kernel(g, D, H);
    const bool need_q = !fold_q || !typed;
    {
        GemmArgs ga;
        ga.split_bf16 = 1;
        ga.X = h; ga.ldx = D; ga.gather = g->dev.ntype_perm; ga.scatter = g->dev.ntype_perm;
        ga.K = D;
        ga.tiles = g->gemm_tiles(kRowsNodes);
        if (D == 64 && !need_q) {   // K | V in one GEMM
            ga.W[0] = Wk; ga.W[1] = Wv; ga.nparts = 2;
            ga.Nc = 2 * D;
            ga.Y = w.KV; ga.ldy = 2 * D;
            if ((st = launch_typed_gemm(ga, s)) != RGNN_OK) return st;
        } else if (D == 64) {   // K | V | Q in one GEMM
            ga.W[0] = Wk; ga.W[1] = Wv; ga.W[2] = Wq; ga.nparts = 3;
            ga.Nc = 3 * D;
            ga.Y = w.KV; ga.ldy = 2 * D;
            ga.ep.Y2 = w.Q; ga.ep.ldy2 = D; ga.ep.split = 2 * D;
            if ((st = launch_typed_gemm(ga, s)) != RGNN_OK) return st;
        } else {
            ga.Nc = D;
            const float *Wp[3] = {Wk, Wv, Wq};
            float *Yp[3] = {w.KV, w.KV + D, w.Q};
            const int64_t ld[3] = {2 * D, 2 * D, D};
            for (int p = 0; p < (need_q ? 3 : 2); ++p) {
                ga.W[0] = Wp[p]; ga.Y = Yp[p]; ga.ldy = ld[p];
                if ((st = launch_typed_gemm(ga, s)) != RGNN_OK) return st;
            }
        }
    }
    if (need_q && (st = launch_hgt_qp_weights(Watt, mu, att_scale, g->R, D, H, w.Wqp, s)) != RGNN_OK) return st;
    if (fold_q && !typed &&
        (st = launch_hgt_qp_fold(Wq, Watt, mu, att_scale, g->dev.rel_dsttype, g->R, D, H, w.Wf, s)) != RGNN_OK)
        return st;
    const bool fold_a = typed && a_linear;
    if (typed) {
        const unsigned nr = blocks_for((int64_t)g->R * D * D, 256);
        {
            LaunchScope ls("hgt_bwd_weights", s);
            const unsigned nc = D <= 64 ? blocks_for((int64_t)g->T * D * 2 * D, 256) : 0;   // Wc's only readers
            hipLaunchKernelGGL(hgt_bwd_weights_kernel, dim3(2 * nr + nc), dim3(256), 0, s, Wk, Wv, Wq,
                               fold_a ? Wa : nullptr, Watt, Wmsg, mu, g->dev.rel_dsttype, att_scale, g->R, g->T, D, H,
                               (int)nr, w.Wf, w.Wg, w.Wc);
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_bwd_weights launch");
    }
    {
        GemmArgs gq;
        gq.split_bf16 = 1;
        gq.X = fold_q ? h : w.Q; gq.ldx = D; gq.gather = g->dev.vsegdst_byrel; gq.scatter = g->dev.vseg_byrel;
        gq.W[0] = fold_q ? w.Wf : w.Wqp; gq.K = D; gq.Nc = D;
        gq.tiles = g->gemm_tiles(kRowsVsegsDst);
        gq.Y = w.QD; gq.ldy = 2 * D; gq.ep.diag_blocks = fold_q ? 1 : H;
        if ((st = launch_typed_gemm(gq, s)) != RGNN_OK) return st;
    }
    if (!saved) {
        HgtArgs ha;
        ha.g = g; ha.KV = w.KV; ha.QP = w.QD; ha.ldq = 2 * D; ha.Wmsg = Wmsg;
        ha.heads = H; ha.d = D; ha.agg = w.agg; ha.partial = w.partial; ha.saved = w.saved;
        ha.Sv = w.Sal; ha.stat = w.stat; ha.Wt = w.Wmt; ha.T = w.Tq;
        if ((st = launch_hgt_traverse(ha, s)) != RGNN_OK) return st;
    }
    // ---- output linear (general path): dagg = G Wa^T, dWa = sum agg^T G per node
    //      type (with the forward's statistics agg is rebuilt after the destination pass)
    const float *dagg = Gm;
    if (a_linear && !typed) {
        if ((st = node_gemm_t(g, D, Gm, D, Wa, w.dagg, nullptr, 0, s)) != RGNN_OK) return st;
        dagg = w.dagg;
        if (dWa && !saved && (st = type_outer(g, D, w.agg, D, Gm, D, w.chunks, dWa, s)) != RGNN_OK) return st;
    }
    // ---- dP = dagg_t Wmsg[r]^T per segment (vseg order); typed: G_t Wg[r]
    if (g->V > 0) {
        if (!typed && (st = launch_hgt_msgT_weights(Wmsg, g->R, D, H, w.Wmt, s)) != RGNN_OK) return st;
        GemmArgs gp;
        gp.split_bf16 = 1;
        gp.X = dagg; gp.ldx = D; gp.gather = g->dev.vsegdst_byrel; gp.scatter = g->dev.vseg_byrel;
        gp.W[0] = typed ? w.Wg : w.Wmt; gp.K = D; gp.Nc = D;
        gp.tiles = g->gemm_tiles(kRowsVsegsDst);
        gp.Y = w.QD + D; gp.ldy = 2 * D; gp.ep.diag_blocks = fold_a ? 1 : H;
        if ((st = launch_typed_gemm(gp, s)) != RGNN_OK) return st;
    }
    // ---- destination-major pass: Salpha, A, B per segment; s per destination
    if (g->n_items > 0) {
        DKArgs k{};
        k.n_items = g->n_items; k.items = g->dev.items; k.item_slot = g->dev.item_slot;
        k.dst_vsegptr = g->dev.dst_vsegptr; k.vseg_ptr = g->dev.vseg_ptr; k.in_src = g->dev.in_src;
        k.vseg_pos = g->dev.vseg_pos;
        k.KV = w.KV; k.QD = w.QD; k.saved = stats;
        k.Sal = w.Sal; k.dQP = w.dQP; k.Bac = w.Bac; k.spart = w.spart; k.rec = reinterpret_cast<float4 *>(w.rec);
        const unsigned nb = blocks_for(g->n_items, GPB);
        {
            LaunchScope ls("hgt_bwd_dst", s);
            if (H == 1) hipLaunchKernelGGL((hgt_bwd_dst_kernel<D, 1>), dim3(nb), dim3(256), 0, s, k);
            else if (H == 2) hipLaunchKernelGGL((hgt_bwd_dst_kernel<D, 2>), dim3(nb), dim3(256), 0, s, k);
            else if constexpr (D >= 64) {
                if (H == 4) hipLaunchKernelGGL((hgt_bwd_dst_kernel<D, 4>), dim3(nb), dim3(256), 0, s, k);
                else if constexpr (D >= 128) hipLaunchKernelGGL((hgt_bwd_dst_kernel<D, 8>), dim3(nb), dim3(256), 0, s, k);
            }
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_bwd_dst launch");
    }
    if (g->n_split > 0) {
        {
            LaunchScope ls("hgt_bwd_merge_s", s);
            hipLaunchKernelGGL(hgt_bwd_merge_s_kernel, dim3(blocks_for(g->n_split * H, 256)), dim3(256), 0, s,
                               g->n_split, H, g->dev.split_dst, g->dev.split_slotptr, w.spart, stats,
                               reinterpret_cast<float4 *>(w.rec));
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_bwd_merge_s launch");
    }
    // ---- agg_t = sum over t's segments of Salpha_vs Wmsg[r] (the messages are
    //      linear in V_s, so the alpha-weighted V sums of the destination pass
    //      give the forward's aggregate), then dWa = sum agg^T G per node type
    if (a_linear && dWa && saved && !typed) {
        if (g->V > 0) {
            GemmArgs gm;
            gm.split_bf16 = 1;
            gm.X = w.Sal; gm.ldx = D; gm.W[0] = w.Wmt; gm.trans_b = 1; gm.K = D; gm.Nc = D;
            gm.tiles = g->gemm_tiles(kRowsVsegs);
            gm.Y = w.Tq; gm.ldy = D; gm.scatter = g->dev.vseg_byrel; gm.ep.diag_blocks = H;
            if ((st = launch_typed_gemm(gm, s)) != RGNN_OK) return st;
        }
        if ((st = launch_vseg_reduce(g, w.Tq, nullptr, D, w.agg, 0, 0, s)) != RGNN_OK) return st;
        if ((st = type_outer(g, D, w.agg, D, Gm, D, w.chunks, dWa, s)) != RGNN_OK) return st;
    }
    // ---- dQP and its product with the query weights (general: dQ_t's terms dQP
    //      Wqp[r]^T; typed: dh_t's terms dQP Wf[r]^T), in vseg order
    if (g->V > 0) {
        {
            LaunchScope ls("hgt_bwd_dqp", s);
            hipLaunchKernelGGL(hgt_bwd_dqp_kernel, dim3(blocks_for(g->V, GPB * kDqpRows)), dim3(256), 0, s,
                               g->V, D, H, g->dev.vsegdst_byrel, g->dev.dst_vsegptr, g->dev.rowptr, w.Bac,
                               reinterpret_cast<const float4 *>(w.rec), w.dQP);
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_bwd_dqp launch");
        GemmArgs gt;
        gt.split_bf16 = 1;
        gt.X = w.dQP; gt.ldx = D; gt.W[0] = typed ? w.Wf : w.Wqp; gt.trans_b = 1; gt.K = D; gt.Nc = D;
        gt.tiles = g->gemm_tiles(kRowsVsegs);
        gt.Y = w.Tq; gt.ldy = D; gt.scatter = g->dev.vseg_byrel; gt.ep.diag_blocks = typed ? 1 : H;
        if ((st = launch_typed_gemm(gt, s)) != RGNN_OK) return st;
    }
    const int ldk = typed ? 2 * D : 3 * D;
    if (!typed && (st = launch_vseg_reduce(g, w.Tq, nullptr, D, w.dKV + 2 * D, 0, 0, s, ldk)) != RGNN_OK) return st;
    // ---- per-relation outer products (typed: with h and G, else with Q and
    //      dagg) and the weight gradients that follow from them
    if (g->V > 0 && (st = launch_outer_chunks(g->dev.tiles_outer, g->n_tiles_outer, g->dev.vsegdst_byrel, 0, w.dQP, D,
                                              typed ? h : w.Q, D, w.chunks, D, s, w.Sal, dagg, w.chunks2)) != RGNN_OK)
        return st;
    if ((st = launch_chunk_sum(w.chunks, g->dev.rel_chunkptr, g->R, w.OT, D, s, w.chunks2, w.M2)) != RGNN_OK) return st;
    if (g->R > 0 && typed) {
        const int nrb = rel_blocks(D, H), nb = g->T * D * D / 64, wa = a_linear && dWa ? 1 : 0;
        {
            LaunchScope ls("hgt_bwd_rel", s);
            hipLaunchKernelGGL(hgt_bwd_rel_typed_kernel, dim3((unsigned)g->R, (unsigned)nrb), dim3(256), 0, s, w.OT,
                               w.M2, Wq, a_linear ? Wa : nullptr, Watt, mu, g->dev.rel_dsttype, g->dev.rel_vsegptr,
                               att_scale, D, H, dWatt, dWmsg, w.mupart);
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_bwd_rel launch");
        {
            LaunchScope ls("hgt_bwd_type", s);
            hipLaunchKernelGGL(hgt_bwd_type_kernel, dim3((unsigned)((1 + wa) * nb) + blocks_for(g->R, 1024)),
                               dim3(1024), 0, s, w.OT, w.M2, Watt, Wmsg, mu, g->dev.rel_dsttype, g->dev.rel_vsegptr,
                               att_scale, g->R, D, H, nb, wa, w.mupart, nrb, dWq, dWa, dmu);
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_bwd_type launch");
    } else if (g->R > 0) {
        {
            LaunchScope ls("hgt_bwd_rel", s);
            hipLaunchKernelGGL(hgt_bwd_rel_kernel, dim3((unsigned)g->R), dim3(256), 0, s, w.OT, w.M2, Watt, mu,
                               att_scale, D, H, dWatt, dWmsg, dmu);
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_bwd_rel launch");
    }
    // ---- source-major pass: dK | dV per source (the rows of sources split over
    //      several items are summed with atomics and start from zero)
    if (g->n_osplit > 0) {
        {
            LaunchScope ls("zero", s);
            hipLaunchKernelGGL(zero_rows_kernel, dim3(blocks_for(g->n_osplit * (2 * D / 4), 256)), dim3(256), 0, s,
                               g->dev.osplit, g->n_osplit, 2 * D, ldk, w.dKV);
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "zero launch");
    }
    if (g->n_oitems > 0) {
        SKArgs k{};
        k.n_items = g->n_oitems; k.items = g->dev.oitems; k.out_ptr = g->dev.out_ptr;
        k.out_vs = g->dev.out_vs; k.out_dst = g->dev.out_dst;
        k.KV = w.KV; k.QD = w.QD; k.rec = reinterpret_cast<const float4 *>(w.rec); k.dKV = w.dKV; k.ldk = ldk;
        const unsigned nb = blocks_for(g->n_oitems, GPB);
        {
            LaunchScope ls("hgt_bwd_src", s);
            if (H == 1) hipLaunchKernelGGL((hgt_bwd_src_kernel<D, 1>), dim3(nb), dim3(256), 0, s, k);
            else if (H == 2) hipLaunchKernelGGL((hgt_bwd_src_kernel<D, 2>), dim3(nb), dim3(256), 0, s, k);
            else if constexpr (D >= 64) {
                if (H == 4) hipLaunchKernelGGL((hgt_bwd_src_kernel<D, 4>), dim3(nb), dim3(256), 0, s, k);
                else if constexpr (D >= 128) hipLaunchKernelGGL((hgt_bwd_src_kernel<D, 8>), dim3(nb), dim3(256), 0, s, k);
            }
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "hgt_bwd_src launch");
    }
    // ---- node-level linears: dh and the per-type weight gradients
    const float *res = (flags & RGNN_FLAG_RESIDUAL) ? Gm : nullptr;
    if constexpr (D <= 64) {   // dh = [dK | dV (| dQ)] [Wk | Wv (| Wq)]^T in one GEMM
        const int np = typed ? 2 : 3;
        if (g->T > 0 && !typed) {
            const int64_t n = (int64_t)g->T * D * 3 * D;
            LaunchScope ls("hgt_cat_weights", s);
            hipLaunchKernelGGL(hgt_cat_weights_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, Wk, Wv, Wq, g->T, D,
                               w.Wc);
        }
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "cat weights launch");
        GemmArgs ga;
        ga.split_bf16 = 1;
        ga.X = w.dKV; ga.ldx = ldk; ga.gather = g->dev.ntype_perm; ga.scatter = g->dev.ntype_perm;
        ga.W[0] = w.Wc; ga.trans_b = 1; ga.K = np * D; ga.Nc = D;
        ga.tiles = g->gemm_tiles(kRowsNodes);
        ga.Y = dh; ga.ldy = D;
        if (res) { ga.ep.residual = res; ga.ep.ld_res = D; }
        if ((st = launch_typed_gemm(ga, s)) != RGNN_OK) return st;
    } else {   // a 3D-deep weight tile would not fit LDS at D = 128
        if ((st = node_gemm_t(g, D, w.dKV, ldk, Wk, dh, res, 0, s)) != RGNN_OK) return st;
        if ((st = node_gemm_t(g, D, w.dKV + D, ldk, Wv, dh, nullptr, 1, s)) != RGNN_OK) return st;
        if (!typed && (st = node_gemm_t(g, D, w.dKV + 2 * D, ldk, Wq, dh, nullptr, 1, s)) != RGNN_OK) return st;
    }
    if (typed && (st = launch_vseg_reduce(g, w.Tq, nullptr, D, dh, 1, 0, s)) != RGNN_OK) return st;
    if ((st = launch_outer_chunks(g->dev.tiles_types_outer, g->n_tiles_types_outer, g->dev.ntype_perm, 1, h, D, w.dKV,
                                  ldk, w.chunks, D, s, h, w.dKV + D, w.chunks2)) != RGNN_OK)
        return st;
    if ((st = launch_chunk_sum(w.chunks, g->dev.types_chunkptr, g->T, dWk, D, s, w.chunks2, dWv)) != RGNN_OK) return st;
    if (!typed && (st = type_outer(g, D, h, D, w.dKV + 2 * D, ldk, w.chunks, dWq, s)) != RGNN_OK) return st;
    return RGNN_OK;
}

}  // namespace

rgnn_status hgt_backward_impl(const rgnn_graph *g, const float *h, const float *Wk, const float *Wq,
                              const float *Wv, const float *Wa, const float *Watt, const float *Wmsg,
                              const float *mu, int d, int heads, float att_scale, int flags,
                              const float *Gm, const float *saved, float *dh, float *dWk, float *dWq,
                              float *dWv, float *dWa, float *dWatt, float *dWmsg, float *dmu, void *ws,
                              size_t ws_bytes, hipStream_t s, size_t *need)
{
    const int H = heads;
    const size_t bytes = hgt_bwd_layout(g, d, H > 0 ? H : 1, nullptr, nullptr);
    if (need) { *need = bytes; return RGNN_OK; }
    if (d != 32 && d != 64 && d != 128) return fail(RGNN_EUNSUPPORTED, "HGT backward supports d = 32, 64 or 128");
    if (!(H == 1 || H == 2 || H == 4 || H == 8) || d / H < 16)
        return fail(RGNN_EUNSUPPORTED, "HGT backward heads must be 1, 2, 4 or 8 with d / heads >= 16");
    if (!ws || ws_bytes < bytes)
        return fail(RGNN_EINVAL, "workspace too small: need " + std::to_string(bytes) + " bytes");
#define HB(D) hgt_backward_d<D>(g, h, Wk, Wq, Wv, Wa, Watt, Wmsg, mu, H, att_scale, flags, Gm, saved, dh, dWk, \
                                dWq, dWv, dWa, dWatt, dWmsg, dmu, ws, s)
    if (d == 32) return HB(32);
    if (d == 64) return HB(64);
    return HB(128);
#undef HB
}

}  // namespace rgnn
