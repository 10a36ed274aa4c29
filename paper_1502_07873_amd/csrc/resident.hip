// Leapfrog solves resident in LDS: small grids advanced through their whole
// time loop by one workgroup each, in one launch.
#include <type_traits>
#include <utility>

#include "ce.h"
#include "internal.h"
#include "node_update.h"
#include "stream.h"

namespace eig {

namespace {

// Resident solves (variants 21, 22): a grid whose two field levels fit one
// workgroup's LDS (2 nx nz float2, rows nx nodes apart) is advanced through
// its whole time loop by one workgroup of 16 waves, so the fields never
// leave the CU; one barrier per step separates the levels.  What follows is the
// kernel with the fields in LDS, for nodal media and for depth-only grids that
// resident_class does not give to resident_registers below.  Level m sits in
// LDS half m & 1 and u^{m+1} overwrites u^{m-1} in place (every node is
// read at the old level and written only by its owner).
//
// Work split: the W = nx-2 free columns times the nz-1 free rows are cut
// into nb = floor(1024 / W) row bands, and thread t takes column t mod W of
// band t div W (threads past nb W rest; a grid wider than 1024 columns takes
// several passes of one band).  Lanes are thus packed across band
// boundaries instead of rounding each band up to whole waves: 99 columns
// leave 34 of 1024 lanes idle rather than 29 of every 128.  A thread
// streams down its band keeping rows k-1, k, k+1 as in the one-node
// kernels.  Nothing inside a step waits on device memory: the forcing
// window weights and, for depth-only media, the coefficient table (nz rows
// of kCoefStride floats, read per lane) are staged in LDS after the
// fields, the edge nodes' coefficients are held in registers, the receiver
// map is read once and the series value one step ahead.  Absorbing edge
// nodes follow in the same phase: their relation reads only u^m and the
// node's own u^{m-1}.  The per-node arithmetic is that of the one-node
// kernels (layered_update, nodal_node_at, ce_edge_update), so the fields
// are bitwise those of every variant.
constexpr int kResThreads = 64 * kResWaves;
constexpr int kResEdgePerThread = kResidentMaxEdge / kResThreads;

template <int KIND>
__device__ __forceinline__ void resident_lds(const SolveDesc* d, bool absorbing, float2* res_lds) {
    const int nx = d->nx, nz = d->nz, nsteps = d->nsteps;
    const int plane = nx * nz;
    for (int j = threadIdx.x; j < 2 * plane; j += kResThreads)
        res_lds[j] = make_float2(0.f, 0.f);
    float* const srcw_lds = (float*)(res_lds + 2 * plane);     // 2 kSrcW^2 floats
    float* const coef_lds = srcw_lds + kResSrcwFloats;         // depth-only media
    for (int j = threadIdx.x; j < 2 * kSrcW * kSrcW; j += kResThreads)
        srcw_lds[j] = ld1(d->srcw, j);
    if constexpr (KIND == EIG_MEDIUM_LAYERED)
        for (int j = threadIdx.x; j < nz * kCoefStride; j += kResThreads)
            coef_lds[j] = ld1(d->coef, j);
    const int W = nx - 2;           // free columns 1..nx-2
    const int nrow = nz - 1;        // free rows 0..nz-2
    const int nb = max(1, kResThreads / W);
    const int npair = nb * W;       // (band, column) pairs
    const int nedge = 2 * nz + nx - 2;
    const int si0 = d->src_i0, sk0 = d->src_k0;
    const float* srcs = d->srcs;
    float2* traces = d->traces;
    const int nrec = d->nrec;
    const float2* rfz = d->rforce;
    float2* wrec = d->wrec;
    const float* coef = d->coef;
    const int cpitch = d->pitch;
    const size_t cplane = (size_t)nz * cpitch;
    const float h2 = d->h2;
    CeCoef ecoef[kResEdgePerThread];
#pragma unroll
    for (int q = 0; q < kResEdgePerThread; ++q) {
        const int e = threadIdx.x + q * kResThreads;
        ecoef[q] = CeCoef{0.f, 0.f, 0.f};
        if (absorbing && e < nedge) {
            const int2 ik = ce_edge_pos(nx, nz, e);
            ecoef[q] = ce_coef(*d, ik.x, ik.y);
        }
    }
    // the thread's (band, column) pair of its first pass and its receiver,
    // fixed over the time loop
    const int b_first = (int)threadIdx.x / W;
    const int i_first = (int)threadIdx.x - b_first * W + 1;
    const int kb_first = b_first * nrow / nb, ke_first = (b_first + 1) * nrow / nb;
    int rec_first = -1;   // only read where the band starts at the surface
    if ((int)threadIdx.x < npair && kb_first == 0) rec_first = ldi(d->recmap, i_first);
    __syncthreads();
    float sval_next = nsteps > 0 ? ld1(srcs, 0) : 0.f;
    for (int m = 0; m < nsteps; ++m) {
        const float2* Q = res_lds + ((m & 1) ? plane : 0);  // u^m
        float2* P = res_lds + ((m & 1) ? 0 : plane);        // u^{m-1} -> u^{m+1}
        const float sval = sval_next;
        if (m + 1 < nsteps) sval_next = ld1(srcs, m + 1);
        for (int v = threadIdx.x; v < npair; v += kResThreads) {
            const bool first = v == (int)threadIdx.x;
            int i = i_first, kb = kb_first, ke = ke_first;
            if (!first) {  // grids wider than one pass
                const int b = v / W;
                i = v - b * W + 1;
                kb = b * nrow / nb;
                ke = (b + 1) * nrow / nb;
            }
            const int di = i - si0;
            const bool src_lane = di >= 0 && di < kSrcW;
            int rec = -1;
            if (kb == 0) rec = first ? rec_first : ldi(d->recmap, i);
            if constexpr (KIND == EIG_MEDIUM_LAYERED) {
                auto row = [&](int k) {
                    const float2* r = Q + k * nx + i;
                    const float2 l = r[-1], c = r[0], rr = r[1];
                    return node_row(c.x, c.y, l.x, l.y, rr.x, rr.y);
                };
                // rows of the source window and the surface row take the
                // forcing and receiver paths; the other rows are the plain
                // update
                auto update = [&](int k, const NodeRow& rm, const NodeRow& rc,
                                  const NodeRow& rn) {
                    LayerCoef cf;
#pragma unroll
                    for (int j = 0; j <= kFco; ++j) cf.c[j] = coef_lds[k * kCoefStride + j];
                    const float2 up = P[k * nx + i];
                    const int dk = k - sk0;
                    if (k != 0 && (unsigned)dk >= (unsigned)kSrcW) {
                        P[k * nx + i] = layered_update(cf, rm, rc, rn, up.x, up.y, false, 0.f,
                                                       0.f, 0.f);
                        return;
                    }
                    const bool in_win = src_lane && dk >= 0 && dk < kSrcW;
                    bool src = in_win;
                    float wu = 0.f, wv = 0.f, fsv = cf.c[kFco] * sval;
                    if (src) {
                        wu = srcw_lds[(0 * kSrcW + dk) * kSrcW + di];
                        wv = srcw_lds[(1 * kSrcW + dk) * kSrcW + di];
                    }
                    if (rfz && k == 0 && rec >= 0) {  // dual solve: receiver injection
                        const float2 rf = ld2(rfz, (size_t)m * nrec + rec);
                        src = true;
                        fsv = cf.c[kFco];
                        wu = rf.x;
                        wv = rf.y;
                    }
                    const float2 nw = layered_update(cf, rm, rc, rn, up.x, up.y, src, fsv, wu, wv);
                    P[k * nx + i] = nw;
                    if (k == 0 && rec >= 0) st2(traces, (size_t)(m + 1) * nrec + rec, nw);
                    if (wrec && in_win)
                        st2(wrec, (size_t)m * (kSrcW * kSrcW) + dk * kSrcW + di, nw);
                };
                NodeRow r0 = NodeRow{0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                if (kb > 0) r0 = row(kb - 1);
                NodeRow r1 = row(kb);
                int k = kb;
                // three rows per trip: the rows rotate through registers
                for (; k + 3 <= ke; k += 3) {
                    const NodeRow r2 = row(k + 1);
                    update(k, r0, r1, r2);
                    const NodeRow r3 = row(k + 2);
                    update(k + 1, r1, r2, r3);
                    const NodeRow r4 = row(k + 3);
                    update(k + 2, r2, r3, r4);
                    r0 = r3;
                    r1 = r4;
                }
                for (; k < ke; ++k) {
                    const NodeRow r2 = row(k + 1);
                    update(k, r0, r1, r2);
                    r0 = r1;
                    r1 = r2;
                }
            } else {
                const float* LAM = coef;
                const float* MU = coef + cplane;
                const float* SC = coef + 2 * cplane;
                auto U = [&](int ii, int kk) { return Q[kk * nx + ii]; };
                for (int k = kb; k < ke; ++k) {
                    const int dk = k - sk0;
                    const bool in_win = src_lane && dk >= 0 && dk < kSrcW;
                    int inj = 0;
                    float w0 = 0.f, w1 = 0.f;
                    if (rfz && k == 0 && rec >= 0) {  // dual solve: receiver injection
                        const float2 rf = ld2(rfz, (size_t)m * nrec + rec);
                        inj = 1;
                        w0 = rf.x;
                        w1 = rf.y;
                    } else if (in_win) {
                        inj = 2;
                        w0 = srcw_lds[(0 * kSrcW + dk) * kSrcW + di];
                        w1 = srcw_lds[(1 * kSrcW + dk) * kSrcW + di];
                    }
                    const float2 nw = nodal_node_at(U, P[k * nx + i], LAM, MU, SC, cpitch, i, k,
                                                    inj, h2, sval, w0, w1);
                    P[k * nx + i] = nw;
                    if (k == 0 && rec >= 0) st2(traces, (size_t)(m + 1) * nrec + rec, nw);
                    if (wrec && in_win)
                        st2(wrec, (size_t)m * (kSrcW * kSrcW) + dk * kSrcW + di, nw);
                }
            }
        }
        if (absorbing) {
#pragma unroll
            for (int q = 0; q < kResEdgePerThread; ++q) {
                const int e = threadIdx.x + q * kResThreads;
                if (e < nedge) ce_edge_update(*d, Q, P, nx, e, ecoef[q]);
            }
        }
        __syncthreads();
    }
}

// resident_registers: depth-only grids of one strip keep both levels in
// registers.  A wave owns a band of rows, N = 2 neighbouring columns per lane (1
// where 64 lanes hold the row), and takes from LDS what its neighbours hold: the
// row above and the row below of u^m, which every wave leaves there a step ahead.
// With rigid edges lane 0 holds column 1 (what lies beyond the wave is zero) and
// nodes past column nx-2 are kept zero; with absorbing ones lane 0 holds column
// 0, the side columns' lanes load them from LDS, and the inner columns are left
// there for them: the edge nodes, 64 to a group, are the business of the last
// waves, which have the fewest rows.  Everything in LDS is double-buffered by the
// parity of its level, so that one barrier per step suffices.  The number of rows
// is a template argument (a runtime one cost 30 registers in merged branches).
//
// Bound: vector issue, 28 instructions per node (one column per lane) or 24 (two),
// and the lanes past the last column; then the barrier with what follows it (the
// neighbours' rows from LDS).  The kernel with the fields in LDS reads five LDS
// words and 13 coefficients per node, 61 instructions.  Measured, against it, per
// launch: 120 solves of 64 x 64 x 400 (one workgroup per CU) 1.08 -> 0.55 ms, 1600
// of them on average 5.9 -> 2.3 ms; 15000 of 101 x 76 x 320 with absorbing edges
// 67.3 -> 42.5 ms (5.5e11 -> 8.7e11 updates/s).
struct ResSolve {
    const SolveDesc* d;
    const float* coef;
    const float2* rfz;
    float2 *traces, *wrec;
    int nx, nz, nrec, si0, sk0, nsteps;
    // LDS: two buffers, kept apart by `half` float2
    float2* rows;       // [kResWaves + 2][2][64 N]: a wave's first and last row
    float2* side;       // [2][nz] side columns
    float2* inner;      // [2][nz] columns 1 and nx-2
    int half;
    const float2* srcw;  // [7][8] window weights, the last column zero
    const struct EdgeRow* edge;
};
struct EdgeRow {  // of a row: 1 / (1 + a_p), 1 / (1 + a_s) and a_p, a_s, l (ce.h)
    double rp, rs;
    float ap, as, l, pad;
};

template <int N>
__device__ __forceinline__ Pt<N> lds_pt(const float2* p) {
    Pt<N> w;
    if constexpr (N == 2) {
        const float4 q = *(const float4*)p;
        w.u[0] = q.x;
        w.v[0] = q.y;
        w.u[1] = q.z;
        w.v[1] = q.w;
    } else {
        w.u[0] = p->x;
        w.v[0] = p->y;
    }
    return w;
}
template <int N>
__device__ __forceinline__ void lds_put(float2* p, const Pt<N>& w) {
    if constexpr (N == 2)
        *(float4*)p = make_float4(w.u[0], w.v[0], w.u[1], w.v[1]);
    else
        *p = make_float2(w.u[0], w.v[0]);
}

// Edge node e (ce_edge_pos), u^m in LDS buffer half par, u^{m-1} in the other one,
// which takes u^{m+1}.  The relation of ce.h, its quotients as products with the
// FP64 reciprocals (the same bits, as absorbing_columns says).  last: the wave that owns row nz-2.
template <int N>
__device__ __forceinline__ void resident_edge(const ResSolve& g, int par, int e, int last) {
#pragma clang fp contract(off)
    const int nx = g.nx, nz = g.nz, q = par ? g.half : 0, p = par ? 0 : g.half;
    const int bot = ((last + 2) * 2) * 64 * N;  // row nz-1 lies below the last wave's
    const bool bottom = e >= 2 * nz, left = e < nz;
    const int s = left ? 0 : nz, k = bottom ? nz - 1 : e - s;
    const int i = bottom ? e - 2 * nz + 1 : left ? 0 : nx - 1;
    const float2 *up, *dn, *in, *old;
    if (bottom) {
        up = g.rows + q + bot + i + 1;
        dn = g.rows + q + bot + i - 1;
        in = g.rows + q + ((last + 1) * 2 + 1) * 64 * N + i;
        old = g.rows + p + bot + i;
    } else {
        up = g.side + q + s + min(k + 1, nz - 1);
        dn = g.side + q + s + max(k - 1, 0);
        in = k == nz - 1 ? g.rows + q + bot + (left ? 1 : nx - 2) : g.inner + q + s + k;
        old = g.side + p + s + k;
    }
    const float half = !bottom && (k == 0 || k == nz - 1) ? 1.f : 0.5f;
    const EdgeRow t = g.edge[k];
    const float sg = left && !bottom ? 1.f : -1.f;
    const float a1 = bottom ? t.as : t.ap, a2 = bottom ? t.ap : t.as;
    const double r1 = bottom ? t.rs : t.rp, r2 = bottom ? t.rp : t.rs;
    const float t1 = sg * (bottom ? t.as : t.l), t2 = sg * (bottom ? t.l : t.as);
    const float dx = half * (up->x - dn->x), dy = half * (up->y - dn->y);
    auto edge = [](float a, double r, float prev, float inn, float tang) {
        return (float)(__builtin_fmaf(1.f - a, prev, 2.f * __builtin_fmaf(a, inn, tang)) * r);
    };
    const float2 w = make_float2(edge(a1, r1, old->x, in->x, t1 * dy),
                                 edge(a2, r2, old->y, in->y, t2 * dx));
    if (!bottom) g.side[p + s + k] = w;
    if (k == nz - 1) g.rows[p + bot + i] = w;
}

// What a lane keeps over the time loop.
template <int N, int ABS>
struct ResLane {
    int at;             // the lane's first node in an LDS row
    bool in[N];         // rigid: columns 1..nx-2
    int win[N];         // column of the forcing window, kSrcW: none
    int rec[N];         // receiver, -1: none
    // absorbing: the LDS places of the nodes that are side columns and of those
    // next to them, -1: none
    int side[N], inner[N];
};

// One step: cur holds u^m, prv u^{m-1} and then u^{m+1}, rows [k0, k0 + R).
// ABS: 0 rigid, 1 + (nx - 1) % N absorbing.
template <int N, int R, int ABS>
__device__ __forceinline__ void resident_step(const ResSolve& g, const ResLane<N, ABS>& l, int w,
                                              int k0, int m, int par, float sval,
                                              Pt<N> (&cur)[R + 1], Pt<N> (&prv)[R + 1]) {
    // opaque, so that what follows from them for each row is formed where it is
    // used rather than held in scalar registers over the time loop
    __asm__ volatile("" : "+s"(k0));
    const float2* q = g.rows + (par ? g.half : 0) + l.at;
    float2* o = g.rows + (par ? 0 : g.half) + (w + 1) * 2 * 64 * N + l.at;
    Pt<N> above = lds_pt<N>(q + (w * 2 + 1) * 64 * N);
    cur[R] = lds_pt<N>(q + (w + 2) * 2 * 64 * N);
    if constexpr (ABS != 0) {
        // rows k0 - 1 .. k0 + R (above the surface: any value, it meets zeros)
#pragma unroll
        for (int j = -1; j <= R; ++j)
#pragma unroll
            for (int n = 0; n < N; ++n) {
                if (n != 0 && ABS != 2) continue;
                if (l.side[n] >= 0) {
                    const float2 s = g.side[(par ? g.half : 0) + max(l.side[n] + j, 0)];
                    Pt<N>& row = j < 0 ? above : cur[j < 0 ? 0 : j];
                    row.u[n] = s.x;
                    row.v[n] = s.y;
                }
            }
    }
    ScalarRow crow = (ScalarRow)((uintptr_t)g.coef) + (ptrdiff_t)k0 * kCoefStride;
    __asm__ volatile("" : "+s"(crow));
    LayerCoef cf_next = scalar_coef(crow);
    Pt<N> p = above, dp = x_diff<N>(above), dc = x_diff<N>(cur[0]);
    auto row = [&](auto jc) {
        constexpr int j = jc.value;
        const int k = k0 + j;
        const LayerCoef cf = cf_next;
        __asm__ volatile("" ::"s"(cf.c[0]));
        cf_next = scalar_coef(crow + (j + 1) * kCoefStride);
        __builtin_amdgcn_sched_barrier(0);
        const Pt<N>&c = cur[j], &n = cur[j + 1];
        const Pt<N> dn = x_diff<N>(n), sx = x_sum<N>(c);
        float2 a[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const NodeRow rm{p.u[i], p.v[i], dp.u[i], dp.v[i], 0.f, 0.f};
            const NodeRow rc{c.u[i], c.v[i], 0.f, 0.f, sx.u[i], sx.v[i]};
            const NodeRow rn{n.u[i], n.v[i], dn.u[i], dn.v[i], 0.f, 0.f};
            a[i] = layered_accel<false>(cf, rm, rc, rn);
        }
        const int dk = k - g.sk0;
        const bool window = (unsigned)dk < (unsigned)kSrcW;
        if (__builtin_expect(k == 0 || window, 0)) {
            const ScalarRow here = crow + j * kCoefStride;
            const float fco = here[kFco], fsv = fco * sval;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (k == 0) {
                    a[i].x = __builtin_fmaf(here[kCm0U], dc.v[i], a[i].x);
                    a[i].y = __builtin_fmaf(here[kCm0V], dc.u[i], a[i].y);
                }
                if (g.rfz && k == 0 && l.rec[i] >= 0) {  // dual solve: receiver injection
                    const float2 f = ld2(g.rfz, (size_t)m * g.nrec + l.rec[i]);
                    a[i].x = __builtin_fmaf(fco, f.x, a[i].x);
                    a[i].y = __builtin_fmaf(fco, f.y, a[i].y);
                } else if (window && l.win[i] != kSrcW) {
                    const float2 f = g.srcw[dk * 8 + l.win[i]];
                    a[i].x = __builtin_fmaf(fsv, f.x, a[i].x);
                    a[i].y = __builtin_fmaf(fsv, f.y, a[i].y);
                }
            }
        }
        Pt<N> nw;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float2 x = layered_new(a[i], c.u[i], c.v[i], prv[j].u[i], prv[j].v[i]);
            nw.u[i] = x.x;
            nw.v[i] = x.y;
            if constexpr (ABS == 0) {
                nw.u[i] = l.in[i] ? nw.u[i] : 0.f;
                nw.v[i] = l.in[i] ? nw.v[i] : 0.f;
            }
        }
        if (__builtin_expect(k == 0 || (g.wrec && window), 0)) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float2 x = make_float2(nw.u[i], nw.v[i]);
                if (k == 0 && l.rec[i] >= 0) st2(g.traces, (size_t)(m + 1) * g.nrec + l.rec[i], x);
                if (g.wrec && window && l.win[i] != kSrcW)
                    st2(g.wrec, (size_t)m * (kSrcW * kSrcW) + dk * kSrcW + l.win[i], x);
            }
        }
        if constexpr (ABS != 0) {
            // (two columns per lane: column 1 is node 1; column nx-2 the other node than nx-1's)
#pragma unroll
            for (int i = 0; i < N; ++i)
                if ((i != 0 || N == 1 || ABS == 2) && l.inner[i] >= 0)
                    g.inner[(par ? 0 : g.half) + l.inner[i] + j] = make_float2(nw.u[i], nw.v[i]);
        }
        if (j == 0) lds_put<N>(o, nw);
        if (j == R - 1) lds_put<N>(o + 64 * N, nw);
        prv[j] = nw;
        p = c;
        dp = dc;
        dc = dn;
    };
    [&]<int... J>(std::integer_sequence<int, J...>) {
        (row(std::integral_constant<int, J>()), ...);
    }(std::make_integer_sequence<int, R>());
}

// The time loop of wave w, which owns R rows from k0 on.
template <int N, int R, int ABS>
__device__ __forceinline__ void resident_band(const ResSolve& g, int w, int k0, int last) {
    const int lane = threadIdx.x & 63, nx = g.nx, nz = g.nz;
    ResLane<N, ABS> l;
    l.at = N * lane;
    const int col = l.at + (ABS ? 0 : 1);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = col + i;
        l.in[i] = c >= 1 && c <= nx - 2;
        l.win[i] = l.in[i] ? (int)min((unsigned)(c - g.si0), (unsigned)kSrcW) : kSrcW;
        l.rec[i] = w == 0 && l.in[i] ? ldi(g.d->recmap, c) : -1;
        l.side[i] = c == 0 ? k0 : c == nx - 1 ? nz + k0 : -1;
        l.inner[i] = c == 1 ? k0 : c == nx - 2 ? nz + k0 : -1;
    }
    const int nedge = ABS ? 2 * nz + nx - 2 : 0;
    Pt<N> a[R + 1], b[R + 1];
#pragma unroll
    for (int j = 0; j <= R; ++j) a[j] = b[j] = Pt<N>{};
    ScalarRow srcs = (ScalarRow)((uintptr_t)g.d->srcs);
    float sval = g.nsteps > 0 ? srcs[0] : 0.f;
    auto step = [&](int m, int par, Pt<N>(&cur)[R + 1], Pt<N>(&prv)[R + 1]) {
        const float s = sval;
        sval = srcs[min(m + 1, g.nsteps - 1)];
        if constexpr (R > 0) resident_step<N, R, ABS>(g, l, w, k0, m, par, s, cur, prv);
        if constexpr (ABS != 0)
            for (int e = (kResWaves - 1 - w) * 64 + lane; e < nedge; e += kResThreads)
                resident_edge<N>(g, par, e, last);
        // LDS only: the records' stores need not have landed
        __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    for (int m = 0; m < g.nsteps; m += 2) {
        step(m, 0, a, b);
        if (m + 1 < g.nsteps) step(m + 1, 1, b, a);
    }
}

// Waves own nrow / 16 rows, or one more; RMAX: the instances' largest number.
template <int N, int RMAX, int ABS>
__device__ __forceinline__ void resident_run(const ResSolve& g) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nrow = g.nz - 1;
    const int per = nrow / kResWaves, more = nrow % kResWaves;
    const int k0 = w * per + min(w, more), cnt = per + (w < more);
    const int last = per ? kResWaves - 1 : more - 1;
    [&]<int... R>(std::integer_sequence<int, R...>) {
        ((cnt == R ? resident_band<N, R, ABS>(g, w, k0, last) : void()), ...);
    }(std::make_integer_sequence<int, RMAX + 1>());
}

// Sets up LDS and runs the grid's instance.
template <bool WIDE>
__device__ __forceinline__ void resident_registers(const SolveDesc* d, bool absorbing,
                                                   float4* lds) {
    ResSolve g;
    g.d = d;
    g.coef = d->coef;
    g.rfz = d->rforce;
    g.traces = d->traces;
    g.wrec = d->wrec;
    g.nx = d->nx;
    g.nz = d->nz;
    g.nrec = d->nrec;
    g.si0 = d->src_i0;
    g.sk0 = d->src_k0;
    g.nsteps = d->nsteps;
    const int N = resident_columns(g.nx, absorbing);
    const int nrows = (kResWaves + 2) * 2 * 64 * N;
    g.half = nrows + (absorbing ? 4 * g.nz : 0);
    g.rows = (float2*)lds;
    g.side = g.rows + nrows;
    g.inner = g.side + 2 * g.nz;
    float2* srcw = g.rows + 2 * g.half;
    EdgeRow* edge = (EdgeRow*)(srcw + 64);
    for (int j = threadIdx.x; j < g.half; j += kResThreads)
        lds[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (threadIdx.x < 64) {
        const int dk = threadIdx.x / 8, di = threadIdx.x % 8;
        float2 x = make_float2(0.f, 0.f);
        if (dk < kSrcW && di < kSrcW)
            x = make_float2(ld1(d->srcw, dk * kSrcW + di), ld1(d->srcw, (kSrcW + dk) * kSrcW + di));
        srcw[threadIdx.x] = x;
    }
    if (absorbing) {
        const double* ce = (const double*)(d->coef + ce_table(g.nz));
        for (int k = threadIdx.x; k < g.nz; k += kResThreads) {
            const float* c = d->coef + (size_t)k * kCoefStride;
            edge[k] = {ce[k * (kCeStride / 2)], ce[k * (kCeStride / 2) + 1], c[kCeP], c[kCeS],
                       c[kCeL], 0.f};
        }
    }
    g.srcw = srcw;
    g.edge = edge;
    __syncthreads();
    constexpr int R1 = WIDE ? kResRows1 : kResRows1Small;
    if (N == 1) {
        if (absorbing) resident_run<1, R1, 1>(g);
        else resident_run<1, R1, 0>(g);
    } else if constexpr (WIDE) {
        if (!absorbing) resident_run<2, kResRows2, 0>(g);
        else if (g.nx & 1) resident_run<2, kResRows2, 1>(g);
        else resident_run<2, kResRows2, 2>(g);
    }
}

// ANY: grids of every class; without, all of the launch's are of the smallest one,
// whose registers leave room for two workgroups on a CU.
template <bool ANY>
__global__ void __launch_bounds__(kResThreads, ANY ? 4 : 8)
stencil_resident_layered(const SolveDesc* __restrict__ descs, const int2* __restrict__ tiles,
                         int ntiles) {
    extern __shared__ float4 res_lds4[];
    if ((int)blockIdx.x >= ntiles) return;
    const int2 te = tiles[blockIdx.x];
    const SolveDesc* d = descs + __builtin_amdgcn_readfirstlane(te.x);
    const bool absorbing = __builtin_amdgcn_readfirstlane(te.y) != 0;
    if (ANY && resident_class(d->nx, d->nz, absorbing) == 2)
        resident_lds<EIG_MEDIUM_LAYERED>(d, absorbing, (float2*)res_lds4);
    else
        resident_registers<ANY>(d, absorbing, res_lds4);
}

__global__ void __launch_bounds__(kResThreads)
stencil_resident_nodal(const SolveDesc* __restrict__ descs, const int2* __restrict__ tiles,
                       int ntiles) {
    extern __shared__ float4 res_lds4[];
    if ((int)blockIdx.x >= ntiles) return;
    const int2 te = tiles[blockIdx.x];
    resident_lds<EIG_MEDIUM_NODAL>(descs + __builtin_amdgcn_readfirstlane(te.x),
                                   __builtin_amdgcn_readfirstlane(te.y) != 0, (float2*)res_lds4);
}

}  // namespace

void launch_resident(const SolveDesc* descs, const int2* tiles, int ntiles, int kind, int cls,
                     size_t lds_bytes, hipStream_t s) {
    if (ntiles <= 0) return;
    const auto fn = kind == EIG_MEDIUM_NODAL ? stencil_resident_nodal
                    : cls == 0               ? stencil_resident_layered<false>
                                             : stencil_resident_layered<true>;
    // allow dynamic LDS up to the whole 160 KiB of a CU for this kernel (on
    // the current device; idempotent, once per wave)
    (void)hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)kResidentLdsBytes);
    (void)hipGetLastError();
    fn<<<ntiles, kResThreads, lds_bytes, s>>>(descs, tiles, ntiles);
}

}  // namespace eig
