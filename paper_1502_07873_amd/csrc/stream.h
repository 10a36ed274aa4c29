// What the streaming kernels share (stream.hip, stream_nodal.hip): rows of a
// strip held by a wave, x-neighbours across its lanes, a tile's geometry and
// the feed of field rows.
#pragma once

#include "internal.h"
#include "node_update.h"
#include "tile.h"

namespace eig {

namespace {

// A tile's forcing tables: the window's weights (two components), dt^2 / rho
// of its rows (depth-only media), and the series values of the K steps.
constexpr int kSwFco = 2 * kSrcW * kSrcW, kSwSeries = kSwFco + kSrcW;

// A row of a coefficient table through the scalar cache.
#if defined(__HIP_DEVICE_COMPILE__)
#define CAS __attribute__((address_space(4)))
#else
#define CAS
#endif
typedef const CAS float* ScalarRow;
__device__ __forceinline__ LayerCoef scalar_coef(ScalarRow c) {
    LayerCoef r;
#pragma unroll
    for (int j = 0; j < kFco; ++j) r.c[j] = c[j];
    return r;
}

// N neighbouring nodes of one row held by a lane.
template <int N>
struct Pt {
    float u[N], v[N];
};

// Values of the neighbouring lane; lanes 0 / 63 receive zero.
__device__ __forceinline__ float lane_left(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_right(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x130, 0xf, 0xf, true));
}

template <int N>
__device__ __forceinline__ void x_neighbours(const float (&w)[N], float (&l)[N], float (&r)[N]) {
    l[0] = lane_left(w[N - 1]);
    r[N - 1] = lane_right(w[0]);
#pragma unroll
    for (int n = 1; n < N; ++n) {
        l[n] = w[n - 1];
        r[n - 1] = w[n];
    }
}

template <int N>
__device__ __forceinline__ Pt<N> x_diff(const Pt<N>& w) {
    float l[N], r[N];
    Pt<N> d;
    x_neighbours<N>(w.u, l, r);
#pragma unroll
    for (int n = 0; n < N; ++n) d.u[n] = r[n] - l[n];
    x_neighbours<N>(w.v, l, r);
#pragma unroll
    for (int n = 0; n < N; ++n) d.v[n] = r[n] - l[n];
    return d;
}

template <int N>
__device__ __forceinline__ Pt<N> x_sum(const Pt<N>& w) {
    float l[N], r[N];
    Pt<N> d;
    x_neighbours<N>(w.u, l, r);
#pragma unroll
    for (int n = 0; n < N; ++n) d.u[n] = r[n] + l[n];
    x_neighbours<N>(w.v, l, r);
#pragma unroll
    for (int n = 0; n < N; ++n) d.v[n] = r[n] + l[n];
    return d;
}

template <int N>
__device__ __forceinline__ Pt<N> ld_pt(const float2* row, int col) {
    Pt<N> p;
    if constexpr (N == 2) {
        const float4 q = ld4(row, col);
        p.u[0] = q.x;
        p.v[0] = q.y;
        p.u[1] = q.z;
        p.v[1] = q.w;
    } else {
        const float2 q = ld2(row, col);
        p.u[0] = q.x;
        p.v[0] = q.y;
    }
    return p;
}
template <int N>
__device__ __forceinline__ void st_pt(float2* row, int col, const Pt<N>& p) {
    if constexpr (N == 2)
        st4(row, col, make_float4(p.u[0], p.v[0], p.u[1], p.v[1]));
    else
        st2(row, col, make_float2(p.u[0], p.v[0]));
}

template <int K, int N>
struct StreamTile {
    const float* coef;
    float2 *out0, *out1;       // levels m + K and m + K - 1
    float2* traces;
    int nz, pitch, m, nsteps, nrec;
    int kb, nstore;            // rows stored (none in the last pass)
    int x0, col;               // the strip's and the lane's first column (within the pitch)
    bool st_ok;                // the lane stores its nodes
    bool free_col[N];          // columns 1..nx-2
    bool left, right;          // the lane holds column 0 / nx-1
    const int* rec;            // the strip's receivers, -1 where none (LDS)
    int sk0, si0;              // forcing window: first row and column
    const float* sw;           // forcing tables (LDS)
    int f0, f1, w0, w1;        // plain rows: [f0, f1) but [w0, w1)
};

// Geometry, buffers and receivers of the strip from x0 on, rows [kb, ke), of
// the pass that starts at level m (pin: the buffer pair it reads).
template <int K, int N>
__device__ __forceinline__ void tile_init(StreamTile<K, N>& t, const SolveDesc* d, int m, int pin,
                                          int x0, int kb, int ke, const float* sw,
                                          int* rec) {
    const int nx = d->nx;
    constexpr int W = 64 * N;
    const int cs = x0 == 0 ? 0 : x0 + K, ce = x0 + W >= nx ? nx : x0 + W - K;
    t.coef = d->coef;
    t.nz = d->nz;
    t.pitch = d->pitch;
    t.m = m;
    t.nsteps = d->nsteps;
    t.nrec = d->nrec;
    t.traces = d->traces;
    t.kb = kb;
    t.nstore = m + K >= t.nsteps ? 0 : ke - kb;
    const int col = x0 + N * (int)threadIdx.x;
    t.x0 = x0;
    t.col = min(col, t.pitch - N);  // lanes past the pitch hold what no column reads
    t.st_ok = col >= cs && col < ce;
    t.sk0 = d->src_k0;
    t.si0 = d->src_i0;
    t.sw = sw;
    t.rec = rec;
    t.left = col == 0;
    t.right = col <= nx - 1 && col + N > nx - 1;
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int c = col + q;
        t.free_col[q] = c >= 1 && c <= nx - 2;
        // (a chunk below the first may form the surface row in its halo)
        rec[N * threadIdx.x + q] =
            kb == 0 && t.free_col[q] && c >= cs && c < ce ? ldi(d->recmap, c) : -1;
    }
    // m is even: level m in slot 0 of the pair, m - 1 in slot 1
    t.out0 = pin ? d->buf0 : d->buf2;
    t.out1 = pin ? d->buf1 : d->buf3;
    // rows i whose K levels are all free ones below the surface, and off the
    // forcing window where it meets this strip
    const bool win = t.si0 < x0 + W && t.si0 + kSrcW > x0;
    t.f0 = K + 1;
    t.f1 = t.nz;
    t.w0 = win ? t.sk0 + 1 : t.f1;
    t.w1 = win ? t.sk0 + kSrcW + K : t.f1;
}

template <int K, int N>
__device__ __forceinline__ bool plain_row(const StreamTile<K, N>& t, int i) {
    return i >= t.f0 && i < t.f1 && (i < t.w0 || i >= t.w1);
}

// The lane's first column, formed anew (off the plain path).
template <int K, int N>
__device__ __forceinline__ int lane_col(const StreamTile<K, N>& t) {
    int lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    __asm__ volatile("" : "+v"(lane));
    return t.x0 + N * lane;
}

// The field rows a tile reads, three pipeline rows ahead: row i of u^m and row
// i - 1 of u^{m-1}, held at the grid's last ones.
template <int N>
struct RowFeed {
    const float2 *cur, *prev;
    size_t pitch;
    int col, nz;
    Pt<N> c[3], p[3];  // rows i, i + 1, i + 2
    __device__ __forceinline__ void init(const SolveDesc* d, int pin, int i0, int cld) {
        pitch = d->pitch;
        col = cld;
        nz = d->nz;
        const float2* b1 = pin ? d->buf3 : d->buf1;
        cur = (pin ? d->buf2 : d->buf0) + (size_t)i0 * pitch;
        prev = b1 + (size_t)i0 * pitch;
        c[0] = ld_pt<N>(cur, col);
        p[0] = ld_pt<N>(b1 + (size_t)max(i0 - 1, 0) * pitch, col);
        c[1] = ld_pt<N>(cur + pitch, col);
        p[1] = ld_pt<N>(prev, col);
        c[2] = ld_pt<N>(cur + 2 * pitch, col);
        p[2] = ld_pt<N>(prev + pitch, col);
        cur += 2 * pitch;
        prev += pitch;
    }
    // row i is done: its slot takes row i + 3 (of prev, i + 2: rigid grids do not
    // need its last row)
    template <bool ABS = false>
    __device__ __forceinline__ void next(int i, int slot) {
        const size_t inc = i + 3 < nz ? pitch : 0;
        cur += inc;
        prev += ABS ? (i + 2 < nz ? pitch : 0) : inc;
        c[slot] = ld_pt<N>(cur, col);
        p[slot] = ld_pt<N>(prev, col);
    }
};

// Zero at the rigid columns.
template <int K, int N>
__device__ __forceinline__ void zero_rigid(const StreamTile<K, N>& t, Pt<N>& w) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
        w.u[q] = t.free_col[q] ? w.u[q] : 0.f;
        w.v[q] = t.free_col[q] ? w.v[q] : 0.f;
    }
}

// Receivers of the surface row at level j.
template <int K, int N>
__device__ __forceinline__ void record_row(const StreamTile<K, N>& t, int j, const Pt<N>& nw) {
    const int* rec = t.rec + (lane_col(t) - t.x0);
#pragma unroll
    for (int q = 0; q < N; ++q)
        if (rec[q] >= 0)
            st2(t.traces, (size_t)(t.m + j) * t.nrec + rec[q], make_float2(nw.u[q], nw.v[q]));
}

// A tile entry's geometry; false: the solve does not run in this pass.
struct StreamEntry {
    const SolveDesc* d;
    int m, pin, x0, kb, ke;
    bool narrow;
};
// (absorbing grids: the last row is formed as well)
template <int K, bool ABS = false>
__device__ __forceinline__ bool stream_entry(const SolveDesc* descs, int2 te, int pass, int rows,
                                             StreamEntry& e) {
    e.d = descs + __builtin_amdgcn_readfirstlane(te.x);
    const unsigned sc = (unsigned)__builtin_amdgcn_readfirstlane(te.y);
    const int L = pass - e.d->start;
    e.m = K * L;
    e.pin = L & 1;
    e.x0 = (int)(sc >> 17) * 2;
    e.narrow = (sc & 0x10000) != 0;
    e.kb = (int)(sc & 0xffff) * rows;
    e.ke = min(e.kb + rows, e.d->nz - (ABS ? 0 : 1));
    return L >= 0 && e.m < e.d->nsteps;
}

// Weights and series values of a tile's forcing tables.
template <int K>
__device__ __forceinline__ void load_forcing(const SolveDesc* d, int m, float* sw) {
    for (int e = threadIdx.x; e < 2 * kSrcW * kSrcW; e += 64) sw[e] = ld1(d->srcw, e);
    if (threadIdx.x < K)
        sw[kSwSeries + threadIdx.x] =
            m + (int)threadIdx.x < d->nsteps ? ld1(d->srcs, m + threadIdx.x) : 0.f;
}

}  // namespace

}  // namespace eig
