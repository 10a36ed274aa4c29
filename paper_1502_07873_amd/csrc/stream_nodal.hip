// Nodal media with rigid edges, K = 6 leapfrog steps per launch streamed through
// registers (variant 24, the temporal_blocking 4 family's default; strips,
// passes and levels as in stream.hip).
//
// The medium's rows the levels work on sit in LDS, a ring of nine rows per wave
// (13.8 KB; eight waves per CU): three rows of lambda, mu and s enter per trip,
// loaded a trip ahead, and every level reads its own row once (lambda and mu of
// the row below are the level before's).  A wave is its own workgroup, so the
// ring needs no barrier.  Products and fluxes an update shares with its
// neighbours are formed once: an x-flux by the node to its left (across lanes as
// a DPP operand), the depth flux and the mixed terms' lambda D_x u, mu D_x v of
// a row kept for the row below.  Same operands and roundings as nodal_accel, so
// the fields are bitwise those of every nodal variant.
//
// Bound: vector issue, 50 instructions per update before the strips' overlap and
// the halo rows (63 counted on 512 x 256; the kernel with tile and medium in
// LDS 144, most of it LDS addresses, operand copies and band set-up): at 0.70 of
// the issue limit there, and on 30 solves of 2048 x 1024 in 0.85 of the cycles, with
// memory at 0.6 of a large copy's rate.  K = 6 is what 256 VGPRs hold, and only if
// lambda D_x u of the row above is formed a second time when needed (held, it
// spills).
// Measured, against four steps with the tile in LDS: 15 solves of 2048 x 1024
// 4.7e11 updates/s against 2.7e11 (K = 4: 4.7e11), 360 of 512 x 256 4.5e11
// against 2.9e11 (4.4e11), 960 of 512^2 5.6e11 against 2.9e11 (5.0e11); small
// launches run the LDS kernel (small_launch_variant).
#include "stream.h"

namespace eig {

namespace {

// Levels 0..K-1 of a strip between two rows: level j holds its row i - 1 - j
// in c and the row above in p; lambda D_x u and mu D_x v of the latter (sp);
// and the depth fluxes between them (q).
template <int K, int N>
struct NodalState {
    Pt<N> c[K], p[K], sp[K], q[K];
};

// lambda and mu of a row at the lane's columns, and a = lambda + 2 mu.
template <int N>
struct NodeCoef {
    float lam[N], mu[N], a[N];
};

// The medium's rows a strip works on, in LDS: trips of three rows, the last
// kRingTrips of them kept.  A row holds lambda, mu and s of the strip's columns.
template <int K>
constexpr int kRingTrips = (K + 3 + 2) / 3;
constexpr int kRingRow = 3 * 128;              // floats per row
constexpr int kRingTrip = 3 * kRingRow;

template <int K, int N>
struct Ring {
    float* lds;
    int at[kRingTrips<K>];  // this lane's place in the current trip, the one before, ...
    int head;               // slot of the current trip
    __device__ __forceinline__ void init(float* mem) {
        lds = mem;
        head = 0;
#pragma unroll
        for (int q = 0; q < kRingTrips<K>; ++q) at[q] = place(q ? kRingTrips<K> - q : 0);
    }
    __device__ __forceinline__ int place(int slot) const {
        return slot * kRingTrip + N * (int)threadIdx.x;
    }
    __device__ __forceinline__ void advance() {
        head = head + 1 == kRingTrips<K> ? 0 : head + 1;
#pragma unroll
        for (int q = kRingTrips<K> - 1; q > 0; --q) at[q] = at[q - 1];
        at[0] = place(head);
    }
    // row O of the current trip (negative: of the trips before)
    template <int O>
    __device__ __forceinline__ float* row() const {
        constexpr int back = O >= 0 ? 0 : (-O + 2) / 3;
        return lds + at[back] + (O + 3 * back) * kRingRow;
    }
    __device__ __forceinline__ static void put1(float* p, const float (&w)[N]) {
        if constexpr (N == 2)
            *(float2*)p = make_float2(w[0], w[1]);
        else
            *p = w[0];
    }
    __device__ __forceinline__ static void get1(const float* p, float (&w)[N]) {
        if constexpr (N == 2) {
            const float2 v = *(const float2*)p;
            w[0] = v.x;
            w[1] = v.y;
        } else {
            w[0] = *p;
        }
    }
    template <int O>
    __device__ __forceinline__ void put(const NodeCoef<N>& c, const float (&s)[N]) {
        float* p = row<O>();
        put1(p, c.lam);
        put1(p + 128, c.mu);
        put1(p + 256, s);
    }
    template <int O>
    __device__ __forceinline__ void get(NodeCoef<N>& c) const {
        const float* p = row<O>();
        get1(p, c.lam);
        get1(p + 128, c.mu);
    }
    template <int O>
    __device__ __forceinline__ void get_s(float (&s)[N]) const {
        get1(row<O>() + 256, s);
    }
};

template <int N>
__device__ __forceinline__ void set_a(NodeCoef<N>& c) {
#pragma unroll
    for (int q = 0; q < N; ++q) c.a[q] = __builtin_fmaf(2.f, c.mu[q], c.lam[q]);
}

// w at the column to the right / left of each of the lane's columns.
template <int N>
__device__ __forceinline__ float right_of(const float (&w)[N], int q) {
    return q + 1 < N ? w[q + 1 < N ? q + 1 : 0] : lane_right(w[0]);
}
template <int N>
__device__ __forceinline__ float left_of(const float (&w)[N], int q) {
    return q > 0 ? w[q > 0 ? q - 1 : 0] : lane_left(w[N - 1]);
}

// x-fluxes of one component: a_h (w_{i+1} - w_i) less the one to the left,
// a_h the sum of b over the two columns (b = lambda + 2 mu or mu).
template <int N>
__device__ __forceinline__ void x_flux(const float (&b)[N], const float (&w)[N], float (&x)[N]) {
#pragma clang fp contract(off)
    float h[N], d[N], f[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        h[q] = right_of<N>(b, q) + b[q];
        d[q] = right_of<N>(w, q) - w[q];
        f[q] = h[q] * d[q];
    }
#pragma unroll
    for (int q = 0; q < N; ++q) x[q] = __builtin_fmaf(h[q], d[q], -left_of<N>(f, q));
}

// The surface row's acceleration (its mixed terms one-sided in depth).
// xu, xv: the x-fluxes; dn: D_x of row 1.
template <int N>
__device__ __forceinline__ void surface_accel(const NodeCoef<N>& cr, const NodeCoef<N>& cn,
                                              const Pt<N>& c, const Pt<N>& n, const Pt<N>& dn,
                                              const float (&xu)[N], const float (&xv)[N],
                                              float2 (&acc)[N]) {
#pragma clang fp contract(off)
    const Pt<N> dc = x_diff<N>(c);
    float p[N], z[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        p[q] = cr.lam[q] * (n.v[q] - c.v[q]);
        z[q] = cr.mu[q] * (n.u[q] - c.u[q]);
    }
#pragma unroll
    for (int q = 0; q < N; ++q) {
        float au = __builtin_fmaf(cr.mu[q] + cn.mu[q], n.u[q] - c.u[q], 0.5f * xu[q]);
        float av = __builtin_fmaf(cr.a[q] + cn.a[q], n.v[q] - c.v[q], 0.5f * xv[q]);
        au = __builtin_fmaf(0.5f,
                            (right_of<N>(p, q) - left_of<N>(p, q)) +
                                __builtin_fmaf(cr.mu[q], dc.v[q], cn.mu[q] * dn.v[q]),
                            au);
        av = __builtin_fmaf(0.5f,
                            __builtin_fmaf(cr.lam[q], dc.u[q], cn.lam[q] * dn.u[q]) +
                                (right_of<N>(z, q) - left_of<N>(z, q)),
                            av);
        acc[q] = make_float2(au, av);
    }
}

// Level j's row r off the plain path: the surface row's acceleration, the
// forcing, rows past the grid's (zero), and the receivers.
template <int K, int N, bool EDGE>
__device__ __forceinline__ void nodal_special(const StreamTile<K, N>& t, int j, int r, float h2,
                                              const NodeCoef<N>& cr, const NodeCoef<N>& cn,
                                              const float (&sc)[N], const Pt<N>& c, const Pt<N>& n,
                                              const Pt<N>& dn, const Pt<N>& up,
                                              const float (&xu)[N], const float (&xv)[N],
                                              float2 (&acc)[N], Pt<N>& nw) {
    if (r < 0 || r >= t.nz - 1) {
#pragma unroll
        for (int q = 0; q < N; ++q) nw.u[q] = nw.v[q] = 0.f;
        return;
    }
    const int col = lane_col(t);
    const int dk = r - t.sk0;
    const bool win = (unsigned)dk < (unsigned)kSrcW;
    if (r == 0 || win) {
        if (r == 0) surface_accel<N>(cr, cn, c, n, dn, xu, xv, acc);
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int di = col + q - t.si0;
            const bool src = win && (unsigned)di < (unsigned)kSrcW;
            float w0 = 0.f, w1 = 0.f;
            if (src) {
                const float* w = t.sw + dk * kSrcW + di;
                w0 = w[0];
                w1 = w[kSrcW * kSrcW];
            }
            const float2 w = nodal_new(acc[q], sc[q], c.u[q], c.v[q], up.u[q], up.v[q],
                                       src ? 2 : 0, h2, t.sw[kSwSeries + j - 1], w0, w1);
            nw.u[q] = w.x;
            nw.v[q] = w.y;
        }
        if constexpr (EDGE) zero_rigid<K, N>(t, nw);
    }
    if (r == 0 && t.m + j <= t.nsteps) record_row<K, N>(t, j, nw);
}

// One row of the pipeline, as in stream.hip.  S: the row's place in its trip;
// ci: lambda and mu of row i (loaded by the caller), cr1 / s1: of row i - 1,
// replaced by row i's for the next row.
template <int K, int N, bool EDGE, int S, int J>
__device__ __forceinline__ void nodal_level(const StreamTile<K, N>& t, NodalState<K, N>& s,
                                            const Ring<K, N>& ring, int i, bool plain, float h2,
                                            NodeCoef<N>& cn, NodeCoef<N>& next, float (&snext)[N],
                                            Pt<N>& n, Pt<N>& up) {
#pragma clang fp contract(off)
    const int r = i - J;
    NodeCoef<N> cr = next;
    float sr[N];
#pragma unroll
    for (int q = 0; q < N; ++q) sr[q] = snext[q];
    // the next level's row (or level 1's of the next row) while this one works
    constexpr int O = J < K ? S - (J + 1) : S;
    ring.template get<O>(next);
    ring.template get_s<O>(snext);
    __builtin_amdgcn_sched_barrier(0);
    set_a<N>(cr);
    const Pt<N> dn = x_diff<N>(n), c = s.c[J - 1], p = s.p[J - 1];
    const Pt<N> dc = x_diff<N>(c);
    Pt<N> sc, qn, nw;
    float xu[N], xv[N], pz[N], qz[N];
    x_flux<N>(cr.a, c.u, xu);
    x_flux<N>(cr.mu, c.v, xv);
#pragma unroll
    for (int q = 0; q < N; ++q) {
        sc.u[q] = cr.lam[q] * dc.u[q];
        sc.v[q] = cr.mu[q] * dc.v[q];
        pz[q] = cr.lam[q] * (n.v[q] - p.v[q]);
        qz[q] = cr.mu[q] * (n.u[q] - p.u[q]);
    }
    float2 acc[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const float mz = cr.mu[q] + cn.mu[q], az = cr.a[q] + cn.a[q];
        const float du = n.u[q] - c.u[q], dv = n.v[q] - c.v[q];
        float au = 0.5f * (xu[q] + __builtin_fmaf(mz, du, -s.q[J - 1].u[q]));
        float av = 0.5f * (xv[q] + __builtin_fmaf(az, dv, -s.q[J - 1].v[q]));
        qn.u[q] = mz * du;
        qn.v[q] = az * dv;
        au = __builtin_fmaf(0.25f,
                            (right_of<N>(pz, q) - left_of<N>(pz, q)) +
                                __builtin_fmaf(cn.mu[q], dn.v[q], -s.sp[J - 1].v[q]),
                            au);
        av = __builtin_fmaf(0.25f,
                            __builtin_fmaf(cn.lam[q], dn.u[q], -s.sp[J - 1].u[q]) +
                                (right_of<N>(qz, q) - left_of<N>(qz, q)),
                            av);
        acc[q] = make_float2(au, av);
        const float2 w = nodal_new(acc[q], sr[q], c.u[q], c.v[q], up.u[q], up.v[q], 0, 0.f, 0.f,
                                   0.f, 0.f);
        nw.u[q] = w.x;
        nw.v[q] = w.y;
    }
    if constexpr (EDGE) zero_rigid<K, N>(t, nw);
    if (__builtin_expect(!plain, 0))
        nodal_special<K, N, EDGE>(t, J, r, h2, cr, cn, sr, c, n, dn, up, xu, xv, acc, nw);
    if (J == K && (unsigned)(r - t.kb) < (unsigned)t.nstore && t.st_ok) {
        st_pt<N>(t.out1 + (size_t)r * t.pitch, t.col, c);
        st_pt<N>(t.out0 + (size_t)r * t.pitch, t.col, nw);
    }
    up = p;
    s.p[J - 1] = c;
    s.c[J - 1] = n;
    s.sp[J - 1] = sc;
    s.q[J - 1] = qn;
    cn = cr;
    n = nw;
    if constexpr (J < K)
        nodal_level<K, N, EDGE, S, J + 1>(t, s, ring, i, plain, h2, cn, next, snext, n, up);
}

// lambda, mu and s of a row of the medium's planes.
template <int N>
__device__ __forceinline__ void ld_coef(const float* row, size_t plane, int col, NodeCoef<N>& c,
                                        float (&s)[N]) {
    if constexpr (N == 2) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        const f2 l = *(const GAS f2*)((const GAS float*)row + col);
        const f2 m = *(const GAS f2*)((const GAS float*)row + plane + col);
        const f2 z = *(const GAS f2*)((const GAS float*)row + 2 * plane + col);
        c.lam[0] = l.x;
        c.lam[1] = l.y;
        c.mu[0] = m.x;
        c.mu[1] = m.y;
        s[0] = z.x;
        s[1] = z.y;
    } else {
        c.lam[0] = ld1(row, col);
        c.mu[0] = ld1(row, plane + col);
        s[0] = ld1(row, 2 * plane + col);
    }
}

template <int K, int N, bool EDGE>
__device__ __forceinline__ void nodal_strip(const StreamEntry& e, const float* sw, int* rec,
                                            float* mem) {
    StreamTile<K, N> t;
    tile_init<K, N>(t, e.d, e.m, e.pin, e.x0, e.kb, e.ke, sw, rec);
    const float h2 = e.d->h2;
    NodalState<K, N> s{};
    const int i0 = max(e.kb - K, 0), i1 = e.ke + K, nz = t.nz;
    const size_t plane = (size_t)nz * t.pitch;
    Ring<K, N> ring;
    ring.init(mem);
    // rows before the first: zero (their levels form nothing that is kept)
#pragma unroll
    for (int q = 0; q < kRingTrips<K> * kRingTrip / 64; ++q) mem[q * 64 + threadIdx.x] = 0.f;
    const float* crow = t.coef + (size_t)i0 * t.pitch;
    NodeCoef<N> cf[3];
    float sf[3][N];
#pragma unroll
    for (int q = 0; q < 3; ++q)
        ld_coef<N>(crow + (size_t)q * t.pitch, plane, t.col, cf[q], sf[q]);
    crow += (size_t)2 * t.pitch;
    RowFeed<N> f;
    f.init(e.d, e.pin, i0, t.col);
    NodeCoef<N> next{};
    float snext[N] = {};
    for (int i = i0; i < i1; i += 3) {
        NodeCoef<N> cn = cf[0];
        ring.template put<0>(cf[0], sf[0]);
        ring.template put<1>(cf[1], sf[1]);
        ring.template put<2>(cf[2], sf[2]);
#pragma unroll
        for (int q = 0; q < 3; ++q) {  // rows i + 3 .., held at the last one
            crow += i + 3 + q < nz ? t.pitch : 0;
            ld_coef<N>(crow, plane, t.col, cf[q], sf[q]);
        }
        auto row = [&](auto slot) {
            constexpr int S = decltype(slot)::value;
            if constexpr (S > 0) ring.template get<S>(cn);
            set_a<N>(cn);
            Pt<N> n = f.c[S], up = f.p[S];
            nodal_level<K, N, EDGE, S, 1>(t, s, ring, i + S, plain_row(t, i + S), h2, cn, next,
                                          snext, n, up);
            f.next(i + S, S);
        };
        row(std::integral_constant<int, 0>());
        row(std::integral_constant<int, 1>());
        row(std::integral_constant<int, 2>());
        ring.advance();
    }
}

template <int K>
__global__ void __launch_bounds__(64, 2)
stencil_nodal_stream(const SolveDesc* __restrict__ descs, const int2* __restrict__ tiles,
                     int ntiles, int pass, int rows) {
    __shared__ __attribute__((aligned(16))) float ring[kRingTrips<K> * kRingTrip];
    __shared__ float sw[kSwSeries + K];
    __shared__ int rec[128];
    const int b = xcd_block(blockIdx.x, gridDim.x);
    if (b >= ntiles) return;
    StreamEntry e;
    if (!stream_entry<K>(descs, tiles[b], pass, rows, e)) return;  // uniform
    load_forcing<K>(e.d, e.m, sw);
    __syncthreads();
    if (e.narrow)
        nodal_strip<K, 1, true>(e, sw, rec, ring);
    else if (e.x0 == 0 || e.x0 + 128 > e.d->nx - 1)
        nodal_strip<K, 2, true>(e, sw, rec, ring);
    else
        nodal_strip<K, 2, false>(e, sw, rec, ring);
}

}  // namespace

void launch_nodal_stream(const SolveDesc* descs, const int2* tiles, int ntiles, int pass,
                         int rows, hipStream_t s) {
    if (ntiles > 0)
        stencil_nodal_stream<kNodalStreamSteps><<<ntiles, 64, 0, s>>>(descs, tiles, ntiles, pass,
                                                                     rows);
}

}  // namespace eig
