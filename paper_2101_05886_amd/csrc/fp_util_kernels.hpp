// fp_util_kernels.hpp -- setup and utility kernels (metrics, periodic ghost
// copy, CFL limit, state check).  Included by fp_api.hip only.
#pragma once
#include "fp_kernels.hpp"

namespace fpk {

// ---------------------------------------------------------------------------
// symmetric conservative metrics (setup)
// ---------------------------------------------------------------------------

struct CGeoK {
    int gc;
    long csd[3];
    long cvol;
    long cbase;  // offset of node (0,0,0) in the coordinate arrays
};

// antisymmetric central first-derivative weights c_m, m = 1..Y/2:
// D f = sum_m c_m (f_{+m} - f_{-m})
template <int Y>
__device__ __forceinline__ double dcoef(int m) {
    if constexpr (Y == 2) {
        return 0.5;
    } else if constexpr (Y == 4) {
        return m == 1 ? 8.0 / 12.0 : -1.0 / 12.0;
    } else if constexpr (Y == 6) {
        return m == 1 ? 45.0 / 60.0 : (m == 2 ? -9.0 / 60.0 : 1.0 / 60.0);
    } else {
        return m == 1 ? 672.0 / 840.0 : (m == 2 ? -168.0 / 840.0 : (m == 3 ? 32.0 / 840.0 : -3.0 / 840.0));
    }
}

template <int Y>
struct Coord {
    const double* xyz;
    CGeoK C;
    __device__ __forceinline__ double X(int c, long off) const { return xyz[c * C.cvol + off]; }
    // derivative of coordinate c along axis e at the node with offset off
    __device__ __forceinline__ double D(int c, int e, long off) const {
        double s = 0.0;
#pragma unroll
        for (int m = 1; m <= Y / 2; ++m)
            s += dcoef<Y>(m) * (X(c, off + m * C.csd[e]) - X(c, off - m * C.csd[e]));
        return s;
    }
};

// Stores one computed node's metric v at (i, j, k) and at its periodic
// images in the ghost layers (every array of the layout is then complete:
// no fill pass).  A node within g of an end of a periodic axis has an image
// beyond the other end; an axis of fewer than 2 g nodes gives both.
struct MetPlace {
    unsigned off;  // the node
    unsigned img;  // per axis two bits: an image a period below, above
};
template <int DIM>
__device__ __forceinline__ MetPlace met_place(const GeoK& G, int i, int j, int k) {
    const int p[3] = {i, j, k};
    unsigned img = 0;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
        if (G.bc[d] != 0) continue;
        img |= (p[d] >= G.n[d] - G.g ? 1u : 0u) << (2 * d);
        img |= (p[d] < G.g ? 2u : 0u) << (2 * d);
    }
    return {(unsigned)(G.base + i + j * G.sd[1] + k * G.sd[2]), img};
}
__device__ __forceinline__ void met_put(const GeoK& G, double* a, const MetPlace& P, double x) {
    a[P.off] = x;
    if (P.img == 0) return;
    auto lo = [&](int d) { return P.img >> (2 * d) & 1 ? -1 : 0; };
    auto hi = [&](int d) { return P.img >> (2 * d) & 2 ? 1 : 0; };
    for (int c = lo(2); c <= hi(2); ++c)
        for (int b = lo(1); b <= hi(1); ++b)
            for (int e = lo(0); e <= hi(0); ++e)
                a[(long)P.off + e * G.n[0] + b * G.n[1] * G.sd[1] + c * G.n[2] * G.sd[2]] = x;
}
template <int DIM>
__device__ __forceinline__ void met_store(const GeoK& G, double* a, int i, int j, int k, double x) {
    met_put(G, a, met_place<DIM>(G, i, j, k), x);
}

// 2D metrics, one lane per node.  Bound by the cache's reads of the windows;
// latency is hidden by other waves, so registers count: a million nodes at
// orders 2, 4, 6 and 8 take 20, 48, 94 and 154 us with at most 112.  The order
// of the loads is held by the stores: with `met` declared __restrict__ the
// whole double sum of 1/J is loaded ahead, into all 512 registers and scratch
// at order 8 (20, 48, 116 and 265 us).
template <int Y>
__global__ __launch_bounds__(128) void k_metrics2(GeoK G, CGeoK C, const double* __restrict__ xyz,
                                                  double* met, int lo0, int lo1, int c0, int c1) {
    const long tid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= (long)c0 * c1) return;
    const int i = lo0 + (int)(tid % c0);
    const int j = lo1 + (int)(tid / c0);
    const Coord<Y> X{xyz, C};
    const long co = C.cbase + i + j * C.csd[1];
    const MetPlace P = met_place<2>(G, i, j, 0);
    met_put(G, met + 0 * G.vol, P, X.D(1, 1, co));
    met_put(G, met + 1 * G.vol, P, -X.D(0, 1, co));
    met_put(G, met + 2 * G.vol, P, -X.D(1, 0, co));
    met_put(G, met + 3 * G.vol, P, X.D(0, 0, co));
    // 1/J = 1/2 [ (x y_eta - y x_eta)_xi + (y x_xi - x y_xi)_eta ]
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int m = 1; m <= Y / 2; ++m) {
        const long p = co + m * C.csd[0], q = co - m * C.csd[0];
        a += dcoef<Y>(m) * ((X.X(0, p) * X.D(1, 1, p) - X.X(1, p) * X.D(0, 1, p)) -
                            (X.X(0, q) * X.D(1, 1, q) - X.X(1, q) * X.D(0, 1, q)));
        const long r = co + m * C.csd[1], s = co - m * C.csd[1];
        b += dcoef<Y>(m) * ((X.X(1, r) * X.D(0, 0, r) - X.X(0, r) * X.D(1, 0, r)) -
                            (X.X(1, s) * X.D(0, 0, s) - X.X(0, s) * X.D(1, 0, s)));
    }
    met_put(G, met + 4 * G.vol, P, 0.5 * (a + b));
}

// 3D metrics.  With (d, e, f) and (c, a, b) cyclic,
//   P_{c,e} = a_e b - a b_e            (the pairing of eq. JBabc),
//   s_{d,c} = 1/2 [ (P_{c,e})_f - (P_{c,f})_e ],
//   1/J     = 1/3 sum_d (x . s_d)_d    (eq. JB).
// The three derivatives of a term run along three different axes, so a node
// reaches the coordinates of the box of half width Y/2 around it and no
// further.  Evaluated node by node, each P and each s_d is recomputed by the
// Y, Y^2 neighbours that use it; here a workgroup owns a tile of nodes and
// forms every P_{c,e} and every x . s_d of its box once, in LDS, one
// component c at a time.  A thread forms four P, or four s_d, that follow one
// another along the axis of a difference, from one window of Y + 4 values in
// registers: LDS reads per value 5 and 8.5 instead of 14 and 12 at sixth
// order.  It keeps the same four nodes for all components, so their places
// are worked out once, and x . s_d adds up in registers.  The next component's
// box is loaded while this one's pairs are formed and written over the
// coordinates when they are done.  160 x 144 x 150, sixth order: 600 us with
// one difference per thread and place, 561 with the windows, 510 with the
// places worked out once, 475 with the loads ahead.  Bound by latency between
// the barriers (16 waves on a CU, LDS 45% and vector issue 45% busy); the
// tile is 16 nodes along i, for whole cache lines, and 4 x 4 across, which
// with 128 registers keeps two workgroups on a CU up to sixth order.
template <int Y>
struct MetTile {
    static constexpr int H = Y / 2, TI = 16, TJ = 4, TK = 4, THREADS = 512;
    static constexpr int BI = TI + Y, BJ = TJ + Y, BK = TK + Y;  // the box of the tile
    // P_{c,e}: the tile's extent along e, the box's along the other axes
    // (the rows of P0 are padded for the writes of four at a time)
    double P0[BK][BJ][TI + 2], P1[BK][TJ][BI], P2[TK][BJ][BI];
    union {
        alignas(16) double X[2][BK][BJ][BI];  // coordinates a, b of the box
        struct {  // in the end, x . s_d: the box's extent along d, the tile's along the other axes
            double S0[TK][TJ][BI], S1[TK][BJ][TI], S2[BK][TJ][TI];
        };
    };
};

// central difference along a stride (in doubles) at p
template <int Y>
__device__ __forceinline__ double met_diff(const double* p, int st) {
    double s = 0.0;
#pragma unroll
    for (int m = 1; m <= Y / 2; ++m) s += dcoef<Y>(m) * (p[m * st] - p[-m * st]);
    return s;
}

// quotient of a small number by a constant, in one full-rate product
template <unsigned D>
__device__ __forceinline__ unsigned met_div(unsigned t) {
    static_assert(D < 512, "exact for t < 2^20 / D");
    return __umul24(t, (1u << 20) / D + 1) >> 20;
}

// central difference from a window in registers, the node at p[Y/2]
template <int Y>
__device__ __forceinline__ double met_diff_reg(const double* p) {
    double s = 0.0;
#pragma unroll
    for (int m = 1; m <= Y / 2; ++m) s += dcoef<Y>(m) * (p[Y / 2 + m] - p[Y / 2 - m]);
    return s;
}

// The Y + 4 nodes that four consecutive differences along a stride reach
template <int Y, int ST>
__device__ __forceinline__ void met_window(const double* p, double w[Y + 4]) {
    if constexpr (ST == 1) {
#pragma unroll
        for (int m = 0; m < Y + 4; m += 2) {
            const double2 x = *reinterpret_cast<const double2*>(p + m);
            w[m] = x.x;
            w[m + 1] = x.y;
        }
    } else {
#pragma unroll
        for (int m = 0; m < Y + 4; ++m) w[m] = p[m * ST];
    }
}

template <int Y>
__global__ __launch_bounds__(MetTile<Y>::THREADS, 4) void k_metrics3(GeoK G, CGeoK C, const double* __restrict__ xyz,
                                                                  double* __restrict__ met, int lo0, int lo1,
                                                                  int lo2, int c0, int c1, int c2) {
    using M = MetTile<Y>;
    constexpr int H = M::H, TI = M::TI, TJ = M::TJ, TK = M::TK, BI = M::BI, BJ = M::BJ, BK = M::BK;
    constexpr int XJ = BI, XK = BI * BJ;  // strides of the box
    __shared__ M L;
    const unsigned nti = (unsigned)(c0 + TI - 1) / TI, ntj = (unsigned)(c1 + TJ - 1) / TJ;
    const unsigned tile = (unsigned)xcd_block(blockIdx.x, gridDim.x);
    // the tile's first node, counted from node (lo0, lo1, lo2)
    const int ti = (int)(tile % nti) * TI, tj = (int)(tile / nti % ntj) * TJ, tk = (int)(tile / nti / ntj) * TK;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = wave_id();
    static_assert(TI % 4 == 0 && TJ == 4 && TK == 4, "differences are formed four nodes at a time");
    // offset of box node (i, j, k) in a coordinate array, clamped to the
    // nodes that the computed nodes reach (tiles may hang over the end)
    const int e0 = c0 - 1 + Y - ti, e1 = c1 - 1 + Y - tj, e2 = c2 - 1 + Y - tk;
    const unsigned cs1 = (unsigned)C.csd[1], cs2 = (unsigned)C.csd[2];
    const unsigned cb = (unsigned)(C.cbase + (lo0 - H + ti) + (lo1 - H + tj) * C.csd[1] + (lo2 - H + tk) * C.csd[2]);
    auto coff = [&](int i, int j, int k) {
        return cb + (unsigned)min(i, e0) + (unsigned)min(j, e1) * cs1 + (unsigned)min(k, e2) * cs2;
    };
    // What does not depend on the component is worked out once: the nodes of
    // the box that this thread loads,
    constexpr int NB = BI * BJ * BK, NL = (NB + M::THREADS - 1) / M::THREADS;
    unsigned boff[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const unsigned t = (unsigned)min(tid + l * M::THREADS, NB - 1);
        const unsigned row = met_div<BI>(t), k = met_div<BI * BJ>(t);
        boff[l] = coff((int)(t - row * BI), (int)(row - k * BJ), (int)k);
    }
    // the runs of four P_{c,e} that it forms (waves 0 .. W0 - 1 those of
    // e = 0, the next W1 those of e = 1, the last W2 those of e = 2, and
    // round again),
    constexpr int N0 = BK * BJ * (TI / 4), N1 = BK * BI, N2 = BJ * BI;
    constexpr int W0 = (N0 + 63) / 64, W1 = (N1 + 63) / 64, W2 = (N2 + 63) / 64;
    constexpr int NW = M::THREADS / 64, NP = (W0 + W1 + W2 + NW - 1) / NW;
    unsigned psrc[NP], pdst[NP];  // ~0u: none
#pragma unroll
    for (int l = 0; l < NP; ++l) {
        const int w = wave + l * NW;
        const unsigned t = (unsigned)(w < W0 ? w : w < W0 + W1 ? w - W0 : w - W0 - W1) * 64 + lane;
        psrc[l] = pdst[l] = ~0u;
        if (w < W0) {
            const unsigned seg = met_div<BK * BJ>(t), row = t - seg * (BK * BJ);
            if (t < N0) psrc[l] = row * BI + seg * 4, pdst[l] = row * (TI + 2) + seg * 4;
        } else if (w < W0 + W1) {
            const unsigned k = met_div<BI>(t), i = t - k * BI;
            if (t < N1) psrc[l] = k * (BJ * BI) + i, pdst[l] = k * (TJ * BI) + i;
        } else if (t < N2) {
            psrc[l] = pdst[l] = t;
        }
    }
    // and the four s_{d,c} that it forms: waves 0 .. V0 - 1 those of d = 0,
    // at (s0, s1) of the task across k, the next V1 those of d = 1, across k,
    // the last V2 those of d = 2, across j
    constexpr int M0 = TJ * BI, M1 = BJ * TI, M2 = BK * TI;
    constexpr int V0 = (M0 + 63) / 64, V1 = (M1 + 63) / 64, V2 = (M2 + 63) / 64;
    static_assert(V0 + V1 + V2 <= M::THREADS / 64, "one task per wave");
    const int sd = wave < V0 ? 0 : wave < V0 + V1 ? 1 : wave < V0 + V1 + V2 ? 2 : 3;
    const unsigned st = (unsigned)tid - (sd == 0 ? 0u : sd == 1 ? V0 : V0 + V1) * 64;
    const int s1 = (int)(sd == 0 ? met_div<BI>(st) : st / TI), s0 = (int)(sd == 0 ? st - s1 * BI : st % TI);
    const bool mine = sd == 0 ? st < M0 : sd == 1 ? st < M1 : sd == 2 && st < M2;
    // the run starts at box node (b0, b1, b2), H along its axis
    const int b0 = sd == 0 ? s0 : s0 + H, b1 = sd == 0 ? s1 + H : sd == 1 ? s1 : H, b2 = sd == 2 ? s1 : H;
    const int ni = b0 - H, nj = b1 - H, nk = b2 - H;
    const bool own = mine && ni >= 0 && ni < min(TI, c0 - ti) && nj >= 0 && nj < min(TJ, c1 - tj) && nk >= 0 &&
                     nk < min(TK, c2 - tk);
    const MetPlace first = met_place<3>(G, lo0 + ti + ni, lo1 + tj + nj, lo2 + tk + nk);
    const int ra = sd == 2 ? 1 : 2;  // the run's axis; the rest of it in uniform registers
    const int er = ra == 1 ? e1 : e2, rn = (ra == 1 ? c1 - tj : c2 - tk), r0 = ra == 1 ? lo1 + tj : lo2 + tk;
    const unsigned csr = ra == 1 ? cs1 : cs2, gsr = (unsigned)G.sd[ra];
    auto place = [&](int m) {
        const unsigned img = G.bc[ra] != 0 ? 0u : (r0 + m >= G.n[ra] - G.g ? 1u : 0u) | (r0 + m < G.g ? 2u : 0u);
        return MetPlace{first.off + (unsigned)m * gsr, (first.img & ~(3u << (2 * ra))) | img << (2 * ra)};
    };
    unsigned xoff[4];
    double xs[4] = {0.0, 0.0, 0.0, 0.0};  // x . s_d, by component
    xoff[0] = mine ? coff(b0, b1, b2) : cb;
#pragma unroll
    for (int m = 1; m < 4; ++m) xoff[m] = xoff[m - 1] + (mine && H + m <= er ? csr : 0u);
    double va[NL], vb[NL];
    auto load_box = [&](int c) {  // coordinates a, b of component c
        const double* xa = xyz + (c == 2 ? 0 : c + 1) * C.cvol;
        const double* xb = xyz + (c == 0 ? 2 : c - 1) * C.cvol;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            va[l] = xa[boff[l]];
            vb[l] = xb[boff[l]];
        }
    };
    auto fill_box = [&] {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int t = min(tid + l * M::THREADS, NB - 1);
            (&L.X[0][0][0][0])[t] = va[l];
            (&L.X[1][0][0][0])[t] = vb[l];
        }
    };
    load_box(0);
    fill_box();
    __syncthreads();
#pragma unroll 1
    for (int c = 0; c < 3; ++c) {
        // the next component's box is on its way while this one's pairs are
        // formed, and takes the place of the coordinates that they have read
        if (c < 2) load_box(c + 1);
        const double* xc = xyz + c * C.cvol;
        double x[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) x[m] = xc[xoff[m]];
        // P_{c,e} of four nodes along e from their windows, at src of the box
        auto pairs = [&](auto stride, unsigned src, double* out, int ost) {
            double wa[Y + 4], wb[Y + 4];
            met_window<Y, decltype(stride)::value>(&L.X[0][0][0][0] + src, wa);
            met_window<Y, decltype(stride)::value>(&L.X[1][0][0][0] + src, wb);
#pragma unroll
            for (int m = 0; m < 4; ++m)
                out[m * ost] = met_diff_reg<Y>(wa + m) * wb[H + m] - wa[H + m] * met_diff_reg<Y>(wb + m);
        };
#pragma unroll
        for (int l = 0; l < NP; ++l) {
            const int w = wave + l * NW;
            if (psrc[l] == ~0u) continue;
            if (w < W0)
                pairs(std::integral_constant<int, 1>(), psrc[l], &L.P0[0][0][0] + pdst[l], 1);
            else if (w < W0 + W1)
                pairs(std::integral_constant<int, XJ>(), psrc[l], &L.P1[0][0][0] + pdst[l], BI);
            else
                pairs(std::integral_constant<int, XK>(), psrc[l], &L.P2[0][0][0] + pdst[l], BJ * BI);
        }
        __syncthreads();
        if (c < 2) fill_box();
        // s_{d,c} on the box's extent along d: its part of x . s_d, and the
        // tile's own nodes to memory
        auto put = [&](int m, double s) {
            xs[m] = c == 0 ? x[m] * s : xs[m] + x[m] * s;
            if (own && m < rn) met_put(G, met + (3 * sd + c) * G.vol, place(m), s);
        };
        double win[Y + 4];
        if (mine && sd == 0) {  // (P_{c,1})_2 - (P_{c,2})_1
            met_window<Y, TJ * BI>(&L.P1[0][s1][s0], win);
#pragma unroll
            for (int m = 0; m < 4; ++m)
                put(m, 0.5 * (met_diff_reg<Y>(win + m) - met_diff<Y>(&L.P2[m][s1 + H][s0], BI)));
        } else if (mine && sd == 1) {  // (P_{c,2})_0 - (P_{c,0})_2
            met_window<Y, BJ * (TI + 2)>(&L.P0[0][s1][s0], win);
#pragma unroll
            for (int m = 0; m < 4; ++m)
                put(m, 0.5 * (met_diff<Y>(&L.P2[m][s1][s0 + H], 1) - met_diff_reg<Y>(win + m)));
        } else if (mine) {  // (P_{c,0})_1 - (P_{c,1})_0
            met_window<Y, TI + 2>(&L.P0[s1][0][s0], win);
#pragma unroll
            for (int m = 0; m < 4; ++m)
                put(m, 0.5 * (met_diff_reg<Y>(win + m) - met_diff<Y>(&L.P1[s1][m][s0 + H], 1)));
        }
        __syncthreads();
    }
    if (mine) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            if (sd == 0)
                L.S0[m][s1][s0] = xs[m];
            else if (sd == 1)
                L.S1[m][s1][s0] = xs[m];
            else
                L.S2[s1][m][s0] = xs[m];
        }
    }
    __syncthreads();
    for (int t = tid; t < TK * TJ * TI; t += M::THREADS) {
        const int i = t % TI, j = t / TI % TJ, k = t / (TI * TJ);
        if (ti + i >= c0 || tj + j >= c1 || tk + k >= c2) continue;
        const double J = met_diff<Y>(&L.S0[k][j][i + H], 1) + met_diff<Y>(&L.S1[k][j + H][i], TI) +
                         met_diff<Y>(&L.S2[k + H][j][i], TJ * TI);
        met_store<3>(G, met + 9 * G.vol, lo0 + ti + i, lo1 + tj + j, lo2 + tk + k, J / 3.0);
    }
}
template <int Y>
inline long met_tiles(const int c[3]) {
    using M = MetTile<Y>;
    return (long)((c[0] + M::TI - 1) / M::TI) * ((c[1] + M::TJ - 1) / M::TJ) * ((c[2] + M::TK - 1) / M::TK);
}

// Nodes of the ghost slabs of the frozen axes: for each frozen axis d, the
// g layers on each side along d with the other coordinates interior (the
// only ghost nodes the sweeps read).
__host__ __device__ inline long frozen_slab_nodes(const GeoK& G, int ndim) {
    long tot = 0;
    for (int d = 0; d < ndim; ++d) {
        if (G.bc[d] == 0) continue;
        long c = 2L * G.g;
        for (int e = 0; e < ndim; ++e)
            if (e != d) c *= G.n[e];
        tot += c;
    }
    return tot;
}

// Copies slab node t (0 <= t < frozen_slab_nodes) of src into dst1 and dst2:
// the RK3 drivers give their stage registers the caller's boundary values.
__device__ __forceinline__ void frozen_ghost_node(const GeoK& G, int ndim, int nvar, const double* src,
                                                  double* dst1, double* dst2, long t) {
    for (int d = 0; d < ndim; ++d) {
        if (G.bc[d] == 0) continue;
        long c = 2L * G.g;
        for (int e = 0; e < ndim; ++e)
            if (e != d) c *= G.n[e];
        if (t >= c) {
            t -= c;
            continue;
        }
        // the layer ad (both sides) and the transverse indices c1 (axis e1),
        // c2 (axis e2, 3D): consecutive lanes take nodes consecutive in
        // memory, along the layers for the slabs of the i axis, along i else
        const int e1 = d == 0 ? 1 : 0, e2 = d == 2 ? 1 : 2;
        int ad;
        long c1, c2;
        if (d == 0) {
            ad = (int)(t % (2 * G.g));
            c1 = (t / (2 * G.g)) % G.n[e1];
            c2 = (t / (2 * G.g)) / G.n[e1];
        } else {
            c1 = t % G.n[e1];
            ad = (int)((t / G.n[e1]) % (2 * G.g));
            c2 = (t / G.n[e1]) / (2 * G.g);
        }
        long off = G.base + (long)(ad < G.g ? ad - G.g : G.n[d] + ad - G.g) * G.sd[d] + c1 * G.sd[e1];
        if (ndim == 3) off += c2 * G.sd[e2];
        for (int v = 0; v < nvar; ++v) {
            const double x = gmem(src)[v * G.vol + off];
            gmem(dst1)[v * G.vol + off] = x;
            gmem(dst2)[v * G.vol + off] = x;
        }
        return;
    }
}

__global__ __launch_bounds__(256) void k_frozen_ghosts(GeoK G, int ndim, int nvar,
                                                       const double* __restrict__ src,
                                                       double* __restrict__ dst1,
                                                       double* __restrict__ dst2) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < frozen_slab_nodes(G, ndim)) frozen_ghost_node(G, ndim, nvar, src, dst1, dst2, t);
}

// Batched form: one item = 256 slab nodes of one block.
__global__ __launch_bounds__(256) void kb_frozen_ghosts(const int* __restrict__ t_nblk,
                                                        const long* __restrict__ t_start,
                                                        const BBlock* __restrict__ t_blk, int cap, int ndim) {
    const int nblk = *t_nblk;
    const long* __restrict__ st = t_start + BK_GHOST * (cap + 1);
    const long total = st[nblk];
    const int* __restrict__ ord = kind_order(t_start, cap, BK_GHOST);
    int b = blockIdx.x < total ? find_block(st, nblk, blockIdx.x) : 0;
    for (long item = blockIdx.x; item < total; item += gridDim.x) {
        b = advance_block(st, nblk, b, item);
        const BBlock& B = t_blk[ord[b]];
        const long node = (item - st[b]) * 256 + threadIdx.x;
        if (node < frozen_slab_nodes(B.G, ndim))
            frozen_ghost_node(B.G, ndim, ndim + 2, B.q, B.A, B.B, node);
    }
}

// Interface exchange: for every link, the g ghost layers of block a on its
// side are copied from the interior layers of block b next to the opposite
// side.  which = 0, 1, 2: the state registers of RK stage 1 (q), 2 (A),
// 3 (B); which = 3: the metric arrays.  Node t of all links' ghost slabs
// (prefix sums lstart) per thread, its link found by binary search.  Within
// a slab consecutive lanes take nodes consecutive in memory: along the layer
// for a face of the i axis, along i for the other faces.
__global__ __launch_bounds__(256) void kb_halo(const int* __restrict__ t_nlink,
                                               const long* __restrict__ t_lstart,
                                               const LinkK* __restrict__ t_links,
                                               const BBlock* __restrict__ t_blk, int ndim, int which) {
    const int nl = *t_nlink;
    const long total = t_lstart[nl];
    for (long t = (long)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (long)gridDim.x * blockDim.x) {
        // the link of node t: the last li with lstart[li] <= t (binary search)
        int li = 0, hi = nl - 1;
        while (li < hi) {
            const int mid = (li + hi + 1) >> 1;
            if (t_lstart[mid] <= t)
                li = mid;
            else
                hi = mid - 1;
        }
        const LinkK L = t_links[li];
        const BBlock& A = t_blk[L.a];
        const BBlock& B = t_blk[L.b];
        const int g = A.G.g;
        // the transverse axes e1 < e2 (e2 = 2 only in 3D), then the node's
        // layer l and transverse indices c1, c2
        const int e1 = L.axis == 0 ? 1 : 0, e2 = L.axis == 2 ? 1 : 2;
        const long u = t - t_lstart[li];
        long c1, c2;
        int l;
        if (L.axis == 0) {
            l = (int)(u % g);
            c1 = (u / g) % A.G.n[e1];
            c2 = (u / g) / A.G.n[e1];
        } else {
            c1 = u % A.G.n[e1];
            l = (int)((u / A.G.n[e1]) % g);
            c2 = (u / A.G.n[e1]) / g;
        }
        long oa = A.G.base + c1 * A.G.sd[e1], ob = B.G.base + c1 * B.G.sd[e1];
        if (ndim == 3) {
            oa += c2 * A.G.sd[e2];
            ob += c2 * B.G.sd[e2];
        }
        const int ia = L.side ? A.G.n[L.axis] + l : -1 - l;
        const int ib = L.side ? l : B.G.n[L.axis] - 1 - l;
        oa += (long)ia * A.G.sd[L.axis];
        ob += (long)ib * B.G.sd[L.axis];
        if (which == 3) {
            gdouble* dst = gmem(const_cast<double*>(A.met));
            const int nmet = ndim == 3 ? 10 : 5;
            for (int v = 0; v < nmet; ++v) dst[v * A.G.vol + oa] = gmem(B.met)[v * B.G.vol + ob];
        } else {
            gdouble* dst = gmem(which == 0 ? A.q : (which == 1 ? A.A : A.B));
            const gdouble* src = gmem(which == 0 ? B.q : (which == 1 ? B.A : B.B));
            for (int v = 0; v < ndim + 2; ++v) dst[v * A.G.vol + oa] = src[v * B.G.vol + ob];
        }
    }
}

// ---------------------------------------------------------------------------
// boundary faces
// ---------------------------------------------------------------------------

struct BcK {
    int kind[3][2];  // 0 hold, 1 extrapolate, 2 slip wall, 3 moving planar shock
    const unsigned char* mask[3][2];
    const double* nodes;
    double pre[5], post[5];
    double normal[3];
    double offset, speed;
};

// ghost nodes (boundary nodes x layers) of face (a, side)
__device__ __host__ __forceinline__ long bc_face_nodes(const GeoK& G, int a) {
    const int e1 = a == 0 ? 1 : 0, e2 = a == 2 ? 1 : 2;
    return (long)G.n[e1] * G.n[e2] * G.g;
}

// Ghost node tt (boundary node fastest, then layer l = 1..g) of face
// (a, side) at time t: extrapolation copies the boundary node; the slip wall
// takes the mirror node l (from the boundary) with the momentum's component
// along the boundary node's unit metric vector of axis a reversed; the shock
// sets post or pre by the side of the moving plane. Masked nodes are left.
template <int DIM>
__device__ void apply_bc_node(const GeoK& G, const BcK& bc, int a, int side, const double* __restrict__ met,
                              double* __restrict__ q, double t, long tt) {
    constexpr int NV = DIM + 2, E = NV - 1;
    const int e1 = a == 0 ? 1 : 0, e2 = a == 2 ? 1 : 2;
    const long n1 = G.n[e1];
    const int g = G.g, kind = bc.kind[a][side], nb = G.n[a];
    const unsigned char* mask = bc.mask[a][side];
    const long sa = G.sd[a];
    const long i1 = tt % n1, r = tt / n1;
    const int l = (int)(r % g) + 1;
    const long i2 = r / g;
    if (mask && !mask[i2 * n1 + i1]) return;
    const long line = G.base + i1 * G.sd[e1] + i2 * G.sd[e2];
    const long og = line + (long)(side ? nb - 1 + l : -l) * sa;
    double Q[NV];
    if (kind == 1) {
        const long os = line + (long)(side ? nb - 1 : 0) * sa;
#pragma unroll
        for (int v = 0; v < NV; ++v) Q[v] = q[v * G.vol + os];
    } else if (kind == 2) {
        const long ob = line + (long)(side ? nb - 1 : 0) * sa;
        double nw[DIM], nn = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            nw[c] = met[(a * DIM + c) * G.vol + ob];
            nn += nw[c] * nw[c];
        }
        nn = sqrt(nn);
#pragma unroll
        for (int c = 0; c < DIM; ++c) nw[c] /= nn;
        const long os = line + (long)(side ? nb - 1 - l : l) * sa;
        double un = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) un += nw[c] * q[(1 + c) * G.vol + os];
        Q[0] = q[os];
#pragma unroll
        for (int c = 0; c < DIM; ++c) Q[1 + c] = q[(1 + c) * G.vol + os] - 2.0 * un * nw[c];
        Q[E] = q[E * G.vol + os];
    } else {
        double xn = 0.0;
#pragma unroll
        for (int c = 0; c < DIM; ++c) xn += bc.normal[c] * bc.nodes[c * G.vol + og];
        const bool behind = xn < bc.offset + bc.speed * t;
#pragma unroll
        for (int v = 0; v < NV; ++v) Q[v] = behind ? bc.post[v] : bc.pre[v];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) q[v * G.vol + og] = Q[v];
}

// The ghost layers of every face whose kind is not hold, in one launch at
// time t (or *tdev + t when the time lives on the device, as in a captured
// step): the ghost nodes of those faces (axis-major, low side first) are
// numbered one after another, one thread per ghost node.
template <int DIM>
__global__ __launch_bounds__(256) void k_bc_face(GeoK G, BcK bc, const double* __restrict__ met,
                                                  double* __restrict__ q, double t,
                                                  const double* __restrict__ tdev) {
    if (tdev) t += *tdev;
    long total = 0;
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int side = 0; side < 2; ++side)
            if (bc.kind[a][side]) total += bc_face_nodes(G, a);
    for (long u = (long)blockIdx.x * blockDim.x + threadIdx.x; u < total; u += (long)gridDim.x * blockDim.x) {
        // the face of ghost node u
        int a = 0, side = 0;
        long tt = u;
        for (int fi = 0; fi < 2 * DIM; ++fi) {
            const int fa = fi >> 1, fs = fi & 1;
            if (!bc.kind[fa][fs]) continue;
            const long cnt = bc_face_nodes(G, fa);
            if (tt < cnt) {
                a = fa;
                side = fs;
                break;
            }
            tt -= cnt;
        }
        apply_bc_node<DIM>(G, bc, a, side, met, q, t, tt);
    }
}

__global__ void k_time_set(double* T, double t0) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        T[0] = t0;
        T[1] = t0;
        T[2] = 0.0;
    }
}
__global__ void k_time_advance(double* T, double dt) {
    if (threadIdx.x == 0 && blockIdx.x == 0) time_advance(T, dt);
}

// ---------------------------------------------------------------------------
// viscous fluxes (periodic axes): node fluxes, then their central difference
// ---------------------------------------------------------------------------

// The node of this thread in the viscous kernels: a workgroup of 256 takes
// 64 (i) x 4 (j) nodes of one plane k.  The grid is cut into pencils of
// 64 x 32 nodes along k; within a pencil the workgroups run through its
// eight row groups fastest, then k, and each XCD takes a contiguous range of
// pencils (xcd_block).  A node's neighbours along the second and third axes
// then lie in the rows and planes its XCD read moments before (about 0.7 MB
// of L2 back): in plane order, every such neighbour three planes away was an
// L2 miss, and with one 64 x 4 column per k-run the row neighbours were.
constexpr int kViscRows = 4, kViscPencil = 8;  // rows per workgroup, row groups per pencil
__device__ __forceinline__ bool visc_node(const GeoK& G, int (&idx)[3]) {
    const unsigned L = (unsigned)xcd_block(blockIdx.x, gridDim.x);
    const unsigned nk = (unsigned)G.n[2], nit = ((unsigned)G.n[0] + 63u) / 64u;
    const unsigned r = L / kViscPencil, r2 = r / nk;
    idx[2] = (int)(r % nk);
    idx[0] = (int)((r2 % nit) * 64u + (threadIdx.x & 63u));
    idx[1] = (int)(((r2 / nit) * kViscPencil + L % kViscPencil) * kViscRows + (threadIdx.x >> 6));
    return idx[0] < G.n[0] && idx[1] < G.n[1];
}
inline long visc_blocks(const int n[3]) {
    const int pj = kViscRows * kViscPencil;
    return (long)((n[0] + 63) / 64) * ((n[1] + pj - 1) / pj) * kViscPencil * n[2];
}

// sixth-order central first derivative, offsets 1..3 (antisymmetric)
__device__ __forceinline__ double d6w(int o) { return o == 1 ? 45.0 / 60.0 : (o == 2 ? -9.0 / 60.0 : 1.0 / 60.0); }

// interior node `off` shifted by s along axis d with the periodic wrap
__device__ __forceinline__ long wrap_node(const GeoK& G, long off, int idx, int d, int s) {
    int t = idx + s;
    t = t < 0 ? t + G.n[d] : (t >= G.n[d] ? t - G.n[d] : t);
    return off + (long)(t - idx) * G.sd[d];
}

// primitives (u_1 .. u_DIM, T = p / rho) of node o
template <int DIM>
__device__ __forceinline__ void visc_prim(const double* __restrict__ q, long vol, long o, double gm1,
                                          double (&w)[DIM + 1]) {
    const double rho = q[o];
    const double ir = drcp(rho);
    double k2 = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        const double m = q[(1 + c) * vol + o];
        w[c] = m * ir;
        k2 += m * w[c];
    }
    w[DIM] = gm1 * (q[(DIM + 1) * vol + o] - 0.5 * k2) * ir;
}

// The contravariant viscous fluxes at node o from the sixth-order
// differences dphi[d][a] = D6_d(phi_a) of the primitives phi = (u, T) along
// every direction and the node's own primitives w: gradients by the chain
// rule dphi/dx_j = (1/V) sum_d s_{d,j} D6_d(phi), tau_ij = mu (du_i/dx_j +
// du_j/dx_i - 2/3 delta_ij div u), the physical fluxes (tau_1j .. tau_nj,
// u_i tau_ij + kappa dT/dx_j) and Fv~_d = sum_j s_{d,j} Fv_j.  fv: [DIM
// directions][DIM + 1 components] arrays in the state layout (the mass
// component, zero, is not stored).  m: the node's metrics, 1/J last.
template <int DIM>
__device__ __forceinline__ void visc_node_fluxes(const GeoK& G, double mu, double kappa,
                                                 const double (&m)[DIM * DIM + 1], long o,
                                                 const double (&dphi)[DIM][DIM + 1], const double (&w)[DIM + 1],
                                                 double* __restrict__ fv) {
    constexpr int NP = DIM + 1;
    const double iV = drcp(m[DIM * DIM]);
    double grad[NP][DIM];
#pragma unroll
    for (int a = 0; a < NP; ++a)
#pragma unroll
        for (int j = 0; j < DIM; ++j) grad[a][j] = 0.0;
#pragma unroll
    for (int d = 0; d < DIM; ++d)
#pragma unroll
        for (int j = 0; j < DIM; ++j) {
            const double sdj = m[d * DIM + j] * iV;
#pragma unroll
            for (int a = 0; a < NP; ++a) grad[a][j] += sdj * dphi[d][a];
        }
    double div = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) div += grad[c][c];
    double F[DIM][NP];  // physical fluxes Fv_j, components 1..DIM+1
#pragma unroll
    for (int j = 0; j < DIM; ++j) {
        double work = 0.0;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const double tau = mu * (grad[a][j] + grad[j][a] - (a == j ? 2.0 / 3.0 * div : 0.0));
            F[j][a] = tau;
            work += w[a] * tau;
        }
        F[j][DIM] = work + kappa * grad[DIM][j];
    }
#pragma unroll
    for (int d = 0; d < DIM; ++d)
#pragma unroll
        for (int v = 0; v < NP; ++v) {
            double sum = 0.0;
#pragma unroll
            for (int j = 0; j < DIM; ++j) sum += m[d * DIM + j] * F[j][v];
            fv[(d * NP + v) * G.vol + o] = sum;
        }
}

// The viscous node fluxes of a 2D block, one lane per node: the primitives
// of the stencil neighbours are gathered along each direction.
template <int DIM>
__global__ __launch_bounds__(256) void k_visc_flux(GeoK G, double gamma, double mu, double kappa,
                                                    const double* __restrict__ met,
                                                    const double* __restrict__ q, double* __restrict__ fv) {
    constexpr int NP = DIM + 1;
    int idx[3];
    if (!visc_node(G, idx)) return;
    const long o = G.base + idx[0] + idx[1] * G.sd[1] + (long)idx[2] * G.sd[2];
    const double gm1 = gamma - 1.0;
    double dphi[DIM][NP];
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
#pragma unroll
        for (int a = 0; a < NP; ++a) dphi[d][a] = 0.0;
#pragma unroll
        for (int s = 1; s <= 3; ++s) {
            double wp[NP], wm[NP];
            visc_prim<DIM>(q, G.vol, wrap_node(G, o, idx[d], d, s), gm1, wp);
            visc_prim<DIM>(q, G.vol, wrap_node(G, o, idx[d], d, -s), gm1, wm);
#pragma unroll
            for (int a = 0; a < NP; ++a) dphi[d][a] += d6w(s) * (wp[a] - wm[a]);
        }
    }
    double w[NP];
    visc_prim<DIM>(q, G.vol, o, gm1, w);
    double m[DIM * DIM + 1];
#pragma unroll
    for (int c = 0; c <= DIM * DIM; ++c) m[c] = met[c * G.vol + o];
    visc_node_fluxes<DIM>(G, mu, kappa, m, o, dphi, w, fv);
}

// R = sum_d D6_d(Fv~_d) at every interior node of a 2D block (the mass
// component 0), one lane per node: the viscous part of the residual
// accumulator, before the inviscid sweeps subtract their flux differences.
template <int DIM>
__global__ __launch_bounds__(256) void k_visc_div(GeoK G, const double* __restrict__ fv, double* __restrict__ R) {
    constexpr int NP = DIM + 1;
    int idx[3];
    if (!visc_node(G, idx)) return;
    const long o = G.base + idx[0] + idx[1] * G.sd[1] + (long)idx[2] * G.sd[2];
    double acc[NP];
#pragma unroll
    for (int v = 0; v < NP; ++v) acc[v] = 0.0;
#pragma unroll
    for (int d = 0; d < DIM; ++d)
#pragma unroll
        for (int s = 1; s <= 3; ++s) {
            const long op = wrap_node(G, o, idx[d], d, s), om = wrap_node(G, o, idx[d], d, -s);
#pragma unroll
            for (int v = 0; v < NP; ++v)
                acc[v] += d6w(s) * (fv[(d * NP + v) * G.vol + op] - fv[(d * NP + v) * G.vol + om]);
        }
    R[o] = 0.0;
#pragma unroll
    for (int v = 0; v < NP; ++v) R[(1 + v) * G.vol + o] = acc[v];
}

// 3D blocks: a workgroup (one lane per column) owns a kVmI (i) x kVmJ (j)
// tile of columns and a run of planes, and marches along k.  Each lane keeps
// the seven planes k-3 .. k+3 of its own column in registers (the zeta
// differences) and per plane the tile with a halo of three nodes in i and j
// is staged in LDS (the xi and eta differences): the tile from the lanes'
// registers, the halo by one load per lane at most.  Everything a plane needs
// from memory is asked for a plane ahead, and the LDS plane is double
// buffered, so that one barrier a plane is all that waits.  All axes are
// periodic, so every index wraps; lanes past the grid's edge load wrapped
// nodes and store nothing.
// Bound by HBM: 352 algorithmic bytes per node.  The tile is 32 x 16: half
// the halo of 64 x 8 and, with 160 nodes, no idle lanes.  Runs of 16 planes
// (six more fill the registers) give a 160^3 block 800 workgroups; 32 planes
// left a workgroup per CU.  160^3: fluxes 227 us, divergence 157,
// against 329 and 200 with the halo and the tile loaded again from memory,
// two barriers a plane, and no load ahead.
constexpr int kVmI = 32, kVmJ = 16, kVmK = 16, kVmHI = kVmI + 6, kVmHJ = kVmJ + 6, kVmT = kVmI * kVmJ;
inline long visc_march_blocks(const int n[3]) {
    return (long)((n[0] + kVmI - 1) / kVmI) * ((n[1] + kVmJ - 1) / kVmJ) * ((n[2] + kVmK - 1) / kVmK);
}
struct VmTile {
    int i0, j0, k0, k1;  // tile origin, planes [k0, k1)
    int i, j;            // this lane's column (wrapped into the grid)
    bool mine;           // the column is a node of the grid
};
__device__ __forceinline__ int wrapi(int t, int n) { return t < 0 ? t + n : (t >= n ? t - n : t); }
__device__ __forceinline__ VmTile vm_tile(const GeoK& G) {
    const unsigned L = (unsigned)xcd_block(blockIdx.x, gridDim.x);
    const unsigned nit = ((unsigned)G.n[0] + kVmI - 1) / kVmI, njt = ((unsigned)G.n[1] + kVmJ - 1) / kVmJ;
    VmTile t;
    t.i0 = (int)(L % nit) * kVmI;
    t.j0 = (int)((L / nit) % njt) * kVmJ;
    t.k0 = (int)(L / (nit * njt)) * kVmK;
    t.k1 = min(t.k0 + kVmK, G.n[2]);
    const int i = t.i0 + (int)(threadIdx.x % kVmI), j = t.j0 + (int)(threadIdx.x / kVmI);
    t.mine = i < G.n[0] && j < G.n[1];
    t.i = i % G.n[0];
    t.j = j % G.n[1];
    return t;
}
// the halo entry e (0 .. kVmHalo - 1) of the tile: columns left and right of
// it, then rows below and above (with the corners, which the fluxes' and the
// divergence's differences do not read, left out): entry (hi, hj) of the
// kVmHI x kVmHJ box
constexpr int kVmHalo = 6 * kVmJ + 6 * kVmI;
static_assert(kVmHalo <= kVmT, "one halo entry per lane");
__device__ __forceinline__ void vm_halo(int e, int& hi, int& hj) {
    if (e < 6 * kVmJ) {
        hi = e % 6;
        hj = 3 + e / 6;
        if (hi >= 3) hi += kVmI;
    } else {
        e -= 6 * kVmJ;
        hi = 3 + e % kVmI;
        hj = e / kVmI;
        if (hj >= 3) hj += kVmJ;
    }
}
// element offset of node (i, j, k)
__device__ __forceinline__ unsigned vm_off(const GeoK& G, int i, int j, int k) {
    return (unsigned)(G.base + i + (long)j * G.sd[1] + (long)k * G.sd[2]);
}

__global__ __launch_bounds__(kVmT) void k_visc_flux3(GeoK G, double gamma, double mu, double kappa,
                                                     const double* __restrict__ met,
                                                     const double* __restrict__ q, double* __restrict__ fv) {
    __shared__ double L[2][4][kVmHJ][kVmHI];  // primitives of plane k, tile and halo
    const VmTile t = vm_tile(G);
    const double gm1 = gamma - 1.0;
    const int li = (int)(threadIdx.x % kVmI) + 3, lj = (int)(threadIdx.x / kVmI) + 3;
    const bool halo = (int)threadIdx.x < kVmHalo;
    int hi = 0, hj = 0;
    if (halo) vm_halo((int)threadIdx.x, hi, hj);
    const unsigned col = vm_off(G, t.i, t.j, 0);
    const unsigned hcol =
        vm_off(G, (t.i0 - 3 + hi + 2 * G.n[0]) % G.n[0], (t.j0 - 3 + hj + 2 * G.n[1]) % G.n[1], 0);
    const unsigned sk = (unsigned)G.sd[2];
    auto load = [&](unsigned o, double (&v)[5]) {
#pragma unroll
        for (int c = 0; c < 5; ++c) v[c] = q[c * G.vol + o];
    };
    // (u, T) of a node from its conserved state
    auto prim = [&](const double (&v)[5], double (&w)[4]) {
        const double ir = drcp(v[0]);
        double k2 = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            w[c] = v[1 + c] * ir;
            k2 += v[1 + c] * w[c];
        }
        w[3] = gm1 * (v[4] - 0.5 * k2) * ir;
    };
    double P[7][4];  // this column's primitives at planes k-3 .. k+3
    double qc[5], qh[5];
#pragma unroll
    for (int r = 0; r < 6; ++r) {
        load(col + (unsigned)wrapi(t.k0 - 3 + r, G.n[2]) * sk, qc);
        prim(qc, P[r]);
    }
    load(col + (unsigned)wrapi(t.k0 + 3, G.n[2]) * sk, qc);
    if (halo) load(hcol + (unsigned)t.k0 * sk, qh);
    for (int k = t.k0; k < t.k1; ++k) {
        double(*Lk)[kVmHJ][kVmHI] = L[(k - t.k0) & 1];
        prim(qc, P[6]);
#pragma unroll
        for (int a = 0; a < 4; ++a) Lk[a][lj][li] = P[3][a];
        if (halo) {
            double w[4];
            prim(qh, w);
#pragma unroll
            for (int a = 0; a < 4; ++a) Lk[a][hj][hi] = w[a];
        }
        if (k + 1 < t.k1) {
            load(col + (unsigned)wrapi(k + 4, G.n[2]) * sk, qc);
            if (halo) load(hcol + (unsigned)(k + 1) * sk, qh);
        }
        const unsigned o = col + (unsigned)k * sk;
        double m[10];
#pragma unroll
        for (int c = 0; c < 10; ++c) m[c] = met[c * G.vol + o];
        // one barrier a plane: a lane overwrites this buffer two planes on,
        // past the next plane's barrier, which every lane reaches only after
        // its reads of this plane
        lds_barrier();
        double dphi[3][4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            dphi[0][a] = 0.0;
            dphi[1][a] = 0.0;
            dphi[2][a] = 0.0;
#pragma unroll
            for (int s = 1; s <= 3; ++s) {
                dphi[0][a] += d6w(s) * (Lk[a][lj][li + s] - Lk[a][lj][li - s]);
                dphi[1][a] += d6w(s) * (Lk[a][lj + s][li] - Lk[a][lj - s][li]);
                dphi[2][a] += d6w(s) * (P[3 + s][a] - P[3 - s][a]);
            }
        }
        if (t.mine) visc_node_fluxes<3>(G, mu, kappa, m, o, dphi, P[3], fv);
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int a = 0; a < 4; ++a) P[r][a] = P[r + 1][a];
    }
}

__global__ __launch_bounds__(kVmT) void k_visc_div3(GeoK G, const double* __restrict__ fv, double* __restrict__ R) {
    __shared__ double Lx[2][4][kVmJ][kVmHI];  // Fv~_xi of plane k: tile rows, halo in i
    __shared__ double Ly[2][4][kVmHJ][kVmI];  // Fv~_eta of plane k: tile columns, halo in j
    const VmTile t = vm_tile(G);
    const int ti = (int)(threadIdx.x % kVmI), tj = (int)(threadIdx.x / kVmI);
    const bool halo = (int)threadIdx.x < kVmHalo;
    int hi = 0, hj = 0;
    if (halo) vm_halo((int)threadIdx.x, hi, hj);
    const bool hx = (int)threadIdx.x < 6 * kVmJ;  // the halo entry is one of Lx
    const unsigned col = vm_off(G, t.i, t.j, 0);
    const unsigned hcol =
        vm_off(G, (t.i0 - 3 + hi + 2 * G.n[0]) % G.n[0], (t.j0 - 3 + hj + 2 * G.n[1]) % G.n[1], 0);
    const unsigned sk = (unsigned)G.sd[2];
    auto load = [&](int d, unsigned o, double (&v)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = fv[(4 * d + c) * G.vol + o];
    };
    double Z[7][4];  // this column's Fv~_zeta at planes k-3 .. k+3
    double X[4], Yv[4], H[4], Zn[4];
#pragma unroll
    for (int r = 0; r < 6; ++r) load(2, col + (unsigned)wrapi(t.k0 - 3 + r, G.n[2]) * sk, Z[r]);
    auto ahead = [&](int k) {
        load(2, col + (unsigned)wrapi(k + 3, G.n[2]) * sk, Zn);
        load(0, col + (unsigned)k * sk, X);
        load(1, col + (unsigned)k * sk, Yv);
        if (halo) load(hx ? 0 : 1, hcol + (unsigned)k * sk, H);
    };
    ahead(t.k0);
    for (int k = t.k0; k < t.k1; ++k) {
        double(*Xk)[kVmJ][kVmHI] = Lx[(k - t.k0) & 1];
        double(*Yk)[kVmHJ][kVmI] = Ly[(k - t.k0) & 1];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            Z[6][v] = Zn[v];
            Xk[v][tj][ti + 3] = X[v];
            Yk[v][tj + 3][ti] = Yv[v];
        }
        if (halo) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (hx)
                    Xk[v][hj - 3][hi] = H[v];
                else
                    Yk[v][hj][hi - 3] = H[v];
            }
        }
        if (k + 1 < t.k1) ahead(k + 1);
        lds_barrier();
        double acc[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            acc[v] = 0.0;
#pragma unroll
            for (int s = 1; s <= 3; ++s) acc[v] += d6w(s) * (Xk[v][tj][ti + 3 + s] - Xk[v][tj][ti + 3 - s]);
#pragma unroll
            for (int s = 1; s <= 3; ++s) acc[v] += d6w(s) * (Yk[v][tj + 3 + s][ti] - Yk[v][tj + 3 - s][ti]);
#pragma unroll
            for (int s = 1; s <= 3; ++s) acc[v] += d6w(s) * (Z[3 + s][v] - Z[3 - s][v]);
        }
        if (t.mine) {
            const unsigned o = col + (unsigned)k * sk;
            R[o] = 0.0;
#pragma unroll
            for (int v = 0; v < 4; ++v) R[(1 + v) * G.vol + o] = acc[v];
        }
#pragma unroll
        for (int r = 0; r < 6; ++r)
#pragma unroll
            for (int v = 0; v < 4; ++v) Z[r][v] = Z[r + 1][v];
    }
}

// ---------------------------------------------------------------------------
// CFL limit and state check
// ---------------------------------------------------------------------------

__global__ void k_dt_init(unsigned long long* bits) { *bits = 0ull; }

// sum_d (|s_d . u| + c |s_d|) (1/J)^{-1} at interior node t (0 past the last)
template <int DIM>
__device__ __forceinline__ double dt_node(const GeoK& G, double gamma, const double* __restrict__ met,
                                          const double* __restrict__ q, long t, long tot) {
    constexpr int NV = DIM + 2, NMET = DIM == 3 ? 10 : 5;
    if (t >= tot) return 0.0;
    const long r = t / G.n[0];
    const int i = (int)(t - r * G.n[0]);
    const int j = (int)(r % G.n[1]);
    const int k = (int)(r / G.n[1]);
    const long off = G.base + i + j * G.sd[1] + (long)k * G.sd[2];
    const double rho = q[off];
    double u[DIM], m2 = 0.0;
    for (int c = 0; c < DIM; ++c) {
        u[c] = q[(1 + c) * G.vol + off] / rho;
        m2 += q[(1 + c) * G.vol + off] * u[c];
    }
    const double p = (gamma - 1.0) * (q[(NV - 1) * G.vol + off] - 0.5 * m2);
    const double cs = sqrt(gamma * p / rho);
    double sum = 0.0;
    for (int d = 0; d < DIM; ++d) {
        double su = 0.0, ss = 0.0;
        for (int c = 0; c < DIM; ++c) {
            const double s = met[(d * DIM + c) * G.vol + off];
            su += s * u[c];
            ss += s * s;
        }
        sum += fabs(su) + cs * sqrt(ss);
    }
    return sum / met[(NMET - 1) * G.vol + off];
}

// A wave takes runs of 256 interior nodes (four per lane).  fmax drops the
// NaN of a non-physical node beside others, but a run of nothing else stays
// NaN, whose bits are above every number's (non-negative doubles order as
// their bit patterns do), and the state's dt is NaN.  Bound by HBM:
// 160x144x150 (15 arrays read, 415 MB) takes 86 us, 80 where waves do not keep
// to runs (and lose their NaN), 170 with a workgroup and an atomic per run.
constexpr int kDtRun = 256;
template <int DIM>
__global__ __launch_bounds__(256) void k_dt_reduce(GeoK G, double gamma,
                                                    const double* __restrict__ met,
                                                    const double* __restrict__ q,
                                                    unsigned long long* bits) {
    const long tot = (long)G.n[0] * G.n[1] * G.n[2];
    const int lane = threadIdx.x & 63;
    unsigned long long most = 0;
    for (long t = ((long)blockIdx.x * 4 + wave_id()) * kDtRun; t < tot; t += (long)gridDim.x * 4 * kDtRun) {
        double val = dt_node<DIM>(G, gamma, met, q, t + lane, tot);
#pragma unroll
        for (int h = 1; h < kDtRun / 64; ++h) val = fmax(val, dt_node<DIM>(G, gamma, met, q, t + 64 * h + lane, tot));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) val = fmax(val, __shfl_xor(val, o));
        most = max(most, (unsigned long long)__double_as_longlong(val));
    }
    __shared__ unsigned long long red[4];
    if (lane == 0) red[threadIdx.x >> 6] = most;
    __syncthreads();
    if (threadIdx.x == 0) {
        most = max(max(red[0], red[1]), max(red[2], red[3]));
        if (most > __hip_atomic_load(bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(bits, most);
    }
}

__global__ void k_dt_final(unsigned long long* bits, double cfl) {
    const double mx = __longlong_as_double((long long)*bits);
    *reinterpret_cast<double*>(bits) = cfl / mx;
}

template <int DIM>
__global__ __launch_bounds__(256) void k_check_state(GeoK G, double gamma, const double* __restrict__ q,
                                                      int* flag) {
    constexpr int NV = DIM + 2;
    const long tid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long tot = (long)G.n[0] * G.n[1] * G.n[2];
    if (tid >= tot) return;
    const int i = (int)(tid % G.n[0]);
    const int j = (int)((tid / G.n[0]) % G.n[1]);
    const int k = (int)(tid / ((long)G.n[0] * G.n[1]));
    const long off = G.base + i + j * G.sd[1] + (long)k * G.sd[2];
    double Q[NV];
    bool bad = false;
    for (int v = 0; v < NV; ++v) {
        Q[v] = q[v * G.vol + off];
        bad |= !isfinite(Q[v]);
    }
    double m2 = 0.0;
    for (int c = 0; c < DIM; ++c) m2 += Q[1 + c] * Q[1 + c];
    const double p = (gamma - 1.0) * (Q[NV - 1] - 0.5 * m2 / Q[0]);
    bad |= !(Q[0] > 0.0) || !(p > 0.0);
    if (bad) *flag = 1;
}

}  // namespace fpk
