// fp_kernels.hpp -- gfx950 kernels of the free-stream-preserving residual:
// direction sweeps, cell-face flux evaluation, metrics, CFL and state checks.
// Instantiated by the fp_inst_*.hip translation units and launched by fp_api.hip.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fp_device.hpp"

// Occupancy target of the face kernels: two waves per SIMD fits the FP64
// WENO face (the 6-node x 5-field characteristic values dominate) without
// spilling.  The FP32-mixed xi sweeps of the six-point stencils (WENO5,
// LU5, WENOCU6 with metrics of order up to 6) and the FP64 LU5 ones fit
// three (at most 168 registers) and run at three: their LDS window buffers
// allow it, the eta/zeta rings (79 KB per workgroup) do not; WENO7 and
// eighth-order metrics would spill at three.
#ifndef FP_SWEEP_ATTR
#define FP_SWEEP_ATTR __attribute__((amdgpu_waves_per_eu(2, 2)))
#endif
#define FP_XWAVES(PREC, RECON, Y) \
    ((((PREC) == 1 && (RECON) != 2) || ((PREC) == 0 && (RECON) == 1)) && (Y) != 8 ? 3 : 2)
#define FP_XSWEEP_ATTR(PREC, RECON, Y) \
    __attribute__((amdgpu_waves_per_eu(FP_XWAVES(PREC, RECON, Y), FP_XWAVES(PREC, RECON, Y))))

namespace fpk {

// Geometry of one structured block as the kernels see it.  Offsets are in
// elements of one variable array; `base` is the offset of interior node
// (0,0,0); sd[d] is the stride of axis d.
struct GeoK {
    int n[3];
    int g;
    int bc[3];
    long sd[3];
    long vol;
    long base;
    int xw;                // faces of a xi item (x_window, for the kernel that sweeps the block)
    float inv_nf, inv_ne;  // 1 / (n0 + 1), 1 / (n0 + 8)
};

// Global Lax-Friedrichs speeds.  The speeds live in sets of three directions; direction d of a set takes
// the three doubles at 16 d (one 128-byte line per direction, so the
// reductions of different directions do not contend for one line).
constexpr int kGlfDirStride = 16;
constexpr int kGlfSetStride = 3 * kGlfDirStride;

// What a sweep does with the flux difference d = F'_{i+1/2} - F'_{i-1/2} of
// its direction at node `off`:
//   FIRST: R = -d        MID: R = R - d
//   LAST_RES: out = (R - d) / (1/J)
//   LAST_RK:  k = (R - d) / (1/J); u = qin + dt k;
//             out = u (first stage) or a qn + b u (TVD RK3 stages 2, 3)
enum { EPI_FIRST = 0, EPI_MID = 1, EPI_LAST_RES = 2, EPI_LAST_RK = 3 };

// The kernels that apply the final epilogues take 1/J and, qin being the array
// they read, its density and energy from the stencil rows they staged.
struct EpiK {
    int mode;
    int stage0;
    double* R;
    double* out;
    const double* qin;
    const double* qn;
    double dt, a, b;
};

// Global-memory view of a pointer the compiler cannot prove global (one read
// from a table in device memory, as the batched kernels' arrays are):
// accesses through it are global_* instructions, counted only in vmcnt,
// instead of flat_* ones, which also count in lgkmcnt and so hold up every
// wait for LDS reads that follows them.
typedef __attribute__((address_space(1))) double gdouble;
__device__ __forceinline__ gdouble* gmem(double* p) { return (gdouble*)p; }
__device__ __forceinline__ const gdouble* gmem(const double* p) { return (const gdouble*)p; }

// Buffer access to one variable array: the resource (base, size) is
// wave-uniform and lives in scalar registers, every lane supplies a 32-bit
// byte offset, so no 64-bit vector address arithmetic is spent per access.
// Reads past `elems` return 0 by the hardware's range check.  A variable array must stay below 4 GiB (checked
// by the host: at most 2^29 nodes per block, ghosts included).
#define FP_BUF_FLAGS 0x00020000
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const double* base, long elems) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)(elems * 8), FP_BUF_FLAGS);
}
__device__ __forceinline__ double ldb(const double* base, long elems, unsigned byteoff) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(buf(base, elems), byteoff, 0, 0));
}
// A wave-uniform pointer the compiler must treat as redefined at this point,
// so that what derives from it (the per-variable buffer resources) is
// rebuilt at the use from a few scalar operations instead of being hoisted
// into long-lived scalar registers, which would spill into vector lanes.
__device__ __forceinline__ const double* rebase(const double* p) {
    asm volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ double* rebase(double* p) {
    asm volatile("" : "+s"(p));
    return p;
}

typedef unsigned int u32x2_t __attribute__((__vector_size__(2 * sizeof(unsigned int))));
__device__ __forceinline__ void stb(double* base, long elems, unsigned byteoff, double x) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, x), buf(base, elems), byteoff, 0, 0);
}

// The epilogue split in two, so that its loads can be issued early (before
// the face computation) and its stores done late: epi_load reads what the
// mode needs at node `off`, epi_store applies the same arithmetic as
// epilogue().
template <int NV>
struct EpiPre {
    double R[NV], qin[NV], qn[NV], V;
};

// (the final epilogues' callers supply 1/J and the stage input's density and
// energy from the rows they staged, which hold its momentum as velocity; they
// may take the momentum later, with epi_load_qin)
// (buffer loads and stores: one 32-bit byte offset per lane serves every
// variable array, whose base goes into the wave-uniform resource)
template <int NV>
__device__ __forceinline__ void epi_load_qin(const EpiK& ep, long vol, long off, EpiPre<NV>& p) {
    if (ep.mode != EPI_LAST_RK) return;
    const double* qin = rebase(ep.qin);
#pragma unroll
    for (int v = 1; v < NV - 1; ++v) p.qin[v] = ldb(qin + v * vol, vol, (unsigned)off * 8u);
}
template <int NV>
__device__ __forceinline__ void epi_load(const EpiK& ep, long vol, long off, EpiPre<NV>& p, bool with_qin) {
    if (ep.mode == EPI_FIRST) return;
    const unsigned bo = (unsigned)off * 8u;
    const double* R = rebase(ep.R);
#pragma unroll
    for (int v = 0; v < NV; ++v) p.R[v] = ldb(R + v * vol, vol, bo);
    if (ep.mode != EPI_LAST_RK) return;
    if (with_qin) epi_load_qin<NV>(ep, vol, off, p);
    if (ep.stage0) return;
    const double* qn = rebase(ep.qn);
#pragma unroll
    for (int v = 0; v < NV; ++v) p.qn[v] = ldb(qn + v * vol, vol, bo);
}

// The same epilogue with its mode fixed to MID (for a sweep that is never
// the last of a stage), so that no final-epilogue code is compiled in.
__device__ __forceinline__ EpiK epi_mid(const EpiK& ep) {
    EpiK e = ep;
    e.mode = EPI_MID;
    return e;
}

template <int NV>
__device__ __forceinline__ void epi_store(const EpiK& ep, long vol, long off, const EpiPre<NV>& p,
                                          const double (&d)[NV]) {
    const unsigned bo = (unsigned)off * 8u;
    if (ep.mode == EPI_FIRST) {
        double* R = rebase(ep.R);
#pragma unroll
        for (int v = 0; v < NV; ++v) stb(R + v * vol, vol, bo, -d[v]);
    } else if (ep.mode == EPI_MID) {
        double* R = rebase(ep.R);
#pragma unroll
        for (int v = 0; v < NV; ++v) stb(R + v * vol, vol, bo, p.R[v] - d[v]);
    } else if (ep.mode == EPI_LAST_RES) {
        const double J = 1.0 / p.V;  // one division per node, not one per variable
        double* out = rebase(ep.out);
#pragma unroll
        for (int v = 0; v < NV; ++v) stb(out + v * vol, vol, bo, (p.R[v] - d[v]) * J);
    } else {
        const double J = 1.0 / p.V;
        double* out = rebase(ep.out);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double k = (p.R[v] - d[v]) * J;
            const double u = p.qin[v] + ep.dt * k;
            stb(out + v * vol, vol, bo, ep.stage0 ? u : ep.a * p.qn[v] + ep.b * u);
        }
    }
}

// Reads the stencil of face i+1/2 of one grid line along axis DIR: slot r
// holds node i-3+r.  Periodic axes wrap to the image inside the interior;
// frozen axes read the ghost layers of the same array (the RK3 driver copies
// the caller's frozen ghost values into its stage arrays).  Metrics are read
// directly: fp_metrics fills their ghost layers.
template <int DIM, int DIR>
struct LineLoader {
    static constexpr bool CT = true;
    const double* __restrict__ met;
    const double* q;
    long vol;       // elements per variable
    unsigned lb;    // element offset of node 0 of the line
    int sd;         // element stride along the line
    int i;          // the face is i+1/2
    int nd;         // interior nodes along the line
    int per;        // periodic axis
    double gm1;     // gamma - 1

    __device__ __forceinline__ LineLoader(const GeoK& G, const double* met_, const double* q_,
                                          long lb_, int i_, double gamma)
        : met(met_), q(q_), vol(G.vol), lb((unsigned)lb_), sd((int)G.sd[DIR]), i(i_),
          nd(G.n[DIR]), per(G.bc[DIR] == 0), gm1(gamma - 1.0) {}

    // A copy whose loads cannot be hoisted above, or merged with loads
    // before, the computation of `dep`: the line offset passes through an
    // empty asm that takes `dep` as input.  This bounds the live range of the
    // stencil values to one phase of the face computation.
    __device__ __forceinline__ LineLoader after(double dep) const {
        LineLoader c = *this;
        asm volatile("" : "+v"(c.lb) : "v"(dep));
        return c;
    }

    __device__ __forceinline__ void cons(int r, double (&qv)[DIM + 2]) const {
        const int t = i - 3 + r;
        int tt = t;
        if (per) tt = t < 0 ? t + nd : (t >= nd ? t - nd : t);
        const unsigned off = (lb + (unsigned)(tt * sd)) * 8u;
#pragma unroll
        for (int v = 0; v < DIM + 2; ++v) qv[v] = ldb(q + v * vol, vol, off);
    }
    __device__ __forceinline__ void prim(int r, Prim<DIM>& P) const {
        double qv[DIM + 2];
        cons(r, qv);
        to_prim<DIM>(qv, gm1, P);
    }
    __device__ __forceinline__ void metric(int r, double& V, double (&s)[DIM]) const {
        constexpr int NMET = DIM == 3 ? 10 : 5;
        const unsigned moff = (lb + (unsigned)((i - 3 + r) * sd)) * 8u;
        V = ldb(met + (NMET - 1) * vol, vol, moff);
#pragma unroll
        for (int c = 0; c < DIM; ++c) s[c] = ldb(met + (DIR * DIM + c) * vol, vol, moff);
    }
    // adds slot r with weight w to the face values of Q/J, 1/J and s
    __device__ __forceinline__ void interp(int r, double w, double (&Qt)[DIM + 2], double& Vf,
                                           double (&sf)[DIM]) const {
        double qv[DIM + 2], V, s[DIM];
        cons(r, qv);
        metric(r, V, s);
        const double wV = w * V;
        Vf += wV;
#pragma unroll
        for (int c = 0; c < DIM; ++c) sf[c] += w * s[c];
#pragma unroll
        for (int v = 0; v < DIM + 2; ++v) Qt[v] = fma(wV, qv[v], Qt[v]);
    }
};

// Slot access of a loader to nodes staged in LDS: `at(r, v)` is
// value v of slot r in the order rho, u, E, 1/J, s, ct.
template <int DIM, class LD>
struct StagedNodes {
    __device__ __forceinline__ const LD& self() const { return static_cast<const LD&>(*this); }
    __device__ __forceinline__ void prim(int r, Prim<DIM>& P) const {
        P.rho = self().at(r, 0);
#pragma unroll
        for (int c = 0; c < DIM; ++c) P.u[c] = self().at(r, 1 + c);
        P.E = self().at(r, DIM + 1);
        if constexpr (LD::CT) P.ct = self().at(r, 2 * DIM + 3);
    }
    __device__ __forceinline__ void metric(int r, double& V, double (&s)[DIM]) const {
        V = self().at(r, DIM + 2);
#pragma unroll
        for (int c = 0; c < DIM; ++c) s[c] = self().at(r, DIM + 3 + c);
    }
    __device__ __forceinline__ void interp(int r, double w, double (&Qt)[DIM + 2], double& Vf,
                                           double (&sf)[DIM]) const {
        double V, s[DIM];
        metric(r, V, s);
        const double wV = w * V, wVr = wV * self().at(r, 0);
        Vf += wV;
#pragma unroll
        for (int c = 0; c < DIM; ++c) sf[c] += w * s[c];
        Qt[0] += wVr;
#pragma unroll
        for (int c = 0; c < DIM; ++c) Qt[1 + c] = fma(wVr, self().at(r, 1 + c), Qt[1 + c]);
        Qt[DIM + 1] = fma(wV, self().at(r, DIM + 1), Qt[DIM + 1]);
    }
};

// XCD-aware workgroup order: the dispatcher hands workgroups to the 8 XCDs
// round-robin (b -> XCD b mod 8), each XCD with its own L2.  Renumbering
// gives XCD x a contiguous range of the work instead of every eighth item,
// so that the reconstruction windows and metric rows that neighbouring items
// share are read into one L2.  Measured on the single-block sweeps: 2D
// Double Mach Reflection 961x241 (LLC-resident) 62.3 -> 54.5 us per RK stage,
// residual 45x33x29 23.9 -> 22.7 us, WENO-CU6 145x113x97 1350 -> 1318 us per
// step, 256^3 WENO5 1-2%.  The batched sweeps keep the plain order: 48 body
// blocks take the same time either way, and 24 serving blocks lost 2%.
__device__ __forceinline__ long xcd_block(long b, long nb) {
    const long per = nb / 8, rem = nb % 8, x = b % 8;
    return x * per + (x < rem ? x : rem) + b / 8;
}

template <int PREC>
using char_t = typename std::conditional<PREC == 1, float, double>::type;

// One dword per lane from a variable array of `elems` doubles into LDS
// (buffer-to-LDS DMA: no registers hold the data; completion is tracked by
// the wave's vmcnt).  Lane l writes the dword at lds + 4 l.  The array's
// base goes into the wave-uniform resource, so the lane supplies only its
// 32-bit byte offset (no per-load 64-bit address arithmetic).
__device__ __forceinline__ void dma_dword(const double* var, long elems, void* lds, unsigned byteoff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buf(var, elems), (__attribute__((address_space(3))) void*)lds, 4,
                                             byteoff, 0, 0, 0);
}

// Barrier of a workgroup for its LDS traffic alone: unlike __syncthreads it
// leaves global loads and stores in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The same for two consecutive doubles per lane: lane l writes 16 bytes at
// lds + 16 l (which must be 16-byte aligned; the memory side needs 4).
__device__ __forceinline__ void dma_pair(const double* var, long elems, void* lds, unsigned byteoff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buf(var, elems), (__attribute__((address_space(3))) void*)lds, 16,
                                             byteoff, 0, 0, 0);
}

// The wave's index in its workgroup, as a value the compiler knows to be
// uniform across the wave (so what derives from it stays in scalar registers).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// ---------------------------------------------------------------------------
// xi sweep
// ---------------------------------------------------------------------------
// The faces of all xi-lines of a block are numbered flat, F = L (n0+1) + f
// (line L, face f-1/2 of it).  A wave item takes W consecutive faces,
// F = (W-1) j + l for lane l < W, so consecutive items overlap by one face:
// lane l > 0 takes its left neighbour's flux by a lane shift and forms the
// flux difference of its node.  The stencil nodes of the item are staged in
// the wave's own LDS buffer by global-to-LDS DMA, indexed by the extended
// flat index e = L (n0+8) + x + 4 (line L with four extra nodes on each side,
// x = -4 .. n0+3): slot r (node f-4+r) of face F is entry e(F) + r with
// e(F) = L (n0+8) + f.  A window of W faces spans W + 7 (lines touched)
// entries; W is the largest width (at most 64) that fits NE entries.  The
// sweeps that run three waves per SIMD stage NE = 88 entries (W = 64 still
// for lines of 30 nodes and more): the workgroup's double buffers then take
// 53.5 KB and three workgroups fit a CU's LDS; the others stage 128.
template <int DIM, int NE_>
struct XLds {
    static constexpr int NE = NE_;          // staged entries per buffer
    static constexpr int NS = 2 * DIM + 3;  // q, 1/J, s_xi; the momentum as velocity once converted
    alignas(16) double b[2][NS][NE];        // double buffer: current item, next item
    double ct[NE];                          // the thermal speed of the current item's nodes
};
__device__ __host__ constexpr int x_entries(int prec, int recon, int Y) {
    return FP_XWAVES(prec, recon, Y) == 3 ? 88 : 128;
}

__device__ __host__ __forceinline__ int x_window(int n0, int ne) {
    int W = 64;
    while (W > 2 && W + 7 * ((W + n0) / (n0 + 1) + 1) > ne) --W;
    return W;
}

// wave items of the xi sweep of one block (ne: the sweep's staged entries)
__device__ __host__ __forceinline__ long sweep_x_items(const int n[3], int ne) {
    const long total = (long)(n[0] + 1) * n[1] * n[2];
    const int W = x_window(n[0], ne);
    return (total - 1 + W - 2) / (W - 1);
}

// floor(k / d) for 0 <= k, d < 2^20, in single precision: exact, since
// (k + 1/2) / d is at least 1/(2 d) away from an integer and the rounding
// error of the product is below k / d * 2^-23.
__device__ __forceinline__ unsigned small_div(unsigned k, float inv_d) {
    return (unsigned)(((float)k + 0.5f) * inv_d);
}

// Line L0 + dL of the xi-lines, from the decomposition (a1, a2) of L0 over
// (n1, n2): (l1, l2) with l1 < n1.
__device__ __forceinline__ void line_step(unsigned a1, unsigned a2, unsigned dL, unsigned n1, unsigned& l1,
                                          unsigned& l2) {
    l1 = a1 + dL;
    l2 = a2;
    while (l1 >= n1) {
        l1 -= n1;
        ++l2;
    }
}

// The place of a xi item: its first face F0 is face f0 of line a1 + n1 a2.
// A wave steps through its items by a fixed number of faces, so the places
// follow from each other by additions with carry.
struct XPos {
    unsigned F0, f0, a1, a2;
};
__device__ __host__ __forceinline__ XPos x_pos(const GeoK& G, unsigned F0) {
    const unsigned nf = (unsigned)G.n[0] + 1, n1 = (unsigned)G.n[1];
    XPos p;
    const unsigned L0 = F0 / nf;
    p.F0 = F0;
    p.f0 = F0 - L0 * nf;
    p.a2 = L0 / n1;
    p.a1 = L0 - p.a2 * n1;
    return p;
}
__device__ __forceinline__ void x_advance(const GeoK& G, const XPos& step, XPos& p) {
    const unsigned nf = (unsigned)G.n[0] + 1, n1 = (unsigned)G.n[1];
    p.F0 += step.F0;
    p.f0 += step.f0;
    p.a1 += step.a1;
    p.a2 += step.a2;
    if (p.f0 >= nf) {
        p.f0 -= nf;
        ++p.a1;
    }
    if (p.a1 >= n1) {
        p.a1 -= n1;
        ++p.a2;
    }
}

// The uniform geometry of a xi item: node 0 of its first line at element
// `line`, its staged entries e(F0) .. e(Fl) + 7 and its faces.
// How its entries are placed (`kind`):
//   X_ROW   one stretch of memory: on one line, no periodic image and no
//           entry past the stored ghosts among them.  Two entries per lane
//           and a handful of instructions stage them all, against some 27
//           vector instructions per 32 entries (two thirds of the items of
//           lines of 256 nodes: a 256^3 WENO5 sweep took 1.10 ms against 1.16
//           in FP64, 0.87 against 0.93 FP32-mixed);
//   X_NEAR  on the first line or the next one of the same plane: a comparison
//           places them;
//   X_FAR   lines are counted by division and wrapped (short lines, ends of
//           planes).
enum { X_ROW = 0, X_NEAR = 1, X_FAR = 2 };
struct XItem {
    unsigned f0, a1, a2, line, count, faces, kind;
};

template <int NE>
__device__ __forceinline__ XItem x_item(const GeoK& G, const XPos& p) {
    XItem it;
    const unsigned nf = (unsigned)G.n[0] + 1, n1 = (unsigned)G.n[1];
    const unsigned total = nf * n1 * (unsigned)G.n[2];
    it.f0 = p.f0;
    it.a1 = p.a1;
    it.a2 = p.a2;
    it.line = (unsigned)G.base + p.a1 * (unsigned)G.sd[1] + p.a2 * (unsigned)G.sd[2];
    it.faces = min((unsigned)G.xw, total - p.F0);
    unsigned dl = 0, fl = it.f0 + it.faces - 1;  // the last face, its line counted from the first
    while (fl >= nf) {
        fl -= nf;
        ++dl;
    }
    it.count = dl * 7 + it.faces + 7;
    // entries x = f0 - 4 .. of the first line; memory holds -gl .. n0 - 1 + gl
    const int gl = G.bc[0] == 0 ? 0 : G.g;
    if (dl == 0 && (int)it.f0 - 4 >= -gl && (int)(it.f0 + it.count) - 5 <= G.n[0] - 1 + gl)
        it.kind = X_ROW;
    else
        it.kind = nf + 7 >= (unsigned)((NE + 31) / 32 * 32) && p.a1 + 1 < n1 ? X_NEAR : X_FAR;
    return it;
}

// Node 0 of line L0 + dL of an item, as an element offset; lines past the
// block's last one (their entries are never read) take that one.
__device__ __forceinline__ unsigned x_line(const GeoK& G, const XItem& it, unsigned dL) {
    unsigned l1, l2;
    line_step(it.a1, it.a2, dL, (unsigned)G.n[1], l1, l2);
    if (l2 >= (unsigned)G.n[2]) {
        l1 = (unsigned)G.n[1] - 1;
        l2 = (unsigned)G.n[2] - 1;
    }
    return (unsigned)G.base + l1 * (unsigned)G.sd[1] + l2 * (unsigned)G.sd[2];
}

// Stage an item's stencil entries into buf (all 64 lanes; asynchronous).
template <int DIM, int NE, bool NEAR>
__device__ __forceinline__ void x_stage_as(const GeoK& G, const double* __restrict__ met, const double* qs,
                                           const XItem& it, double (*buf)[NE]) {
    constexpr int NV = DIM + 2;
    constexpr int NMET = DIM == 3 ? 10 : 5;
    const unsigned lane = threadIdx.x & 63;
    const unsigned n0 = (unsigned)G.n[0], ne = n0 + 8;
    const int g = G.g;
    const int per = G.bc[0] == 0;
    const unsigned np = (it.count + 31) / 32;
#pragma unroll
    for (int p = 0; p < (NE + 31) / 32; ++p) {
        if ((unsigned)p >= np) break;
        // a pass moves 32 entries (two lanes per entry); the last one may be
        // partial, and its lanes past the buffer's end must write nothing
        if (NE % 32 != 0 && 32u * p + (lane >> 1) >= (unsigned)NE) continue;
        const unsigned k = it.f0 + 32u * p + (lane >> 1);  // from the start of line L0's entries
        unsigned lb;
        int x;
        if constexpr (NEAR) {
            lb = k >= ne ? it.line + (unsigned)G.sd[1] : it.line;
            x = (int)min(k, k - ne) - 4;
        } else {
            const unsigned dL = small_div(k, G.inv_ne);
            x = (int)(k - dL * ne) - 4;
            lb = x_line(G, it, dL);
        }
        const int xm = x < -g ? -g : (x > (int)n0 - 1 + g ? (int)n0 - 1 + g : x);
        int xq = xm;
        if (per) {
            xq = x < 0 ? x + (int)n0 : (x >= (int)n0 ? x - (int)n0 : x);
            xq = xq < 0 ? 0 : (xq > (int)n0 - 1 ? (int)n0 - 1 : xq);
        }
        const unsigned oq = (lb + (unsigned)xq) * 8u + (lane & 1) * 4u;
        const unsigned om = (lb + (unsigned)xm) * 8u + (lane & 1) * 4u;
        const double* qp = rebase(qs);
        const double* mp = rebase(met);
#pragma unroll
        for (int v = 0; v < NV; ++v) dma_dword(qp + v * G.vol, G.vol, &buf[v][32 * p], oq);
        dma_dword(mp + (NMET - 1) * G.vol, G.vol, &buf[NV][32 * p], om);
#pragma unroll
        for (int c = 0; c < DIM; ++c) dma_dword(mp + c * G.vol, G.vol, &buf[NV + 1 + c][32 * p], om);
    }
}
template <int DIM, int NE>
__device__ __forceinline__ void x_stage(const GeoK& G, const double* __restrict__ met, const double* qs,
                                        const XItem& it, double (*buf)[NE]) {
    constexpr int NV = DIM + 2;
    constexpr int NMET = DIM == 3 ? 10 : 5;
    static_assert(NE % 2 == 0 && NE <= 128, "a lane stages two entries");
    if (it.kind == X_ROW) {
        const unsigned k = 2u * (threadIdx.x & 63);
        if (k < it.count) {  // (an odd count's last pair brings one entry more)
            const unsigned off = (it.line + it.f0 - 4u + k) * 8u;
            const double* qp = rebase(qs);
            const double* mp = rebase(met);
#pragma unroll
            for (int v = 0; v < NV; ++v) dma_pair(qp + v * G.vol, G.vol, &buf[v][0], off);
            dma_pair(mp + (NMET - 1) * G.vol, G.vol, &buf[NV][0], off);
#pragma unroll
            for (int c = 0; c < DIM; ++c) dma_pair(mp + c * G.vol, G.vol, &buf[NV + 1 + c][0], off);
        }
    } else if (it.kind == X_NEAR) {
        x_stage_as<DIM, NE, true>(G, met, qs, it, buf);
    } else {
        x_stage_as<DIM, NE, false>(G, met, qs, it, buf);
    }
}

// Velocity and thermal speed of an item's entries, the former in place of the
// momentum: each entry serves the six to eight faces around it.
template <int DIM, int NE>
__device__ __forceinline__ void x_convert(unsigned count, double gm1, double (*buf)[NE], double* ct) {
    constexpr int NV = DIM + 2;
    for (unsigned e = threadIdx.x & 63; e < count; e += 64) {
        double q[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) q[v] = buf[v][e];
        Prim<DIM> P;
        to_prim<DIM>(q, gm1, P);
#pragma unroll
        for (int c = 0; c < DIM; ++c) buf[1 + c][e] = P.u[c];
        ct[e] = P.ct;
    }
    // other lanes of the wave read these entries (LDS operations of a wave
    // complete in order)
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// Stencil reads of one lane's xi face from the wave's staged entries.
template <int DIM, int NE>
struct XLoader : StagedNodes<DIM, XLoader<DIM, NE>> {
    static constexpr bool CT = true;
    const double (*buf)[NE];
    const double* ct;
    unsigned ea;  // byte offset of entry e(F) in a variable row

    __device__ __forceinline__ XLoader after(double dep) const {
        XLoader c = *this;
        asm volatile("" : "+v"(c.ea) : "v"(dep));
        return c;
    }

    __device__ __forceinline__ double at(int r, int v) const {
        const char* row = v == 2 * DIM + 3 ? reinterpret_cast<const char*>(ct)
                                           : reinterpret_cast<const char*>(&buf[0][0]) + v * NE * 8;
        return *reinterpret_cast<const double*>(row + ea + r * 8);
    }
};

// Faces of item j from its staged entries, the lane-shift difference and
// the epilogue (all 64 lanes must call this: the lane shift).  The xi sweep
// comes first in a stage, so its epilogue is FIRST (ACC = false: R = -d,
// nothing to load) or MID (ACC = true: R -= d, after the viscous part or a
// caller's accumulation; R loads while the face is computed).
//
// The wave waits for its memory operations between the face and the stores:
// the next item's entries, asked for before the face, have landed by then,
// and no wait ever holds for a store that was just issued.
template <int DIM, int RECON, int Y, int PREC, bool ACC>
__device__ __forceinline__ void x_compute(const GeoK& G, const SchemeK& sk, const EpiK& ep, const XItem& it,
                                          double (*buf)[x_entries(PREC, RECON, Y)], double* ct) {
    constexpr int NV = DIM + 2;
    const unsigned lane = threadIdx.x & 63;
    const unsigned nf = (unsigned)G.n[0] + 1;
    const bool active = lane < it.faces;
    double fl[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) fl[v] = 0.0;
    const unsigned k = it.f0 + lane;  // from the first face of line L0
    unsigned dL, f, noff;
    if (it.kind != X_FAR) {
        dL = k >= nf ? 1 : 0;
        f = min(k, k - nf);
        noff = dL ? it.line + (unsigned)G.sd[1] : it.line;
    } else {
        dL = small_div(k, G.inv_nf);
        f = k - dL * nf;
        noff = x_line(G, it, dL);
    }
    noff += f - 1;
    // lane l > 0 writes node f - 1, between its face and lane l - 1's
    const bool writes = active && lane > 0 && f > 0;
    EpiPre<NV> pre;
    x_convert<DIM, x_entries(PREC, RECON, Y)>(it.count, sk.gamma - 1.0, buf, ct);
    if (ACC && writes) epi_load<NV>(epi_mid(ep), G.vol, noff, pre, false);
    if (active) {
        XLoader<DIM, x_entries(PREC, RECON, Y)> ld;
        ld.buf = buf;
        ld.ct = ct;
        ld.ea = (dL * 7 + lane) * 8u;  // e(F) - e(F0)
        face_flux<DIM, RECON, Y, char_t<PREC>>(ld, sk, fl);
    }
    double d[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) d[v] = fl[v] - __shfl_up(fl[v], 1, 64);
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    if (writes) {
        if (ACC) {
            epi_store<NV>(epi_mid(ep), G.vol, noff, pre, d);
        } else {
            double* R = rebase(ep.R);
#pragma unroll
            for (int v = 0; v < NV; ++v) stb(R + v * G.vol, G.vol, noff * 8u, -d[v]);
        }
    }
}

// Persistent xi sweep of one block.  Where the grid is whole (a multiple of 8)
// each XCD takes an eighth of the items, contiguous, and its waves go through
// it side by side, so that the last items, less than one per wave, are spread
// over all XCDs; in a smaller grid every wave has one item, in XCD-contiguous
// order.  FP64 WENO5 96x80x70, 4.2 items per wave: 40.8 us, 45.4 with the last
// items on the first XCDs, 42.6 with neighbouring items on different XCDs;
// WENOCU6 80x64x60 33.0, 40.4 and 37.3; 256^3 the same.  A wave stages its next
// item, `step` on, while it computes (ACC: the epilogue is MID, not
// FIRST; those kernels run at two waves per SIMD, the accumulator's registers
// do not fit three).
#define FP_XWAVES_ACC(PREC, RECON, Y, ACC) ((ACC) ? 2 : FP_XWAVES(PREC, RECON, Y))
template <int DIM, int RECON, int Y, int PREC, bool ACC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FP_XWAVES_ACC(PREC, RECON, Y, ACC),
                                                                     FP_XWAVES_ACC(PREC, RECON, Y, ACC))))
void k_sweep_x(GeoK G, SchemeK sk, const double* __restrict__ met, const double* qs, EpiK ep, XPos step,
               unsigned items) {
    constexpr int NE = x_entries(PREC, RECON, Y);
    __shared__ XLds<DIM, NE> lds[4];
    XLds<DIM, NE>& L = lds[wave_id()];
    const unsigned b = blockIdx.x, nb = gridDim.x, x = b % 8;
    const unsigned j = nb % 8 ? (unsigned)xcd_block(b, nb) * 4 + wave_id() : items * x / 8 + b / 8 * 4 + wave_id();
    const unsigned end = nb % 8 ? items : items * (x + 1) / 8;
    if (j >= end) return;
    const unsigned W1 = (unsigned)G.xw - 1, lim = end * W1;  // items of W faces start W - 1 apart
    XPos pos = x_pos(G, j * W1);
    XItem it = x_item<NE>(G, pos);
    x_stage<DIM, NE>(G, met, qs, it, L.b[0]);
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    for (int cur = 0;; cur ^= 1) {
        XItem next = it;
        x_advance(G, step, pos);
        const bool more = pos.F0 < lim;
        if (more) {
            next = x_item<NE>(G, pos);
            x_stage<DIM, NE>(G, met, qs, next, L.b[cur ^ 1]);
        }
        x_compute<DIM, RECON, Y, PREC, ACC>(G, sk, ep, it, L.b[cur], L.ct);
        if (!more) break;
        it = next;
    }
}

// LDS of an eta / zeta sweep workgroup: a ring of stencil rows (the q, 1/J
// and s_DIR values of the workgroup's 64 lines at one node index along
// DIR), the four face fluxes of an iteration and the carried last flux of
// the previous one.
constexpr int wide_stencil(int recon, int Y) { return (recon == 2 || Y == 8) ? 1 : 0; }

// WIDE: the face reads slots 0..7 (nodes i-3 .. i+4: eighth-order metrics or
// WENO7), else slots 1..6 (nodes i-2 .. i+3).
template <int DIM, int WIDE>
struct WgLds {
    static constexpr int NV = DIM + 2;
    // values per node: density, velocity, energy, 1/J, s_DIR and, where the
    // LDS has room beside two resident workgroups, the thermal speed; else the
    // faces take the sound speed from the pressure
    static constexpr bool CT = !(WIDE && DIM == 3);
    static constexpr int NS = 2 * DIM + 3 + (CT ? 1 : 0);
    static constexpr int LO = WIDE ? 3 : 2;  // nodes below node i a face i+1/2 reads
    static constexpr int HI = WIDE ? 4 : 3;  // nodes above node i
    static constexpr int WIN = 4 + LO + HI;    // rows read by the four faces of an iteration
    static constexpr int RING = WIN + 4;       // plus the four rows prefetched for the next
    double ring[RING][NS][64];
    double flux[4][NV][64];  // the four faces of the current iteration
    double carry[NV][64];    // the last face of the previous iteration
};
static_assert(2 * sizeof(WgLds<3, 0>) <= 160 * 1024 && 2 * sizeof(WgLds<3, 1>) <= 160 * 1024,
              "two workgroups per CU");

// Stencil reads of face i+1/2 from the LDS ring: slot r (node i-3+r) is ring
// row (b0 + r) mod RING.
template <int DIM, int WIDE>
struct LdsLoader : StagedNodes<DIM, LdsLoader<DIM, WIDE>> {
    using W = WgLds<DIM, WIDE>;
    static constexpr bool CT = W::CT;
    const W* L;
    unsigned la;  // byte offset of this lane in a ring row
    int b0;       // ring row of slot 0, in [0, RING)

    __device__ __forceinline__ LdsLoader after(double dep) const {
        LdsLoader c = *this;
        asm volatile("" : "+v"(c.la) : "v"(dep));
        return c;
    }

    __device__ __forceinline__ double at(int r, int v) const {
        int idx = b0 + r;
        idx = idx >= W::RING ? idx - W::RING : idx;
        return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(&L->ring[idx][0][0]) + la + v * 512);
    }
};

// Velocity and thermal speed of one ring row, the former in place of the
// momentum (a wave, one line per lane; the row's DMA must have landed).
template <int DIM, int WIDE>
__device__ __forceinline__ void wg_convert(WgLds<DIM, WIDE>& L, int slot, double gm1) {
    constexpr int NV = DIM + 2;
    const int lane = threadIdx.x & 63;
    double q[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) q[v] = L.ring[slot][v][lane];
    Prim<DIM> P;
    to_prim<DIM>(q, gm1, P);
#pragma unroll
    for (int c = 0; c < DIM; ++c) L.ring[slot][1 + c][lane] = P.u[c];
    if constexpr (WgLds<DIM, WIDE>::CT) L.ring[slot][2 * DIM + 3][lane] = P.ct;
}

// eta / zeta sweeps: a workgroup of four waves takes a block of 64 grid lines
// along DIR (consecutive in the flattened (i, other) index, so row loads are
// coalesced) and one segment [k0, k1) of their nodes.
// The stencil rows are staged in an LDS ring by global-to-LDS DMA, one row
// per wave per iteration, prefetched one iteration ahead.  Per iteration
// wave w evaluates the face f+1/2, f = k0 - 1 + 4 it + w, on its 64 lines
// from the ring, the fluxes go to LDS and wave w forms node f's difference
// F'_{f+1/2} - F'_{f-1/2}.  Each wave forms its row's velocities and thermal
// speeds once its DMA has landed, before the barrier that publishes it.  Bound
// by vector issue.  With the quotients and roots per node instead of per face,
// no wait for stores between the barriers and the xi sweep's and workgroup
// orders above, an RK3 step of a 256^3 block takes 9.05 ms against 9.71 in
// FP64 WENO5 (three sweeps per stage), 7.96 against 8.21 FP32-mixed, and two
// of 128^3 with LU5 1.53 against 1.73.  (Without the momentum and pressure
// products that keep the residual's rounding down: 8.86, 7.75 and 1.46.)
// Every thread of the workgroup runs the same iterations and barriers.  A
// caller that reuses `L` for another item must synchronise the workgroup
// first.
// (the batched sweep has something to do when the item's first rows have
// arrived)
struct Nothing {
    __device__ __forceinline__ void operator()() const {}
};
template <int DIM, int DIR, int RECON, int Y, int PREC, typename FN = Nothing>
__device__ __forceinline__ void sweep_wg_item(const GeoK& G, const SchemeK& sk,
                                              const double* __restrict__ met, const double* qs,
                                              const EpiK& ep, int lineblk, int k0, int k1,
                                              WgLds<DIM, wide_stencil(RECON, Y)>& L, FN staged = FN()) {
    using W = WgLds<DIM, wide_stencil(RECON, Y)>;
    constexpr int NV = DIM + 2;
    constexpr int NMET = DIM == 3 ? 10 : 5;
    constexpr int OTH = DIR == 1 ? 2 : 1;
    const int lane = threadIdx.x & 63;
    const int w = wave_id();
    const long nlines = (long)G.n[0] * G.n[OTH];
    const long line = lineblk * 64L + lane;
    const bool lane_ok = line < nlines;
    const int i = lane_ok ? (int)(line % G.n[0]) : 0;
    const int o = lane_ok ? (int)(line / G.n[0]) : 0;
    const long lb = G.base + i + (long)o * G.sd[OTH];
    // DMA: lane l moves dword (l & 1) of line 32 h + l / 2 (h = 0, 1) of the
    // block; lines past the end repeat the last one
    unsigned loff[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        long ln = lineblk * 64L + 32 * h + (lane >> 1);
        ln = ln < nlines ? ln : nlines - 1;
        const long off = G.base + ln % G.n[0] + (ln / G.n[0]) * G.sd[OTH];
        loff[h] = (unsigned)off * 8u + (unsigned)(lane & 1) * 4u;
    }
    const int nd = G.n[DIR];
    const int per = G.bc[DIR] == 0;
    const int sdD = (int)G.sd[DIR];
    const long vol = G.vol;
    const int iters = (k1 - k0 + 1 + 3) / 4;  // faces k0-1/2 .. k1-1/2
    const int tb = k0 - 1 - W::LO;            // node index of ring row 0
    const int tmax = k1 - 1 + W::HI;          // last row any needed face reads
    const double gm1 = sk.gamma - 1.0;
    // the stage input's momentum for the final epilogue: FP32 loads it with
    // the other operands, FP64, which would spill, after the face
    constexpr bool late_qin = sizeof(char_t<PREC>) == 8;
    auto load_row = [&](int t) {
        if (t > tmax) return;
        const int slot = (t - tb) % W::RING;
        int tt = t;
        if (per) tt = t < 0 ? t + nd : (t >= nd ? t - nd : t);
        const unsigned qo = (unsigned)(tt * sdD) * 8u, mo = (unsigned)(t * sdD) * 8u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double* qp = rebase(qs);
            const double* mp = rebase(met);
#pragma unroll
            for (int v = 0; v < NV; ++v) dma_dword(qp + v * vol, vol, &L.ring[slot][v][32 * h], loff[h] + qo);
            dma_dword(mp + (NMET - 1) * vol, vol, &L.ring[slot][NV][32 * h], loff[h] + mo);
#pragma unroll
            for (int c = 0; c < DIM; ++c)
                dma_dword(mp + (DIR * DIM + c) * vol, vol, &L.ring[slot][NV + 1 + c][32 * h], loff[h] + mo);
        }
    };
    for (int r = w; r < W::WIN; r += 4) load_row(tb + r);
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    staged();
    for (int r = w; r < W::WIN; r += 4)
        if (tb + r <= tmax) wg_convert(L, r, gm1);
    __syncthreads();
    for (int it = 0; it < iters; ++it) {
        const int f = k0 - 1 + 4 * it + w;
        if (it + 1 < iters) load_row(tb + W::WIN + 4 * it + w);  // a row of the next iteration
        // this wave's node f: its epilogue operands load while the face is
        // computed; 1/J, density and energy are in its ring row already
        const bool mine = lane_ok && f >= k0 && f < k1;
        const long noff = lb + (long)f * G.sd[DIR];
        EpiPre<NV> pre;
        if (mine) epi_load<NV>(ep, G.vol, noff, pre, !late_qin);
        double F[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) F[v] = 0.0;
        if (lane_ok && f < k1) {
            LdsLoader<DIM, wide_stencil(RECON, Y)> ld;
            ld.L = &L;
            ld.la = (unsigned)lane * 8u;
            ld.b0 = (f - 3 - tb + W::RING) % W::RING;
            face_flux<DIM, RECON, Y, char_t<PREC>>(ld, sk, F);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) L.flux[w][v][lane] = F[v];
        // this wave's row of the next iteration, asked for before the face
        __builtin_amdgcn_s_waitcnt(0);
        asm volatile("" ::: "memory");
        if (late_qin && mine) epi_load_qin<NV>(ep, G.vol, noff, pre);
        if (it + 1 < iters && tb + W::WIN + 4 * it + w <= tmax)
            wg_convert(L, (W::WIN + 4 * it + w) % W::RING, gm1);
        // First barrier: the fluxes and the next iteration's rows are in LDS.
        // Second: their readers are done, so that the next iteration may
        // overwrite them.  Only those reads lie between the two; the epilogue
        // and its stores follow, beside the next face.
        lds_barrier();
        double prev[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) prev[v] = (w > 0 ? &L.flux[w - 1][0][0] : &L.carry[0][0])[v * 64 + lane];
        if (ep.mode >= EPI_LAST_RES) {
            const double (*row)[64] = L.ring[(f - tb) % W::RING];
            pre.V = row[NV][lane];
            pre.qin[0] = row[0][lane];
            pre.qin[NV - 1] = row[NV - 1][lane];
        }
        lds_barrier();
        if (w == 3) {  // the next iteration's first face needs this one's last flux
#pragma unroll
            for (int v = 0; v < NV; ++v) L.carry[v][lane] = F[v];
        }
        if (mine) {
            double d[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) d[v] = F[v] - prev[v];
            epi_store<NV>(ep, G.vol, noff, pre, d);
        }
    }
}

// Work items (workgroups) of the eta / zeta sweep of one block.
inline long sweep_wg_items(const int n[3], int dir, int S) {
    const int oth = dir == 1 ? 2 : 1;
    const long lblocks = ((long)n[0] * n[oth] + 63) / 64;
    return lblocks * ((n[dir] + S - 1) / S);
}

// How the eta / zeta sweep of one block is split over `wgs` workgroups.
// Uniform: workgroup b takes segment b / lblocks, of S nodes, of line block
// b % lblocks.  Balanced: the nodes of all line blocks are numbered one block
// after another and each workgroup takes S of them, as one piece or, across
// the end of a line block, more.
struct WgSplit {
    int S;
    bool balanced;
    unsigned wgs;
};

// One launch of the eta / zeta sweep of one block, with its epilogue mode
// (EPI_*) fixed at compile time, as in the batched sweeps, so that only that
// epilogue's registers are allocated.
// (the loop over pieces costs registers, so the splits are kernels apart)
template <int DIM, int DIR, int RECON, int Y, int PREC, int MODE, bool BALANCED>
__global__ __launch_bounds__(256) FP_SWEEP_ATTR void k_sweep_wg(GeoK G, SchemeK sk,
                                                                const double* __restrict__ met,
                                                                const double* qs, EpiK ep, int S) {
    __shared__ WgLds<DIM, wide_stencil(RECON, Y)> lds;
    constexpr int OTH = DIR == 1 ? 2 : 1;
    EpiK e = ep;
    e.mode = MODE;
    const unsigned lblocks = (unsigned)(((long)G.n[0] * G.n[OTH] + 63) / 64);
    const int nd = G.n[DIR];
    const unsigned wg = (unsigned)xcd_block(blockIdx.x, gridDim.x);
    if constexpr (!BALANCED) {
        const int k0 = (int)(wg / lblocks) * S;
        sweep_wg_item<DIM, DIR, RECON, Y, PREC>(G, sk, met, qs, e, (int)(wg % lblocks), k0, min(k0 + S, nd), lds);
    } else {
        const unsigned u = wg * (unsigned)S;
        unsigned lineblk = u / (unsigned)nd;
        int k0 = (int)(u - lineblk * (unsigned)nd);
        for (int left = S; left > 0 && lineblk < lblocks; ++lineblk, k0 = 0) {
            const int k1 = min(nd, k0 + left);
            sweep_wg_item<DIM, DIR, RECON, Y, PREC>(G, sk, met, qs, e, (int)lineblk, k0, k1, lds);
            left -= k1 - k0;
            __syncthreads();  // the next piece rewrites the LDS ring
        }
    }
}

// ---------------------------------------------------------------------------
// both sweeps of a small 2D block in one launch
// ---------------------------------------------------------------------------
// A workgroup owns one row k of up to 56 nodes: wave 0 and 1 evaluate its
// eta faces k -+ 1/2, wave 2 the xi faces along it, from the stencil rows
// that all four waves stage in LDS (64 columns, four beyond the nodes on each
// side); wave 2 then forms both flux differences and applies the final
// epilogue, so the residual accumulator stays in registers.
// Why: on a block of a few thousand nodes a launch lasts as long as one
// chain of load, face and store, whatever its size, and this runs the two
// directions side by side: 7.5 us per RK stage of a 64^2 WENO5 block, launch
// gap included, against 13.9 for the two sweeps (and 10.2 for a workgroup
// that marches along j over a ring of rows, which was tried first).  It
// evaluates every eta face twice, so it pays while the chip has room.  The
// face code, its inputs and the order of the sums are those of the two
// sweeps: the results are bitwise theirs.
constexpr int kRowNodes = 56;
template <int WIDE>
struct RowLds {
    static constexpr int NC = 64;  // columns: x = i0 - 4 .. i0 + 59
    static constexpr int LO = WIDE ? 3 : 2, HI = WIDE ? 4 : 3;
    static constexpr int ROWS = 2 + LO + HI;  // nodes k - 1 - LO .. k + HI
    static constexpr int NS = 8;              // rho, u, v, E, 1/J, s_eta, thermal speed
    double row[ROWS][NS][NC];
    double sx[2][NC];        // s_xi of row k
    double flux[2][4][NC];   // the two eta faces
};

// Stencil reads of a face of either direction (eta: wave-uniform): slot r is
// row b0 + r, or column r of row k.
template <int WIDE>
struct RowLoader : StagedNodes<2, RowLoader<WIDE>> {
    static constexpr bool CT = true;
    using W = RowLds<WIDE>;
    const W* L;
    unsigned la;  // byte offset of this lane's column
    int b0;
    bool eta;

    __device__ __forceinline__ RowLoader after(double dep) const {
        RowLoader c = *this;
        asm volatile("" : "+v"(c.la) : "v"(dep));
        return c;
    }
    __device__ __forceinline__ double at(int r, int v) const {
        const bool s = v == 5 || v == 6;
        const unsigned eo = (unsigned)(((b0 + r) * W::NS + v) * W::NC) * 8u;
        const unsigned xo =
            s ? (unsigned)(W::ROWS * W::NS + v - 5) * W::NC * 8u + (unsigned)r * 8u
              : (unsigned)(((W::LO + 1) * W::NS + v) * W::NC + r) * 8u;
        return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(L) + la + (eta ? eo : xo));
    }
};

// One 2D residual evaluation with its final epilogue `ep` (MODE: EPI_LAST_RES
// or EPI_LAST_RK); ACC: the accumulator holds the viscous part already.
template <int RECON, int Y, int PREC, int MODE, bool ACC>
__global__ __launch_bounds__(256) FP_SWEEP_ATTR void k_row_2d(GeoK G, SchemeK sk, const double* __restrict__ met,
                                                              const double* qs, EpiK ep_, int ti) {
    using W = RowLds<wide_stencil(RECON, Y)>;
    constexpr int NV = 4;
    __shared__ W L;
    EpiK ep = ep_;
    ep.mode = MODE;
    const int lane = threadIdx.x & 63;
    const int w = wave_id();
    const int n0 = G.n[0], nd = G.n[1];
    const int tiles = (n0 + ti - 1) / ti;
    const int k = (int)(blockIdx.x / (unsigned)tiles);
    const int i0 = (int)(blockIdx.x % (unsigned)tiles) * ti, tw = min(ti, n0 - i0);  // nodes i0 .. i0 + tw - 1
    const long vol = G.vol;
    const int sd1 = (int)G.sd[1];
    const double gm1 = sk.gamma - 1.0;
    // DMA: lane l moves dword (l & 1) of column 32 p + l / 2 of a row.  The
    // state's columns wrap on a periodic axis; columns past the stored ghosts
    // (never read) repeat the last.
    unsigned cq[2], cm[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const int x = i0 - 4 + 32 * p + (lane >> 1);
        const int xm = min(max(x, -G.g), n0 - 1 + G.g);
        int xq = xm;
        if (G.bc[0] == 0) {
            xq = x < 0 ? x + n0 : (x >= n0 ? x - n0 : x);
            xq = min(max(xq, 0), n0 - 1);
        }
        cq[p] = (unsigned)(G.base + xq) * 8u + (unsigned)(lane & 1) * 4u;
        cm[p] = (unsigned)(G.base + xm) * 8u + (unsigned)(lane & 1) * 4u;
    }
    for (int r = w; r < W::ROWS; r += 4) {
        const int t = k - 1 - W::LO + r;
        int tt = t;
        if (G.bc[1] == 0) tt = t < 0 ? t + nd : (t >= nd ? t - nd : t);
        const unsigned qo = (unsigned)(tt * sd1) * 8u, mo = (unsigned)(t * sd1) * 8u;
        const double* qp = rebase(qs);
        const double* mp = rebase(met);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
#pragma unroll
            for (int v = 0; v < NV; ++v) dma_dword(qp + v * vol, vol, &L.row[r][v][32 * p], cq[p] + qo);
            dma_dword(mp + 4 * vol, vol, &L.row[r][4][32 * p], cm[p] + mo);
#pragma unroll
            for (int c = 0; c < 2; ++c) dma_dword(mp + (2 + c) * vol, vol, &L.row[r][5 + c][32 * p], cm[p] + mo);
            if (t == k) {
#pragma unroll
                for (int c = 0; c < 2; ++c) dma_dword(mp + c * vol, vol, &L.sx[c][32 * p], cm[p] + mo);
            }
        }
    }
    // wave 2, lane l >= 1, owns the node of column l - 1 of the tile, to the
    // right of its left face
    const bool mine = w == 2 && lane >= 1 && lane <= tw;
    const unsigned noff = (unsigned)(G.base + i0 + lane - 1 + k * sd1);
    EpiPre<NV> pre;
    if (mine) {
        if (ACC) {
            const double* R = rebase(ep.R);
#pragma unroll
            for (int v = 0; v < NV; ++v) pre.R[v] = ldb(R + v * vol, vol, noff * 8u);
        }
        if (MODE == EPI_LAST_RK) {
            epi_load_qin<NV>(ep, vol, noff, pre);
            if (!ep.stage0) {
                const double* qn = rebase(ep.qn);
#pragma unroll
                for (int v = 0; v < NV; ++v) pre.qn[v] = ldb(qn + v * vol, vol, noff * 8u);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    for (int r = w; r < W::ROWS; r += 4) {  // each wave converts the rows it brought
        double q[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) q[v] = L.row[r][v][lane];
        Prim<2> P;
        to_prim<2>(q, gm1, P);
        L.row[r][1][lane] = P.u[0];
        L.row[r][2][lane] = P.u[1];
        L.row[r][7][lane] = P.ct;
    }
    lds_barrier();
    double F[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) F[v] = 0.0;
    const bool eta = w < 2;
    if (w < 3 && (eta ? lane < tw : lane <= tw)) {
        RowLoader<wide_stencil(RECON, Y)> ld;
        ld.L = &L;
        ld.eta = eta;
        ld.la = (unsigned)(eta ? lane + 4 : lane) * 8u;
        ld.b0 = w - 3 + W::LO;  // face k - 1 + w + 1/2: slot r is node k - 1 + w - 3 + r
        SchemeK kd = sk;
        if (eta) kd.glf += kGlfDirStride;  // the direction's speeds
        face_flux<2, RECON, Y, char_t<PREC>>(ld, kd, F);
    }
    if (eta) {
#pragma unroll
        for (int v = 0; v < NV; ++v) L.flux[w][v][lane] = F[v];
    }
    double d[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) d[v] = F[v] - __shfl_up(F[v], 1, 64);
    lds_barrier();
    if (mine) {
        double dy[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            dy[v] = L.flux[1][v][lane - 1] - L.flux[0][v][lane - 1];
            pre.R[v] = ACC ? pre.R[v] - d[v] : -d[v];
        }
        pre.V = L.row[W::LO + 1][4][lane + 3];
        pre.qin[0] = L.row[W::LO + 1][0][lane + 3];
        pre.qin[NV - 1] = L.row[W::LO + 1][NV - 1][lane + 3];
        epi_store<NV>(ep, vol, noff, pre, dy);
    }
}

// Workgroups of the kernel above, and whether it takes the block: two rounds
// of the two that a CU holds.  us per stage against the two sweeps: WENO5 FP64
// in a residual call 170^2 (680 workgroups) 16.1 and 21.9, 30x1000 (1000) 18.7
// and 22.9; in an RK3 step 13.8 and 14.5, 16.5 and 16.9; in a captured step,
// whose launches cost least, 168^2 (504) 11.0 and 13.8, then 13.8 and 13.7,
// 17.0 and 16.1, and beyond the line 300^2 (1800) 28.8 and 18.0.
// WENO7 in a residual call 680 workgroups 19.0 and 21.5, 1000 22.9 and 24.0,
// captured 17.5 and 16.2, 21.6 and 19.5; LU5 captured 11.1 and 11.9, 13.5 and
// 13.3.
inline long row_2d_blocks(const int n[3]) { return (long)((n[0] + kRowNodes - 1) / kRowNodes) * n[1]; }
inline bool row_2d_fits(const int n[3]) { return row_2d_blocks(n) <= 1024; }

// ---------------------------------------------------------------------------
// global Lax-Friedrichs speeds
// ---------------------------------------------------------------------------

// faces per thread of the reduction (neighbours along the face direction)
constexpr int kGlfSeg = 4;

// Zero one speed set (a template: this header is compiled into several objects).
template <int DIM>
__global__ void k_glf_reset(unsigned long long* set) {
    if (threadIdx.x < 9) set[kGlfDirStride * (threadIdx.x / 3) + threadIdx.x % 3] = 0ull;
}

// The time of a captured step sequence, T = {t, t0, steps}: set before the
// replays; at the end of every step steps += 1 and t = t0 + steps dt (the
// step start times of an uncaptured run, without accumulated rounding).
__device__ __forceinline__ void time_advance(double* T, double dt) {
    const double n = T[2] + 1.0;
    T[2] = n;
    T[0] = T[1] + n * dt;
}

// velocity and sound speed of the node at `off` (NaN where the pressure is
// negative: such a node counts for the class u_n alone, as fmax drops NaN).
// One divided node serves up to six faces: plain divisions and roots here.
template <int DIM>
__device__ __forceinline__ void glf_node(const double* __restrict__ q, long vol, long off, double gamma, double* u,
                                         double& cs) {
    const double rho = q[off];
    double k2 = 0.0;
#pragma unroll
    for (int c = 0; c < DIM; ++c) {
        const double mc = q[(1 + c) * vol + off];
        u[c] = mc / rho;
        k2 += mc * u[c];
    }
    const double p = (gamma - 1.0) * (q[(DIM + 1) * vol + off] - 0.5 * k2);
    cs = sqrt(gamma * p / rho);
}

// The largest local Lax-Friedrichs speed over every face of every direction
// (faces f + 1/2, f = -1 .. n_d - 1, of every interior line), per field class
// (u_n - c, u_n, u_n + c): at each face the metric vector and 1/J are
// interpolated (order Y) as for the face's reference state, n = s_f/|s_f|,
// sigma = |s_f|/(1/J)_f, and the speeds sigma |n . u_m + kappa c_m| are
// maximised over the stencil nodes m = f - LO .. f + LO + 1.  As in the
// sweeps, the state's index wraps into the interior on a periodic axis (its
// ghost layers are not filled) and the metrics are read in place.
//
// Blocks [d bpd, (d + 1) bpd) take direction d, each XCD a range of faces
// contiguous in memory, as in the sweeps before and after (961x241: 54.3 ->
// 53.2 us per RK stage; a row kernel of 64^2 gained nothing by it).  A thread takes kGlfSeg
// neighbouring faces of one line and evaluates the velocity and sound speed
// of each node of their stencils once; consecutive threads take consecutive
// face pairs along the line for xi and neighbouring lines (contiguous in
// memory) for eta and zeta.  Each block reduces its maxima and folds them
// into `set` with one integer atomic max per class (non-negative doubles
// order as their bit patterns do): few large blocks, since atomics on one
// cache line serialise.  Four faces a thread evaluate 2.25 nodes per face
// (two faces: 3.5): 13.9 us against 15.7 on a 961x241 grid, where launch, load
// latency and the atomics are the rest.  (The one-step reciprocals and roots
// of the faces' basis would take 13.4: not worth their bits in a speed that
// every face of the block takes as its floor.)  Block 0 also zeroes `next` (the set the following
// reduction folds into; NULL: none) and, in the last stage of a captured
// step, advances the device time `T` that the next step starts from (NULL:
// none; a launch of its own took 4 us of a 190 us step).
template <int DIM, int Y, int LO>
__global__ __launch_bounds__(512) void k_glf(GeoK G, double gamma, const double* __restrict__ met,
                                              const double* __restrict__ q, unsigned long long* set,
                                              unsigned long long* next, int bpd, double* T, double dt) {
    constexpr int NMET = DIM == 3 ? 10 : 5;
    constexpr int NW = kGlfSeg + 2 * LO + 1;  // stencil nodes of one segment
    const int d = blockIdx.x / bpd, bb = (int)xcd_block(blockIdx.x % bpd, bpd);
    if (next && blockIdx.x == 0 && threadIdx.x < 9)
        next[kGlfDirStride * (threadIdx.x / 3) + threadIdx.x % 3] = 0ull;
    if (T && blockIdx.x == 0 && threadIdx.x == 0) time_advance(T, dt);
    const int e1 = d == 0 ? 1 : 0, e2 = d == 2 ? 1 : 2;
    const long n1 = G.n[e1], n12 = n1 * G.n[e2];
    const int nd = G.n[d];
    const int nseg = (nd + kGlfSeg) / kGlfSeg;  // segments of the n_d + 1 faces of a line
    const long total = (long)nseg * n12;
    const long sdd = G.sd[d];
    const bool per = G.bc[d] == 0;
    double m0 = 0.0, m1 = 0.0, m2 = 0.0;
    for (long t = (long)bb * blockDim.x + threadIdx.x; t < total; t += (long)bpd * blockDim.x) {
        long r;
        int seg;
        if (d == 0) {
            seg = (int)(t % nseg);
            r = t / nseg;
        } else {
            r = t % n12;
            seg = (int)(t / n12);
        }
        const int f0 = seg * kGlfSeg - 1;
        const long line = G.base + (r % n1) * G.sd[e1] + (r / n1) * G.sd[e2];
        double u[NW][DIM], cs[NW];
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            // nodes past the last face's stencil are never read: clamp them
            int p = min(f0 - LO + j, nd + LO);
            if (per) p = p < 0 ? p + nd : (p >= nd ? p - nd : p);
            glf_node<DIM>(q, G.vol, line + (long)p * sdd, gamma, u[j], cs[j]);
        }
#pragma unroll
        for (int j = 0; j < kGlfSeg; ++j) {
            const int f = f0 + j;
            if (f >= nd) break;
            double Vf = 0.0, sf[DIM];
#pragma unroll
            for (int c = 0; c < DIM; ++c) sf[c] = 0.0;
#pragma unroll
            for (int m = 0; m < Y; ++m) {
                const long off = line + (long)(f - Y / 2 + 1 + m) * sdd;
                const double w = iw<Y>(m + 4 - Y / 2);
                Vf += w * met[(NMET - 1) * G.vol + off];
#pragma unroll
                for (int c = 0; c < DIM; ++c) sf[c] += w * met[(d * DIM + c) * G.vol + off];
            }
            double s2 = 0.0;
#pragma unroll
            for (int c = 0; c < DIM; ++c) s2 += sf[c] * sf[c];
            const double sn = sqrt(s2);
            const double sigma = sn / Vf;
            double n[DIM];
#pragma unroll
            for (int c = 0; c < DIM; ++c) n[c] = sf[c] / sn;
#pragma unroll
            for (int m = 0; m <= 2 * LO + 1; ++m) {
                double un = 0.0;
#pragma unroll
                for (int c = 0; c < DIM; ++c) un += n[c] * u[j + m][c];
                m0 = fmax(m0, sigma * fabs(un - cs[j + m]));
                m1 = fmax(m1, sigma * fabs(un));
                m2 = fmax(m2, sigma * fabs(un + cs[j + m]));
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        m0 = fmax(m0, __shfl_xor(m0, o));
        m1 = fmax(m1, __shfl_xor(m1, o));
        m2 = fmax(m2, __shfl_xor(m2, o));
    }
    __shared__ double red[3][16];
    const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][w] = m0;
        red[1][w] = m1;
        red[2][w] = m2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int k = threadIdx.x;
        double v = 0.0;
        for (int i = 0; i < nw; ++i) v = fmax(v, red[k][i]);
        atomicMax(set + kGlfDirStride * d + k, (unsigned long long)__double_as_longlong(v));
    }
}

// ---------------------------------------------------------------------------
// batches: many blocks (of one dimensionality and scheme) in shared launches
// ---------------------------------------------------------------------------

// One block of a batch as the batched kernels see it.
struct BBlock {
    GeoK G;
    const double* met;
    double* q;  // Q^n, and the output of RK stage 3
    double* A;  // RK stage registers and residual accumulator (the workspace)
    double* B;
    double* R;
    double dt;
    int S[3];  // eta / zeta segment lengths
};

// Kinds of work items of a batched RK step.
enum { BK_X = 0, BK_ETA = 1, BK_ZETA = 2, BK_GHOST = 3, BK_KINDS = 4 };

// An interface between two blocks of a batch: the ghost layers of block a
// on `side` (0 low, 1 high) of `axis` are the interior layers of block b
// next to its opposite side (the blocks share the other axes' extents and
// orientation).
struct LinkK {
    int a, b, axis, side;
};

// Work-item table of a batch, in device memory.  The number of blocks and
// the prefix sums are read by the kernels at run time, so a captured graph
// stays valid when the table's contents change:
//   *nblk                      blocks in use;
//   start[k * (cap + 1) + b]   first item of block b in kind k; entry nblk is
//                              the kind's total;
//   blk[b]                     the block.
struct BTab {
    const int* nblk;
    const long* start;
    const BBlock* blk;
    int cap;
    unsigned* next;  // per kind, kNextPitch apart: items taken beyond each workgroup's first
};
constexpr int kNextPitch = 32;

// The order of the blocks within a kind's work list: position n of kind k
// holds block kind_order(...)[n] (the list of a kind may put its blocks in
// any order; the eta / zeta lists put the blocks with the longest items
// first, so that the last ones to be taken are short).
// The array follows the prefix sums in the same table.
__device__ __forceinline__ const int* kind_order(const long* t_start, int cap, int kind) {
    return reinterpret_cast<const int*>(t_start + BK_KINDS * (cap + 1)) + kind * cap;
}

// Block of `item` at or after block b, for items that only increase.
__device__ __forceinline__ int advance_block(const long* st, int nblk, int b, long item) {
    while (b + 1 < nblk && st[b + 1] <= item) ++b;
    return b;
}

// Largest b in [0, nblk) with st[b] <= item (blocks without items of a kind
// have st[b] == st[b + 1] and are skipped).
__device__ __forceinline__ int find_block(const long* st, int nblk, long item) {
    int lo = 0, hi = nblk - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (st[mid] <= item)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

__device__ __forceinline__ const double* stage_in(const BBlock& b, int stage) {
    return stage == 0 ? b.q : (stage == 1 ? b.A : b.B);
}

// The epilogue of a sweep of RK stage `stage` (TVD RK3 in Shu-Osher form:
// stage 1 writes A, stage 2 B, stage 3 q), the same values the single-block
// driver uses.
__device__ __forceinline__ EpiK stage_epi(const BBlock& b, int stage, int mode, int ndim) {
    EpiK e;
    e.mode = mode;
    e.stage0 = stage == 0;
    e.R = b.R;
    e.out = stage == 0 ? b.A : (stage == 1 ? b.B : b.q);
    e.qin = stage_in(b, stage);
    e.qn = b.q;
    e.dt = b.dt;
    e.a = stage == 0 ? 0.0 : (stage == 1 ? 3.0 / 4.0 : 1.0 / 3.0);
    e.b = stage == 0 ? 1.0 : (stage == 1 ? 1.0 / 4.0 : 2.0 / 3.0);
    return e;
}

// Persistent batched xi sweep of one RK stage: wave w of the grid takes the
// batch's wave items w, w + (waves of the grid), ..., staging the next item
// (possibly of another block) while it computes.
template <int DIM, int RECON, int Y, int PREC>
__global__ __launch_bounds__(256) FP_XSWEEP_ATTR(PREC, RECON, Y) void kb_sweep_x(const int* __restrict__ t_nblk,
                                                                const long* __restrict__ t_start,
                                                                const BBlock* __restrict__ t_blk, int cap,
                                                                SchemeK sk, int stage) {
    constexpr int NE = x_entries(PREC, RECON, Y);
    __shared__ XLds<DIM, NE> lds[4];
    XLds<DIM, NE>& L = lds[wave_id()];
    const int nblk = *t_nblk;
    const long* __restrict__ st = t_start + BK_X * (cap + 1);
    const long total = st[nblk];
    const int* __restrict__ ord = kind_order(t_start, cap, BK_X);
    const long nw = (long)gridDim.x * 4;
    long item = (long)blockIdx.x * 4 + wave_id();
    int cur = 0;
    int b = 0;
    if (item >= total) return;
    b = find_block(st, nblk, item);
    XPos pos, step;
    XItem it;
    {
        const BBlock& B = t_blk[ord[b]];
        const unsigned W1 = (unsigned)B.G.xw - 1;
        pos = x_pos(B.G, (unsigned)(item - st[b]) * W1);
        step = x_pos(B.G, (unsigned)nw * W1);
        it = x_item<NE>(B.G, pos);
        x_stage<DIM, NE>(B.G, B.met, stage_in(B, stage), it, L.b[0]);
    }
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    for (; item < total; item += nw, cur ^= 1) {
        int bn = b;
        XItem next = it;
        if (item + nw < total) {
            bn = advance_block(st, nblk, b, item + nw);
            const BBlock& N = t_blk[ord[bn]];
            if (bn == b) {
                x_advance(N.G, step, pos);
            } else {
                const unsigned W1 = (unsigned)N.G.xw - 1;
                pos = x_pos(N.G, (unsigned)(item + nw - st[bn]) * W1);
                step = x_pos(N.G, (unsigned)nw * W1);
            }
            next = x_item<NE>(N.G, pos);
            x_stage<DIM, NE>(N.G, N.met, stage_in(N, stage), next, L.b[cur ^ 1]);
        }
        const BBlock& B = t_blk[ord[b]];
        const EpiK ep = stage_epi(B, stage, EPI_FIRST, DIM);
        x_compute<DIM, RECON, Y, PREC, false>(B.G, sk, ep, it, L.b[cur], L.ct);
        b = bn;
        it = next;
    }
}

// Persistent batched eta / zeta sweep of one RK stage; the last direction
// applies the RK3 update.  A long list is handed out: after its first item a
// workgroup takes the next one nobody has, so none is left with a run of long
// items at the end (48 body blocks, 20 million nodes: 9.30 -> 9.00 ms per
// step).  The counter is asked beside the item's first loads and its answer
// read when the item ends.  Every workgroup with a first item asks until it is
// refused, `total` times in all, so the one that gets total - 1 is the last
// and sets the counter back.  A short list is dealt out in turn: all
// workgroups ask at once at first, 11 ns each, and few items follow to make up
// for it (24 serving blocks, few items per workgroup, handed out: 4.84 ->
// 4.93 ms for five steps).  The xi sweep's items are too small to be
// handed out: the same serving blocks took 9.1 ms.
// Two workgroups per CU, but one for FP64 WENO7 in 3D, which spills some 45
// registers at two and none with the registers of one: 16 body blocks 26.7 ms
// per step against 36.2, 12 serving blocks 2.02 against 2.46.  The other wide
// FP64 stencils spill eight at most: WENO5 with eighth-order metrics 20.6 ms
// with one workgroup, 19.4 with two, WENOCU6 27.0 and 26.0, LU5 15.1 and 13.7.
#define FP_BWAVES(DIM, RECON, PREC) ((DIM) == 3 && (RECON) == 2 && (PREC) == 0 ? 1 : 2)
template <int DIM, int DIR, int RECON, int Y, int PREC>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(FP_BWAVES(DIM, RECON, PREC), FP_BWAVES(DIM, RECON, PREC))))
void kb_sweep_wg(const int* __restrict__ t_nblk, const long* __restrict__ t_start,
                 const BBlock* __restrict__ t_blk, int cap, SchemeK sk, int stage, unsigned* next) {
    __shared__ WgLds<DIM, wide_stencil(RECON, Y)> lds;
    constexpr int KIND = DIR == 1 ? BK_ETA : BK_ZETA;
    constexpr int MODE = DIR == DIM - 1 ? EPI_LAST_RK : EPI_MID;
    const int nblk = *t_nblk;
    const long* __restrict__ st = t_start + KIND * (cap + 1);
    const unsigned total = (unsigned)st[nblk];
    const int* __restrict__ ord = kind_order(t_start, cap, KIND);
    if (blockIdx.x >= total) return;
    const bool handed = total > 6 * gridDim.x;
    int b = find_block(st, nblk, blockIdx.x);
    for (unsigned item = blockIdx.x; item < total;) {
        b = advance_block(st, nblk, b, item);
        const BBlock& B = t_blk[ord[b]];
        const EpiK ep = stage_epi(B, stage, MODE, DIM);
        constexpr int OTH = DIR == 1 ? 2 : 1;
        const unsigned lblocks = (unsigned)(((long)B.G.n[0] * B.G.n[OTH] + 63) / 64);
        const unsigned in = item - (unsigned)st[b];
        const int k0 = (int)(in / lblocks) * B.S[DIR];
        unsigned c = 0, taken = 0;
        if (handed && threadIdx.x == 0)
            c = __hip_atomic_fetch_add(next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sweep_wg_item<DIM, DIR, RECON, Y, PREC>(B.G, sk, B.met, stage_in(B, stage), ep, (int)(in % lblocks), k0,
                                                min(k0 + B.S[DIR], B.G.n[DIR]), lds, [&] {
                                                    taken = (unsigned)__builtin_amdgcn_readfirstlane((int)c);
                                                    if (handed && threadIdx.x == 0 && c + 1 == total)
                                                        __hip_atomic_store(next, 0u, __ATOMIC_RELAXED,
                                                                           __HIP_MEMORY_SCOPE_AGENT);
                                                });
        if (handed) {
            // the answer, in a scalar register of the first wave, goes round
            // through a flux that has been read and is written again only
            // after the next item's first barrier: a word of LDS more would
            // leave wide 3D stencils one workgroup per CU
            unsigned* word = reinterpret_cast<unsigned*>(&lds.flux[0][0][0]);
            if (threadIdx.x == 0) *word = taken;
            __syncthreads();
            item = (unsigned)__builtin_amdgcn_readfirstlane((int)*word) + gridDim.x;
        } else {
            __syncthreads();  // the next item rewrites the LDS ring
            item += gridDim.x;
        }
    }
}

// Every face of direction DIR, one lane per face, lanes along i (coalesced):
// the face fluxes of fp_face_fluxes.
template <int DIM, int DIR, int RECON, int Y, int PREC>
__global__ __launch_bounds__(256) FP_SWEEP_ATTR void k_face_flux(GeoK G, SchemeK sk,
                                                                 const double* __restrict__ met,
                                                                 const double* qs, double* out) {
    constexpr int NV = DIM + 2;
    int ext[3] = {G.n[0], G.n[1], G.n[2]};
    ext[DIR] += 1;
    const long total = (long)ext[0] * ext[1] * ext[2];
    const long tid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (tid >= total) return;
    int c[3];
    c[0] = (int)(tid % ext[0]);
    c[1] = (int)((tid / ext[0]) % ext[1]);
    c[2] = (int)(tid / ((long)ext[0] * ext[1]));
    long lb = G.base;
#pragma unroll
    for (int d = 0; d < 3; ++d)
        if (d != DIR) lb += (long)c[d] * G.sd[d];
    const LineLoader<DIM, DIR> ld(G, met, qs, lb, c[DIR] - 1, sk.gamma);
    double fl[NV];
    face_flux<DIM, RECON, Y, char_t<PREC>>(ld, sk, fl);
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v * total + tid] = fl[v];
}

// ---------------------------------------------------------------------------
// launch helpers (defined in the instantiation units)
// ---------------------------------------------------------------------------

// Launch timing of an instrumented step: after each launch the host records
// an event on the stream and the launch's kind (kinds as fp_profile_step
// reports them).  The first error stops the recording.
enum {
    PK_XI = 0, PK_ETA = 1, PK_ZETA = 2, PK_GHOST = 3, PK_GLF = 5, PK_BC = 6, PK_VFLUX = 7, PK_VDIV = 8,
    PK_GLF_RESET = 9
};
struct Probe {
    hipEvent_t* ev;  // ev[0] is recorded before the first launch; ev[i + 1] after launch i
    int32_t* kind;
    int n, cap;
    hipError_t err;
};
inline void probe_mark(Probe* p, int kind, hipStream_t s) {
    if (!p || p->err != hipSuccess) return;
    if (p->n >= p->cap) {
        p->err = hipErrorInvalidValue;
        return;
    }
    p->err = hipGetLastError();
    if (p->err == hipSuccess) p->err = hipEventRecord(p->ev[p->n + 1], s);
    if (p->err == hipSuccess) p->kind[p->n++] = kind;
}

struct SweepArgs {
    GeoK G;
    SchemeK sk;
    const double* met;
    const double* qs;
    EpiK ep_first, ep_mid, ep_last;
    WgSplit split[3];
    int glf;  // 1: reduce the global LF speeds of the stage input into sk.glf first
    double* glf_next;  // the speed set the reduction zeroes for the next stage (or NULL)
    double* glf_time;  // the device time the reduction advances by time_dt (or NULL)
    double time_dt;
    Probe* probe;      // instrumented step (or NULL)
};

// one full residual evaluation (all sweeps) of the given instantiation
using stage_fn = hipError_t (*)(const SweepArgs&, hipStream_t);
using faceflux_fn = hipError_t (*)(const GeoK&, const SchemeK&, const double*, const double*,
                                   double*, hipStream_t);
// one direction sweep of the given instantiation with epilogue `ep`
using dir_fn = hipError_t (*)(const SweepArgs&, int dir, const EpiK& ep, hipStream_t);

// one RK stage of a batch part: the xi, eta (and zeta) persistent sweeps,
// grid[k] workgroups for sweep kind k; only >= 0 launches that kind alone
using batch_stage_fn = hipError_t (*)(const BTab&, const SchemeK&, int stage, const int grid[3],
                                      int only, hipStream_t);
// resident workgroups per CU of the batched sweep of kind k
using batch_occ_fn = int (*)(int kind);

stage_fn get_stage_fn(int ndim, int recon, int Y, int prec);
batch_stage_fn get_batch_stage_fn(int ndim, int recon, int Y, int prec);
batch_occ_fn get_batch_occ_fn(int ndim, int recon, int Y, int prec);
faceflux_fn get_faceflux_fn(int ndim, int dir, int recon, int Y, int prec);
dir_fn get_dir_fn(int ndim, int recon, int Y, int prec);

}  // namespace fpk
