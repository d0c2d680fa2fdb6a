// Particle kernels for gfx950: staggered trilinear gather, relativistic
// Boris push, move, and charge-conserving (Esirkepov, first-order shape)
// current deposition; counting sort of the particles by cell.
//
// Gather.  E^n and B^n = mu0 (H^{n-1/2} + H^{n+1/2})/2 are interpolated on
// each component's own staggered lattice.  The H update also writes the
// average of its two time levels inside the particle box, so B costs one
// array per component.  Along x the two corners of a trilinear stencil are
// adjacent in memory and are fetched with one 8-byte load (4 per component
// instead of 8); a periodic x axis, where the pair can wrap, uses 4-byte loads.
//
// Deposit.  A move x0 -> x1 shorter than one cell touches at most three
// nodes per axis, [b, b+2] with b = min(floor x0, floor x1).  Its current is
// 18 Jx + 18 Jy + 18 Jz edge values on that window, each a product of one
// factor per axis.  Particles are kept sorted by cell, so the lanes of a
// wavefront mostly share a grid row: the sum over the particles of a row is a
// small matrix product (x factors times transverse factors) and runs on the
// matrix cores in FP32 (deposit_rows).  Rows with few lanes use per-lane
// atomics.  Few particles are spread over more wavefronts (k_push_split).  The
// fixed-point deposit sums integers, exactly, as signed bytes on the matrix
// cores (deposit_fixed).
#include "pic_internal.hpp"

namespace pic {

// Index on a periodic axis: a move is shorter than a cell, so window indices
// reach from -1 to n + 1, which is 2 periods away when n = 1.  (No remainder: an
// integer division per node took longer than the rest of an edge row's indices.)
__device__ __forceinline__ int wrapn(int i, int n)
{
    i += i < 0 ? n : 0;
    i -= i >= n ? n : 0;
    return i >= n ? i - n : i;
}

// Fold a finite coordinate that moved less than one period back into [0, n).
__device__ __forceinline__ float fold(float v, int n)
{
    const float L = (float)n;
    if (v >= L) v -= L;
    if (v < 0.f) v += L;
    return v >= L ? 0.f : v;  // v + L may round up to L
}

// Per-axis corner data of the trilinear gather on the two lattices an axis
// can carry: nodes (h = 0) and half nodes (h = 1).  o0/o1 are the linear
// offsets of the two corners (clamped into the box), m0/m1 their weights
// with the wall mask folded in (0 for a corner beyond a wall).
struct Axis2 {
    int o0[2], o1[2];
    float m0[2], m1[2];
};

__device__ __forceinline__ void axis_corners(float x, int n, int per, int stride, Axis2 &A)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float s = h ? x - 0.5f : x;
        const float f = floorf(s);
        const int i = (int)f;
        const float w1 = s - f, w0 = 1.f - w1;
        int i0 = i, i1 = i + 1;
        bool ok0 = i0 >= 0 && i0 < n, ok1 = i1 >= 0 && i1 < n;
        if (per) {
            i0 = i0 < 0 ? i0 + n : (i0 >= n ? i0 - n : i0);
            i1 = i1 < 0 ? i1 + n : (i1 >= n ? i1 - n : i1);
            ok0 = ok1 = true;
        }
        i0 = min(max(i0, 0), n - 1);
        i1 = min(max(i1, 0), n - 1);
        A.o0[h] = i0 * stride;
        A.o1[h] = i1 * stride;
        A.m0[h] = ok0 ? w0 : 0.f;
        A.m1[h] = ok1 ? w1 : 0.f;
    }
}

// x corners as one adjacent pair (st, st+1), st in [0, nx-2] (nx >= 2 on a
// wall axis), with the weights of the two loaded values; a corner beyond a
// wall gets weight 0.
struct XPair {
    int o[2];
    float wa[2], wb[2];
};

__device__ __forceinline__ void x_pairs(float x, int nx, XPair &P)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float s = h ? x - 0.5f : x;
        const float f = floorf(s);
        const int i = (int)f;
        const float w1 = s - f, w0 = 1.f - w1;
        const int st = min(max(i, 0), nx - 2);
        // i == st: both corners in the pair; i < st (i = -1): corner 0 = st
        // carries w1; i > st (i = nx-1): corner nx-1 = st+1 carries w0
        P.o[h] = st;
        P.wa[h] = i == st ? w0 : (i < st ? w1 : 0.f);
        P.wb[h] = i == st ? w1 : (i < st ? 0.f : w0);
    }
}

// dword-aligned 8-byte global load
typedef float float2_a4 __attribute__((ext_vector_type(2), aligned(4)));
__device__ __forceinline__ float2 ld2(const float *p)
{
    const float2_a4 v = *(gp<const float2_a4>)G(p);
    return make_float2(v.x, v.y);
}

// Trilinear value of a component that sits at half nodes along the axes
// flagged (HX, HY, HZ).  The fused operations are written out, in the gathers and
// where the split push puts a value together (quad_pair, quad_scalar), so that every
// kernel rounds alike: a particle's kick does not depend on which one pushes it.
template <int HX, int HY, int HZ>
__device__ __forceinline__ float gather_pair(const float *__restrict__ f, const XPair &X,
                                             const Axis2 &Y, const Axis2 &Z)
{
    float v = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int o = X.o[HX] + (b ? Y.o1[HY] : Y.o0[HY]) + (c ? Z.o1[HZ] : Z.o0[HZ]);
            const float w = (b ? Y.m1[HY] : Y.m0[HY]) * (c ? Z.m1[HZ] : Z.m0[HZ]);
            const float2 p = ld2(f + o);
            v = fmaf(w, fmaf(X.wa[HX], p.x, X.wb[HX] * p.y), v);
        }
    return v;
}

template <int HX, int HY, int HZ>
__device__ __forceinline__ float gather_scalar(const float *__restrict__ f, const Axis2 &X,
                                               const Axis2 &Y, const Axis2 &Z)
{
    float v = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int o = (q ? X.o1[HX] : X.o0[HX]) + (b ? Y.o1[HY] : Y.o0[HY]) +
                              (c ? Z.o1[HZ] : Z.o0[HZ]);
                const float w = (q ? X.m1[HX] : X.m0[HX]) * (b ? Y.m1[HY] : Y.m0[HY]) *
                                (c ? Z.m1[HZ] : Z.m0[HZ]);
                v = fmaf(w, G(f)[o], v);
            }
    return v;
}

__device__ __forceinline__ float clamp01(float v) { return __builtin_amdgcn_fmed3f(v, 0.f, 1.f); }

// Esirkepov factors of one axis of a move x0 -> x1 on the 3-node window
// starting at node `base`, with S0, S1 the first-order shapes before and after
// and dS = S1 - S0: A = (S0 + S1)/2 and D = dS / sqrt(12) per node, and the
// running sum P of dS per edge.  The transverse weight of two axes is
//   S0 S0' + (dS S0' + S0 dS')/2 + dS dS'/3 = A A' + D D',
// and an edge current is P (its own axis) times that of the other two.
struct AxisF {
    float A[3], D[3], P[2];
};
constexpr float RSQRT12 = 0.28867513459481287f;

__device__ __forceinline__ AxisF axis_factors(float x0, float x1, int base)
{
    const float r0 = x0 - (float)base, r1 = x1 - (float)base;
    float dS[3];
    AxisF f;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const float s0 = clamp01(1.f - fabsf(r0 - (float)m));
        const float s1 = clamp01(1.f - fabsf(r1 - (float)m));
        dS[m] = s1 - s0;
        f.A[m] = 0.5f * (s0 + s1);
        f.D[m] = RSQRT12 * dS[m];
    }
    f.P[0] = dS[0];
    f.P[1] = dS[0] + dS[1];
    return f;
}

// The same for one node or edge at grid position n.
struct SlotF {
    float A, D, P;
};
__device__ __forceinline__ SlotF slot_factors(float x0, float x1, int n)
{
    const float e0 = x0 - (float)n, e1 = x1 - (float)n;
    const float s0 = clamp01(1.f - fabsf(e0)), s1 = clamp01(1.f - fabsf(e1));
    return {0.5f * (s0 + s1), RSQRT12 * (s1 - s0), clamp01(1.f - e1) - clamp01(1.f - e0)};
}

// Slot s (0..53) of the deposit window: component and offsets from the base node, the
// 2 edges or 3 nodes along x of a grid row side by side.
//   Jx: s = 6 b + 2 c + a         (edge a in 0..1, nodes b, c in 0..2)
//   Jy: s = 18 + 9 m + 3 c + a    (node a, edge m, node c)
//   Jz: s = 36 + 6 b + 3 m + a    (nodes a, b, edge m)
__device__ __forceinline__ void slot_geom(int s, int &comp, int &oi, int &oj, int &ok)
{
    if (s < 18) {
        comp = 0;
        oi = s % 2;
        oj = s / 6;
        ok = (s / 2) % 3;
    } else if (s < 36) {
        const int t = s - 18;
        comp = 1;
        oi = t % 3;
        oj = t / 9;
        ok = (t / 3) % 3;
    } else {
        const int t = s - 36;
        comp = 2;
        oi = t % 3;
        oj = t / 6;
        ok = (t / 3) % 2;
    }
}

// Current of slot s of a move with factors fx, fy, fz, per unit charge factor.
__device__ __forceinline__ float slot_value(const AxisF &fx, const AxisF &fy, const AxisF &fz, int s)
{
    int comp, oi, oj, ok;
    slot_geom(s, comp, oi, oj, ok);
    if (comp == 0) return fx.P[oi] * (fy.A[oj] * fz.A[ok] + fy.D[oj] * fz.D[ok]);
    if (comp == 1) return fy.P[oj] * (fx.A[oi] * fz.A[ok] + fx.D[oi] * fz.D[ok]);
    return fz.P[ok] * (fx.A[oi] * fy.A[oj] + fx.D[oi] * fy.D[oj]);
}

// Cell index of slot s of the window at (bx, by, bz) after wrapping, or -1
// when it falls outside the grid on a non-periodic axis.
__device__ __forceinline__ int slot_index(const PartArgs &a, int s, int bx, int by, int bz, int &comp)
{
    int oi, oj, ok;
    slot_geom(s, comp, oi, oj, ok);
    int i = bx + oi, j = by + oj, k = bz + ok;
    if (a.per[0]) i = wrapn(i, a.nx);
    else if (i < 0 || i >= a.nx) return -1;
    if (a.per[1]) j = wrapn(j, a.ny);
    else if (j < 0 || j >= a.ny) return -1;
    if (a.per[2]) k = wrapn(k, a.nz);
    else if (k < 0 || k >= a.nz) return -1;
    return i + a.nx * (j + a.ny * k);
}

// Fixed-point deposit: each particle's slot currents are rounded to integer
// units (qscale per V/m, at most 2^24 per slot) before anything is summed, so
// the wavefront sums (at most 2^30) and the 64-bit atomics are exact and the
// result does not depend on which lanes are summed together or on atomic order.
__device__ __forceinline__ void add_fixed(const PartArgs &a, int comp, int q, int units)
{
    unsigned long long *J = comp == 0 ? a.Jq[0] : (comp == 1 ? a.Jq[1] : a.Jq[2]);
    gatomic_add(G(J) + q, (unsigned long long)(long long)units);
}

// Where the three nodes of a window along one axis are stored: linear offsets,
// and whether the node is inside the grid (after wrapping).
struct AxisO {
    int o[3];
    bool ok[3];
};

__device__ __forceinline__ AxisO axis_offsets(int base, int n, int per, int stride)
{
    AxisO r;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const int i = per ? wrapn(base + m, n) : base + m;
        r.ok[m] = i >= 0 && i < n;
        r.o[m] = r.ok[m] ? i * stride : 0;
    }
    return r;
}

// The factors of nodes (and edges) outside the grid set to 0.
__device__ __forceinline__ void mask_outside(AxisF &f, const AxisO &o)
{
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        f.A[m] = o.ok[m] ? f.A[m] : 0.f;
        f.D[m] = o.ok[m] ? f.D[m] : 0.f;
        if (m < 2) f.P[m] = o.ok[m] ? f.P[m] : 0.f;
    }
}

// Window slots of one lane added with per-lane atomics: val(c) is what is added for
// the slot current c, add(comp, cell, v) the atomic.  Slots outside the grid are 0 by
// their factors (three tests in each of the 54 took 200 particles in 96x64x96 cells
// from 7.9 to 11.2 us).
template <class V, class Add>
__device__ __forceinline__ void lane_deposit(const PartArgs &a, const int base[3], AxisF fx, AxisF fy, AxisF fz, V val,
                                             Add add)
{
    const AxisO ox = axis_offsets(base[0], a.nx, a.per[0], 1);
    const AxisO oy = axis_offsets(base[1], a.ny, a.per[1], a.nx);
    const AxisO oz = axis_offsets(base[2], a.nz, a.per[2], a.nx * a.ny);
    mask_outside(fx, ox);
    mask_outside(fy, oy);
    mask_outside(fz, oz);
#pragma unroll
    for (int s = 0; s < 54; ++s) {
        int comp, oi, oj, ok;
        slot_geom(s, comp, oi, oj, ok);
        const auto c = val(slot_value(fx, fy, fz, s));
        if (c != 0) add(comp, ox.o[oi] + (oy.o[oj] + oz.o[ok]), c);
    }
}

// The same with the particle in the 3 lanes of q = 0..2, each for the slots of z
// node (Jx, Jy) or z edge (Jz) q.
__device__ __forceinline__ void quarter_deposit(const PartArgs &a, int q, const int base[3], float x0, float y0,
                                                float z0, float x1, float y1, float z1)
{
    const AxisO ox = axis_offsets(base[0], a.nx, a.per[0], 1);
    const AxisO oy = axis_offsets(base[1], a.ny, a.per[1], a.nx);
    int k = base[2] + q;
    const AxisF fx = axis_factors(x0, x1, base[0]), fy = axis_factors(y0, y1, base[1]);
    const SlotF fz = slot_factors(z0, z1, k);
    if (a.per[2]) k = wrapn(k, a.nz);
    if (q > 2 || (unsigned)k >= (unsigned)a.nz) return;
    const int oz = k * a.nx * a.ny;
    const float P = q < 2 ? fz.P : 0.f;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (!(ox.ok[i] && oy.ok[j])) continue;
            const int o = oz + oy.o[j] + ox.o[i];
            const float jx = i < 2 ? fx.P[i < 2 ? i : 0] * (fy.A[j] * fz.A + fy.D[j] * fz.D) : 0.f;
            const float jy = j < 2 ? fy.P[j < 2 ? j : 0] * (fx.A[i] * fz.A + fx.D[i] * fz.D) : 0.f;
            const float jz = P * (fx.A[i] * fy.A[j] + fx.D[i] * fy.D[j]);
            if (jx != 0.f) gatomic_add(G(a.Jb[0]) + o, a.qd * jx);
            if (jy != 0.f) gatomic_add(G(a.Jb[1]) + o, a.qd * jy);
            if (jz != 0.f) gatomic_add(G(a.Jb[2]) + o, a.qd * jz);
        }
}

// ---- deposit of the lanes of one grid row (matrix cores) ----
// The lanes of a pass share their windows' y and z base (by, bz) and have x
// bases in [X0, X0 + 13], so their windows lie on 16 x nodes X0 + t.  Every
// edge current is a sum over the particles p of (x factor at t) times
// (transverse factor of the slot):
//   Jx[b, c](t) = sum_p Px[p](t) (Ay[p,b] Az[p,c] + Dy[p,b] Dz[p,c])
//   Jy[m, c](t) = sum_p Ax[p](t) Py[p,m] Az[p,c] + Dx[p](t) Py[p,m] Dz[p,c]
//   Jz[m, b](t) = sum_p Ax[p](t) Pz[p,m] Ay[p,b] + Dx[p](t) Pz[p,m] Dy[p,b]
// v_mfma_f32_16x16x4_f32 takes 4 particles at a time: rows are slots (the 9 of
// Jx; the 6 + 6 of Jy and Jz), columns the 16 x nodes.  Lane l holds row or
// column l % 16 of particle l / 16, so the particles' factors pass from their
// own lanes through LDS, and the x factors are evaluated at node t from x0, x1
// (a particle outside the pass is put far away, where they are 0).  Products
// and sums are FP32, each sum of at most 64 terms.
//
// The push issues VALU at 0.7 of the peak beside the gather's vector-cache accesses
// (a tile of the fields in LDS took 12 % of the one and 86 % of the other, and up to a
// fifth of the time), so what counts here is instructions: a
// pass takes about 220 VALU and 48 MFMA (1536 matrix-core cycles, beside other
// wavefronts' VALU) whatever the number and order of the windows, where summing
// every slot over the lanes takes 324 for one ordered row and 220 per window
// otherwise.  512x256x256 cells, 1e7 particles: 351 -> 276 us per launch; 1e6
// particles in a 64x128x128 box periodic along x: 94 -> 63 us.
constexpr int ROW_NODES = 16;
constexpr int ROW_BASES = ROW_NODES - 2;
// Rows with fewer lanes go to the per-lane atomics (lane_deposit), whose cost does not depend
// on how many rows they come from: a pass costs a wavefront a chain of LDS reads
// and matrix products and eight atomics, and the wavefronts of a bunch's tails
// hold many short rows.  Push of 1e5 particles in a 128x64x64 box, the slowest
// wavefronts' time, for a least number of 3, 6, 10, 20 lanes: 19.5, 15.7, 14.3,
// 14.0 us; 1e6 in 64x128x128: 55.4, 52.2, 52.4, 59.4; 1e7 in 512x256x256: 272,
// 271, 270, 273.
constexpr int ROW_LANES = 10;

typedef float fvec4 __attribute__((ext_vector_type(4)));
constexpr float ROW_FAR = 1e9f;

struct RowLds {
    float4 pair[64][3];  // per particle (A, D) at y nodes 0..2, then z nodes 0..2
    float4 pre[64];      // Py[0], Py[1], Pz[0], Pz[1]
    float2 x[64];        // x0, x1
};

__device__ __forceinline__ void row_factors(RowLds &L, int p, const AxisF &fy, const AxisF &fz)
{
    L.pair[p][0] = make_float4(fy.A[0], fy.D[0], fy.A[1], fy.D[1]);
    L.pair[p][1] = make_float4(fy.A[2], fy.D[2], fz.A[0], fz.D[0]);
    L.pair[p][2] = make_float4(fz.A[1], fz.D[1], fz.A[2], fz.D[2]);
    L.pre[p] = make_float4(fy.P[0], fy.P[1], fz.P[0], fz.P[1]);
}

// Adds the 16 particles from p0 on to the sums of a pass whose first x node is
// X0.  MASK: only those whose bit of m16 is set (otherwise L.x has the rest far
// away).
template <bool MASK>
__device__ __forceinline__ void row_chunk(const RowLds &L, int p0, unsigned m16, int lane, int X0, bool yz, fvec4 &jx,
                                          fvec4 &jyz)
{
    const int t = lane & 15, q = lane >> 4;
    // Row t of Jx is (b, c) = (t/2, t%3) for t < 6 and (t - 6, 8 - t) for t =
    // 6..8; row t of Jy, Jz is edge m = t/3, z node c = t%3 of Jy for t < 6,
    // edge (t-6)/3, y node (t-6)%3 of Jz for t = 6..11.  So both use the pair n1
    // (the Jy / Jz row's node), Jx with the other axis's pair n2.
    const int n1 = t < 6 ? 3 + t % 3 : (t < 12 ? (t - 6) % 3 : 0);
    const int n2 = t < 6 ? t >> 1 : (t < 9 ? 11 - t : 0);
    const int np = min(t / 3, 3);
    const float2 *pairs = reinterpret_cast<const float2 *>(L.pair) + q * 6;
    const float *pres = reinterpret_cast<const float *>(L.pre) + q * 4 + np;
    const float ct = (float)(X0 + t);
    const unsigned mq = m16 >> q;
    float2 v1[4], v2[4], xx[4];
    float pr[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int p = p0 + 4 * g;
        v1[g] = pairs[p * 6 + n1];
        v2[g] = pairs[p * 6 + n2];
        xx[g] = L.x[p + q];
        pr[g] = pres[p * 4];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const bool in = !MASK || ((mq >> (4 * g)) & 1u);
        const float e0 = in ? xx[g].x - ct : ROW_FAR, e1 = in ? xx[g].y - ct : ROW_FAR;
        // running sums of the shapes up to node t, after less before
        const float px = clamp01(1.f - e1) - clamp01(1.f - e0);
        const float T = v1[g].x * v2[g].x + v1[g].y * v2[g].y;
        jx = __builtin_amdgcn_mfma_f32_16x16x4f32(T, px, jx, 0, 0, 0);
        if (yz) {
            const float s0 = clamp01(1.f - fabsf(e0)), s1 = clamp01(1.f - fabsf(e1));
            // 2 A and 2 D along x: the factor 1/2 is applied to the sums
            jyz = __builtin_amdgcn_mfma_f32_16x16x4f32(pr[g] * v1[g].x, s0 + s1, jyz, 0, 0, 0);
            jyz = __builtin_amdgcn_mfma_f32_16x16x4f32(pr[g] * v1[g].y, (2.f * RSQRT12) * (s1 - s0), jyz, 0, 0, 0);
        }
    }
}

// Where a pass's sums go.  Lane l holds column t of rows 4 q + j, j = 0..3, of Jx
// and of (Jy, Jz: rows 0..5 and 6..11).  The rows' transverse offsets oj + 3 ok
// are packed four bits each, by q; lane oj + 3 ok works out where that grid row
// starts (-1 outside the grid), and the others fetch it from there.
struct RowOut {
    int i, start, wx, wyz;  // i: the column's x index, or -1
};

__device__ __forceinline__ RowOut row_out(const PartArgs &a, int lane, int X0, int by, int bz)
{
    const int t = lane & 15, q = lane >> 4;
    int i = X0 + t, j = by + t % 3, k = bz + t / 3;
    if (a.per[0]) i = wrapn(i, a.nx);
    if (a.per[1]) j = wrapn(j, a.ny);
    if (a.per[2]) k = wrapn(k, a.nz);
    const bool ok = (unsigned)j < (unsigned)a.ny && (unsigned)k < (unsigned)a.nz;
    RowOut r;
    r.i = (unsigned)i < (unsigned)a.nx ? i : -1;
    r.start = ok ? a.nx * (j + a.ny * k) : -1;
    r.wx = q == 0 ? 0x1730 : (q == 1 ? 0x4685 : 0x2);
    r.wyz = q == 0 ? 0x1630 : (q == 1 ? 0x1074 : 0x5432);
    return r;
}

__device__ __forceinline__ void row_add(const PartArgs &a, const RowOut &r, int lane, int j, bool yz, float jx,
                                        float jyz)
{
    const int q = lane >> 4;
    const int ox = __builtin_amdgcn_ds_bpermute(((r.wx >> (4 * j)) & 15) << 2, r.start);
    if (min(r.i, ox) >= 0 && 4 * q + j < 9 && jx != 0.f) gatomic_add(G(a.Jb[0]) + (ox + r.i), a.qd * jx);
    if (!yz) return;
    const int oyz = __builtin_amdgcn_ds_bpermute(((r.wyz >> (4 * j)) & 15) << 2, r.start);
    float *J = 4 * q + j < 6 ? a.Jb[1] : a.Jb[2];
    if (min(r.i, oyz) >= 0 && q < 3 && jyz != 0.f) gatomic_add(G(J) + (oyz + r.i), (0.5f * a.qd) * jyz);
}

// m: the pass's lanes; yz: some lane of the wavefront moves along y or z.
__device__ __forceinline__ void deposit_rows(const PartArgs &a, RowLds &L, unsigned long long m, int lane, float x0,
                                             float x1, int X0, int by, int bz, bool yz)
{
    const bool mine = (m >> lane) & 1ull;
    // one wavefront per workgroup: its LDS operations execute in program
    // order, the wave barriers keep the compiler from moving them
    __builtin_amdgcn_wave_barrier();
    L.x[lane] = mine ? make_float2(x0, x1) : make_float2(ROW_FAR, ROW_FAR);
    __builtin_amdgcn_wave_barrier();
    fvec4 jx = {0.f, 0.f, 0.f, 0.f}, jyz = {0.f, 0.f, 0.f, 0.f};
    for (int d = 0; d < 4; ++d)
        if ((m >> (16 * d)) & 0xffffull) row_chunk<false>(L, 16 * d, 0, lane, X0, yz, jx, jyz);
    const RowOut r = row_out(a, lane, X0, by, bz);
#pragma unroll
    for (int j = 0; j < 4; ++j) row_add(a, r, lane, j, yz, jx[j], jyz[j]);
}

// relativistic Boris: half kick, rotation, half kick (u in units of c)
__device__ __forceinline__ void boris(float ah, float e0, float e1, float e2, float h0, float h1, float h2, float &u0,
                                      float &u1, float &u2)
{
    const float m0 = u0 + ah * e0, m1 = u1 + ah * e1, m2 = u2 + ah * e2;
    const float gi = rsqrtf(1.f + m0 * m0 + m1 * m1 + m2 * m2);
    const float t0 = ah * h0 * gi, t1 = ah * h1 * gi, t2 = ah * h2 * gi;
    const float f = 2.f / (1.f + t0 * t0 + t1 * t1 + t2 * t2);
    const float s0 = f * t0, s1 = f * t1, s2 = f * t2;
    const float p0 = m0 + (m1 * t2 - m2 * t1);
    const float p1 = m1 + (m2 * t0 - m0 * t2);
    const float p2 = m2 + (m0 * t1 - m1 * t0);
    u0 = m0 + (p1 * s2 - p2 * s1) + ah * e0;
    u1 = m1 + (p2 * s0 - p0 * s2) + ah * e1;
    u2 = m2 + (p0 * s1 - p1 * s0) + ah * e2;
}

// A move that leaves through a wall, or is not finite, deactivates the particle.
__device__ __forceinline__ bool leaves(const PartArgs &a, float x, float y, float z)
{
    return !(isfinite(x) && isfinite(y) && isfinite(z)) || (!a.per[0] && !(x >= 0.f && x < (float)a.nx)) ||
           (!a.per[1] && !(y >= 0.f && y < (float)a.ny)) || (!a.per[2] && !(z >= 0.f && z < (float)a.nz));
}

// ---- fixed-point deposit (matrix cores on bytes) ----
// The sums over the particles of every window of a wavefront are a matrix product:
// 16 windows by 64 particles (1 where the particle has the window) times 64 particles
// by 16 slots, 4 such products for the 54 slots.  A slot's units are split into
// 4 signed bytes, v_mfma_i32_16x16x64_i8 sums each byte exactly, and the sums are
// put together again (at most 2^30).  Lane l holds row or column l % 16 of the
// particles 16 (l / 16) on; the units get there from their particle's lane through
// LDS, 16 slots at a time.  Summing windows one after another, with 220 VALU
// instructions each, and their short ones with 54 atomics per lane, took 30.1 us for
// 2e5 particles in 96x64x96 cells, now 23.5 (2e4: 20.3 -> 13.8, 1e6: 59.1 -> 57.3);
// what is left is the 54 units of every particle and the gather.
//
// A wavefront whose windows do not fit one such product, with less than 8 lanes in any,
// has them added lane by lane, in bunches of up to FIX_LANE_MAX, where the time is the
// slowest wavefront's: 200 particles in 4000 cells 22.7 -> 10.2 us (15.0 in the sums
// over lanes), 2000 21.4 -> 12.1 (15.8), 2e4 in 5e5 cells 29.3 -> 21.0.  Of more, the
// products keep the chip busier: 1e5 in 5e5 cells 51 us, lane by lane 57.
constexpr int FIX_WINDOWS = 16;
constexpr int FIX_LANE_MAX = 1 << 16;
typedef int ivec4 __attribute__((ext_vector_type(4)));
struct FixLds {
    alignas(16) int units[16][68];  // by slot (rows that 16 lanes read at once start 4 banks apart), by particle
    int base[3][64];
};

// The bytes of 4 dwords, transposed: dword b of the result is byte b of each.
__device__ __forceinline__ ivec4 byte_planes(ivec4 v)
{
    const unsigned lo01 = __builtin_amdgcn_perm(v.y, v.x, 0x05010400), hi01 = __builtin_amdgcn_perm(v.y, v.x, 0x07030602);
    const unsigned lo23 = __builtin_amdgcn_perm(v.w, v.z, 0x05010400), hi23 = __builtin_amdgcn_perm(v.w, v.z, 0x07030602);
    return ivec4{(int)__builtin_amdgcn_perm(lo23, lo01, 0x05040100), (int)__builtin_amdgcn_perm(lo23, lo01, 0x07060302),
                 (int)__builtin_amdgcn_perm(hi23, hi01, 0x05040100), (int)__builtin_amdgcn_perm(hi23, hi01, 0x07060302)};
}

// Whether the lanes of rem have more than FIX_WINDOWS windows, none of 8 lanes or more
// among the first of them.
__device__ __forceinline__ bool scattered(unsigned long long rem, int key)
{
    int windows = 0;
    while (rem) {
        const int leader = __ffsll((long long)rem) - 1;
        const unsigned long long m = __ballot(key == __builtin_amdgcn_readlane(key, leader)) & rem;
        rem &= ~m;
        if (__popcll(m) >= 8) return false;
        if (++windows > FIX_WINDOWS) return true;
    }
    return false;
}

template <class Units>
__device__ __forceinline__ void deposit_fixed(const PartArgs &a, FixLds &L, unsigned long long rem, int lane,
                                              const int base[3], int key, Units units)
{
    const int n = lane & 15, q = lane >> 4;
#pragma unroll
    for (int d = 0; d < 3; ++d) L.base[d][lane] = base[d];
    ivec4 B[4][4];  // by 16 slots, by byte
#pragma unroll
    for (int T = 0; T < 4; ++T) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 16 * T; s < (T < 3 ? 16 * T + 16 : 54); ++s)
            L.units[s - 16 * T][lane] = (units(s) + 0x808080) ^ 0x808080;  // signed bytes
        __builtin_amdgcn_wave_barrier();
        ivec4 p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            p[e] = byte_planes(*reinterpret_cast<const ivec4 *>(&L.units[T < 3 ? n : min(n, 5)][16 * q + 4 * e]));
#pragma unroll
        for (int b = 0; b < 4; ++b) B[T][b] = ivec4{p[0][b], p[1][b], p[2][b], p[3][b]};
    }
    // the window's first cell where the window is inside the grid, else -1
    const bool in = base[0] >= 0 && base[0] + 2 < a.nx && base[1] >= 0 && base[1] + 2 < a.ny && base[2] >= 0 &&
                    base[2] + 2 < a.nz;
    const int first = in ? base[0] + a.nx * (base[1] + a.ny * base[2]) : -1;
    int rel[4];
    unsigned long long *J[4];
    // (held in registers: a choice of the argument block's members would go through scratch)
    unsigned long long *J0 = a.Jq[0], *J1 = a.Jq[1], *J2 = a.Jq[2];
    asm("" : "+s"(J0), "+s"(J1), "+s"(J2));
#pragma unroll
    for (int T = 0; T < 4; ++T) {
        int comp, oi, oj, ok;
        slot_geom(min(16 * T + n, 53), comp, oi, oj, ok);
        rel[T] = oi + a.nx * (oj + a.ny * ok);
        J[T] = comp == 0 ? J0 : (comp == 1 ? J1 : J2);
    }
    while (rem) {
        // up to 16 windows: w in row 4 (w % 4) + w / 4, so that few of them lie in
        // the first results of all lanes; lead: the lanes windows 4 j + q lead
        unsigned long long mine = 0;
        int lead[4] = {0, 0, 0, 0}, w = 0;
        for (; w < 16 && rem; ++w) {
            const int leader = __ffsll((long long)rem) - 1;
            const unsigned long long m = __ballot(key == __builtin_amdgcn_readlane(key, leader)) & rem;
            rem &= ~m;
            if (n == 4 * (w & 3) + (w >> 2)) mine = m;
#pragma unroll
            for (int j = 0; j < 4; ++j) lead[j] = w == 4 * j + q ? leader : lead[j];
        }
        const unsigned own = (unsigned)(mine >> (16 * q)) & 0xffffu;
        ivec4 A;
#pragma unroll
        for (int e = 0; e < 4; ++e) A[e] = (int)((((own >> (4 * e)) & 15u) * 0x204081u) & 0x01010101u);
        int at[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) at[j] = __builtin_amdgcn_ds_bpermute(4 * lead[j], first);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (4 * j + q >= w) at[j] = -2;
#pragma unroll
        for (int T = 0; T < 4; ++T) {
            const ivec4 zero = {0, 0, 0, 0};
            const ivec4 s0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, B[T][0], zero, 0, 0, 0);
            const ivec4 s1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, B[T][1], zero, 0, 0, 0);
            const ivec4 s2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, B[T][2], zero, 0, 0, 0);
            const ivec4 s3 = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, B[T][3], zero, 0, 0, 0);
            const int s = 16 * T + n;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (4 * j >= w) continue;
                const int tot = (int)((unsigned)s0[j] + ((unsigned)s1[j] << 8) + ((unsigned)s2[j] << 16) +
                                      ((unsigned)s3[j] << 24));
                if (s >= 54 || tot == 0) continue;
                if (at[j] >= 0) {
                    gatomic_add(G(J[T]) + (at[j] + rel[T]), (unsigned long long)(long long)tot);
                } else if (at[j] == -1) {  // the window wraps or leaves the grid
                    const int p = lead[j];
                    int comp;
                    const int cell = slot_index(a, s, L.base[0][p], L.base[1][p], L.base[2][p], comp);
                    if (cell >= 0) gatomic_add(G(J[T]) + cell, (unsigned long long)(long long)tot);
                }
            }
        }
    }
}

// A row of which a wavefront holds half its lanes or more lies in the dense part of the
// bunch, where most wavefronts add to the same few cache lines and per-lane atomics on
// one address follow each other at 17 ns: there the lanes between its own (of its
// cells, in sorted order: particles that moved back over a face) are passes from
// DENSE_LANES on.  Particles moving every way, without / with: 2e5 in 180 cells 358 /
// 153 us, 1e6 in 4000 cells 590 / 337, 2e5 with 15 % transverse velocities 134 / 72
// (from 3 lanes on 93, from 5 on 126).  The short rows before and after, a cold beam's
// next ones, stay lane by lane: as passes 1e5 in 128x64x64 cells took 15.3 us for 14.2,
// a batch of 16 118 for 116.
constexpr int DENSE_LANES = 2;

// The lanes from the first of m != 0 to the last.
__device__ __forceinline__ unsigned long long between(unsigned long long m)
{
    return (~0ull >> __clzll((long long)m)) & (~0ull << (__ffsll((long long)m) - 1));
}

// The passes of a wavefront's rows; the lanes left over.
__device__ __forceinline__ unsigned long long row_passes(const PartArgs &a, RowLds &L, unsigned long long rem,
                                                         int lane, const int base[3], float x0, float x1, bool yz)
{
    const int lanes = __popcll(rem);
    unsigned long long small = 0, widest = 0;
    for (int least = ROW_LANES;; least = DENSE_LANES) {
        while (rem) {
            const int leader = __ffsll((long long)rem) - 1;
            // a lane behind the leader by less than a cell still joins its pass
            const int X0 = __builtin_amdgcn_readlane(base[0], leader) - 1;
            const int by = __builtin_amdgcn_readlane(base[1], leader);
            const int bz = __builtin_amdgcn_readlane(base[2], leader);
            const unsigned long long m =
                __ballot(base[1] == by && base[2] == bz && (unsigned)(base[0] - X0) < (unsigned)ROW_BASES) & rem;
            rem &= ~m;
            if (__popcll(m) < least) {
                small |= m;
                continue;
            }
            if (__popcll(m) > __popcll(widest)) widest = m;
            deposit_rows(a, L, m, lane, x0, x1, X0, by, bz, yz);
        }
        if (least != ROW_LANES || !widest || 2 * __popcll(widest) < lanes) return small;
        rem = small & between(widest);
        small &= ~rem;
    }
}

template <int MODE, int PX, int FIX>
__device__ __forceinline__ void push_body(const PartArgs &a, int blk)
{
    const int p = blk * PUSH_BLOCK + threadIdx.x;
    const int lane = threadIdx.x & 63;
    // the current set's arrays straight from the device state (one scalar
    // load after the state's address, not the set index and then its arrays)
    const gp<const DevState> st = G(a.st);
    const gp<float> __restrict__ X = G(st->P[0]);
    const gp<float> __restrict__ Y = G(st->P[1]);
    const gp<float> __restrict__ Z = G(st->P[2]);
    const gp<float> __restrict__ UX = G(st->P[3]);
    const gp<float> __restrict__ UY = G(st->P[4]);
    const gp<float> __restrict__ UZ = G(st->P[5]);
    bool dep = false;
    int base[3] = {0, 0, 0};
    float x0 = 0.f, y0 = 0.f, z0 = 0.f, x1 = 0.f, y1 = 0.f, z1 = 0.f;  // the move, x1 before folding
    if (p < a.n) {
        // The gather and Boris run for every lane, with no branch on liveness
        // before them, so that all six particle loads go out together (a
        // branch lets the compiler sink loads below it, each sunk group one
        // more round trip to memory).  A lost particle gathers at the box
        // corner, a valid position, and nothing of it is written.  The
        // particle state streams with the non-temporal hint: it is touched
        // once per step, and the fields around it should stay cached.
        const float x = __builtin_nontemporal_load(X + p), y = __builtin_nontemporal_load(Y + p),
                    z = __builtin_nontemporal_load(Z + p);
        float u0 = __builtin_nontemporal_load(UX + p), u1 = __builtin_nontemporal_load(UY + p),
              u2 = __builtin_nontemporal_load(UZ + p);
        const bool live = live_pos(x, y, z, a.nx, a.ny, a.nz);
        const float xg = live ? x : 0.f, yg = live ? y : 0.f, zg = live ? z : 0.f;
        {
            Axis2 AY, AZ;
            axis_corners(yg, a.ny, a.per[1], a.nx, AY);
            axis_corners(zg, a.nz, a.per[2], a.nx * a.ny, AZ);
            // E^n and Ht^n = (Ht^{n-1/2} + Ht^{n+1/2})/2 at x^n
            float e0, e1, e2, h0, h1, h2;
            if (PX) {
                Axis2 AX;
                axis_corners(xg, a.nx, a.per[0], 1, AX);
                e0 = gather_scalar<1, 0, 0>(a.E[0], AX, AY, AZ);
                e1 = gather_scalar<0, 1, 0>(a.E[1], AX, AY, AZ);
                e2 = gather_scalar<0, 0, 1>(a.E[2], AX, AY, AZ);
                h0 = gather_scalar<0, 1, 1>(a.B[0], AX, AY, AZ);
                h1 = gather_scalar<1, 0, 1>(a.B[1], AX, AY, AZ);
                h2 = gather_scalar<1, 1, 0>(a.B[2], AX, AY, AZ);
            } else {
                XPair XP;
                x_pairs(xg, a.nx, XP);
                e0 = gather_pair<1, 0, 0>(a.E[0], XP, AY, AZ);
                e1 = gather_pair<0, 1, 0>(a.E[1], XP, AY, AZ);
                e2 = gather_pair<0, 0, 1>(a.E[2], XP, AY, AZ);
                h0 = gather_pair<0, 1, 1>(a.B[0], XP, AY, AZ);
                h1 = gather_pair<1, 0, 1>(a.B[1], XP, AY, AZ);
                h2 = gather_pair<1, 1, 0>(a.B[2], XP, AY, AZ);
            }
            boris(a.ah, e0, e1, e2, h0, h1, h2, u0, u1, u2);
        }
        if (live) {
            const float g = rsqrtf(1.f + u0 * u0 + u1 * u1 + u2 * u2);
            const float nx1 = x + a.S * u0 * g, ny1 = y + a.S * u1 * g, nz1 = z + a.S * u2 * g;
            const bool out = leaves(a, nx1, ny1, nz1);
            __builtin_nontemporal_store(u0, UX + p);
            __builtin_nontemporal_store(u1, UY + p);
            __builtin_nontemporal_store(u2, UZ + p);
            if (out) {
                __builtin_nontemporal_store(-1.f, X + p);  // left the box: deactivated, last move not deposited
            } else {
                x0 = x;
                y0 = y;
                z0 = z;
                x1 = nx1;
                y1 = ny1;
                z1 = nz1;
                base[0] = min((int)floorf(x0), (int)floorf(x1));
                base[1] = min((int)floorf(y0), (int)floorf(y1));
                base[2] = min((int)floorf(z0), (int)floorf(z1));
                dep = true;
                __builtin_nontemporal_store(a.per[0] ? fold(x1, a.nx) : x1, X + p);
                __builtin_nontemporal_store(a.per[1] ? fold(y1, a.ny) : y1, Y + p);
                __builtin_nontemporal_store(a.per[2] ? fold(z1, a.nz) : z1, Z + p);
            }
        }
    }
    const unsigned long long live = __ballot(dep);
    // per-wavefront push counter (one slot per wavefront of the launch)
    // (an atomic whose result is unused: the wavefront does not wait for the
    // counter's old value as a load-add-store would)
    if (lane == 0 && live) gatomic_add(G(a.pushes) + (p >> 6), (unsigned long long)__popcll(live));
    unsigned long long rem = live;
    if (!live) return;
    if (FIX) {
        // integer units per slot, each computed once: the sums do not depend on
        // which lanes are summed together
        __shared__ FixLds L;
        const AxisF fx = axis_factors(x0, x1, base[0]), fy = axis_factors(y0, y1, base[1]),
                    fz = axis_factors(z0, z1, base[2]);
        const auto units = [&](float c) { return __float2int_rn(a.qd * c * a.qscale); };
        const int key = (base[0] + 1) + (a.nx + 2) * ((base[1] + 1) + (a.ny + 2) * (base[2] + 1));
        if (a.n <= FIX_LANE_MAX && scattered(rem, key)) {
            if (dep)
                lane_deposit(a, base, fx, fy, fz, units, [&](int comp, int q, int u) { add_fixed(a, comp, q, u); });
        } else {
            deposit_fixed(a, L, rem, lane, base, key, [&](int s) { return units(slot_value(fx, fy, fz, s)); });
        }
        return;
    }
    if (MODE == 0) {
        __shared__ RowLds L;
        // a lane that does not deposit leaves zeros (a factor 0 times an
        // uninitialised value could be NaN)
        const AxisF fy = axis_factors(y0, y1, base[1]), fz = axis_factors(z0, z1, base[2]);
        row_factors(L, lane, fy, fz);
        const bool yz = __ballot(fy.P[0] != 0.f || fy.P[1] != 0.f || fz.P[0] != 0.f || fz.P[1] != 0.f) != 0ull;
        rem = row_passes(a, L, rem, lane, base, x0, x1, yz);
    }
    if ((rem >> lane) & 1ull) {
        const AxisF fx = axis_factors(x0, x1, base[0]), fy = axis_factors(y0, y1, base[1]),
                    fz = axis_factors(z0, z1, base[2]);
        lane_deposit(a, base, fx, fy, fz, [&](float c) { return a.qd * c; },
                     [&](int comp, int q, float v) {
                         // select, not a[comp]: a runtime index into the argument block would put it in scratch
                         float *J = comp == 0 ? a.Jb[0] : (comp == 1 ? a.Jb[1] : a.Jb[2]);
                         gatomic_add(G(J) + q, v);
                     });
    }
}

// Workgroups take the sorted particles from both ends inwards: the ends are the
// bunch's tails along z, whose wavefronts hold many short rows and take longest,
// and started last they would run on alone (1e6 particles in a 448x128x128 box
// 54.0 -> 48.3 us, in 64x128x128 62.2 -> 55.4 us).
__device__ __forceinline__ int ends_first(int b, int n) { return b & 1 ? n - 1 - (b >> 1) : b >> 1; }

// ---- few particles: 16 a wavefront, 4 lanes each ----
// With few particles the push takes as long as its slowest wavefront, and a
// wavefront that has a SIMD to itself takes as long as the instructions it
// issues one after another: of 26000 cycles, 2000 for the gather, 4500 for each
// row's pass, 5500 for the lanes of short rows.  So a wavefront gets 16
// particles: 4 lanes share a particle, each loads one (y, z) corner and adds
// one third of a short row's slots; a pass takes 16 particles.  The four
// wavefronts of a workgroup hold the 64 particles of a plain one's and go through
// the same passes.  One that 3 or 4 of them have particles in is summed in LDS,
// and each adds a quarter of the slots: atomics on one cache line follow each
// other at 12.7 ns, and without this a dense bunch (2e4 particles on 150 lines)
// took 23 us, otherwise 8.  Long loops over wide rows in dense bunches are what
// the plain kernel is for.
//
// Plain kernel / this one, us: 1000 particles 10.8 / 7.8, 4000 in a sheet 12.9 /
// 8.4, 2e4 in a 91x45x53 box 13.0 / 8.6, 3e4 in 448x128x128 10.6 / 8.7, 5e4 in
// 128x64x64 13.5 / 10.6, 6e4 in 448x128x128 11.9 / 10.2, 6e4 periodic along x
// 14.3 / 14.3, 1e5 14.3 / 14.1 and 12.0 / 13.8, 2e5 15.2 / 19.6.
constexpr int SPLIT_MAX = 1 << 16;
// Rows with fewer particles of the workgroup go to quarter_deposit, whose time does
// not depend on their number (2e4 particles, least number 4, 7, 10, 16: 13.4,
// 11.3, 9.8, 8.6 us; 1000: 9.5, 9.0, 8.4, 7.8).
constexpr int SPLIT_LANES = 16;
// But in the dense part of a bunch of more than SPLIT_DENSE, the particles between the
// widest row's form passes from SPLIT_DENSE_LANES on (as for DENSE_LANES above).  Particles moving every way, without / with: 6000 in one
// cell 28.6 / 17.5 us, 2e4 in 180 cells 45 / 27, 65536 130 / 68; fewer than 4096 in one
// cell lose as much to the passes' latency as they gain (2000: 14.3 / 14.8).
constexpr int SPLIT_DENSE = 4096;
constexpr int SPLIT_DENSE_LANES = 3;

// v of the lanes of corner 0..3 of this lane's particle (lanes l, l ^ 16, l ^ 32, l ^ 48).
struct Quad {
    float v[4];
};
__device__ __forceinline__ Quad quad_all(float v)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const auto e = __builtin_amdgcn_permlane32_swap(r[0], r[0], false, false);
    const auto o = __builtin_amdgcn_permlane32_swap(r[1], r[1], false, false);
    return {{__uint_as_float(e[0]), __uint_as_float(o[0]), __uint_as_float(e[1]), __uint_as_float(o[1])}};
}

// Offsets of the (y, z) corner that a lane loads, by node and half node.
struct Corner {
    int y[2], z[2];
};

__device__ __forceinline__ Corner corner(const Axis2 &Y, const Axis2 &Z, int c)
{
    Corner r;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        // sums, as a choice of two members would put them in scratch
        r.y[h] = Y.o0[h] + (c & 1) * (Y.o1[h] - Y.o0[h]);
        r.z[h] = Z.o0[h] + (c >> 1) * (Z.o1[h] - Z.o0[h]);
    }
    return r;
}

// gather_pair and gather_scalar with a corner's loads in each of 4 lanes.
template <int HX, int HY, int HZ>
__device__ __forceinline__ float quad_pair(float2 p, const XPair &X, const Axis2 &Y, const Axis2 &Z)
{
    const Quad t = quad_all(fmaf(X.wa[HX], p.x, X.wb[HX] * p.y));
    float v = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        v = fmaf((c & 1 ? Y.m1[HY] : Y.m0[HY]) * (c & 2 ? Z.m1[HZ] : Z.m0[HZ]), t.v[c], v);
    return v;
}

template <int HX, int HY, int HZ>
__device__ __forceinline__ float quad_scalar(float2 p, const Axis2 &X, const Axis2 &Y, const Axis2 &Z)
{
    const Quad a = quad_all(p.x), b = quad_all(p.y);
    float v = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float my = c & 1 ? Y.m1[HY] : Y.m0[HY], mz = c & 2 ? Z.m1[HZ] : Z.m0[HZ];
        v = fmaf(X.m0[HX] * my * mz, a.v[c], v);
        v = fmaf(X.m1[HX] * my * mz, b.v[c], v);
    }
    return v;
}

template <int HX, int HY, int HZ>
__device__ __forceinline__ float2 corner_pair(const float *__restrict__ f, const XPair &X, const Corner &C)
{
    return ld2(f + (X.o[HX] + C.y[HY] + C.z[HZ]));
}

template <int HX, int HY, int HZ>
__device__ __forceinline__ float2 corner_scalar(const float *__restrict__ f, const Axis2 &X, const Corner &C)
{
    const int o = C.y[HY] + C.z[HZ];
    return make_float2(G(f)[X.o0[HX] + o], G(f)[X.o1[HX] + o]);
}

// DENSE: more than SPLIT_DENSE particles.
template <int PX, int DENSE>
__global__ __launch_bounds__(256) void k_push_split(PartArgs a)
{
    const int lane = threadIdx.x & 63, c = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slot = 16 * wave + (lane & 15);
    const int blk = ends_first(blockIdx.x, gridDim.x), p = blk * PUSH_BLOCK + slot;
    const gp<const DevState> st = G(a.st);
    const gp<float> __restrict__ X = G(st->P[0]);
    const gp<float> __restrict__ Y = G(st->P[1]);
    const gp<float> __restrict__ Z = G(st->P[2]);
    const gp<float> __restrict__ UX = G(st->P[3]);
    const gp<float> __restrict__ UY = G(st->P[4]);
    const gp<float> __restrict__ UZ = G(st->P[5]);
    const int q = min(p, a.n - 1);
    const float x = X[q], y = Y[q], z = Z[q];
    float u0 = UX[q], u1 = UY[q], u2 = UZ[q];
    const bool had = p < a.n && live_pos(x, y, z, a.nx, a.ny, a.nz);
    const float xg = had ? x : 0.f, yg = had ? y : 0.f, zg = had ? z : 0.f;
    {
        Axis2 AY, AZ;
        axis_corners(yg, a.ny, a.per[1], a.nx, AY);
        axis_corners(zg, a.nz, a.per[2], a.nx * a.ny, AZ);
        const Corner C = corner(AY, AZ, c);
        float e0, e1, e2, h0, h1, h2;
        // every load before any exchange
        if (PX) {
            Axis2 AX;
            axis_corners(xg, a.nx, a.per[0], 1, AX);
            const float2 q0 = corner_scalar<1, 0, 0>(a.E[0], AX, C), q1 = corner_scalar<0, 1, 0>(a.E[1], AX, C);
            const float2 q2 = corner_scalar<0, 0, 1>(a.E[2], AX, C), q3 = corner_scalar<0, 1, 1>(a.B[0], AX, C);
            const float2 q4 = corner_scalar<1, 0, 1>(a.B[1], AX, C), q5 = corner_scalar<1, 1, 0>(a.B[2], AX, C);
            e0 = quad_scalar<1, 0, 0>(q0, AX, AY, AZ);
            e1 = quad_scalar<0, 1, 0>(q1, AX, AY, AZ);
            e2 = quad_scalar<0, 0, 1>(q2, AX, AY, AZ);
            h0 = quad_scalar<0, 1, 1>(q3, AX, AY, AZ);
            h1 = quad_scalar<1, 0, 1>(q4, AX, AY, AZ);
            h2 = quad_scalar<1, 1, 0>(q5, AX, AY, AZ);
        } else {
            XPair XP;
            x_pairs(xg, a.nx, XP);
            const float2 q0 = corner_pair<1, 0, 0>(a.E[0], XP, C), q1 = corner_pair<0, 1, 0>(a.E[1], XP, C);
            const float2 q2 = corner_pair<0, 0, 1>(a.E[2], XP, C), q3 = corner_pair<0, 1, 1>(a.B[0], XP, C);
            const float2 q4 = corner_pair<1, 0, 1>(a.B[1], XP, C), q5 = corner_pair<1, 1, 0>(a.B[2], XP, C);
            e0 = quad_pair<1, 0, 0>(q0, XP, AY, AZ);
            e1 = quad_pair<0, 1, 0>(q1, XP, AY, AZ);
            e2 = quad_pair<0, 0, 1>(q2, XP, AY, AZ);
            h0 = quad_pair<0, 1, 1>(q3, XP, AY, AZ);
            h1 = quad_pair<1, 0, 1>(q4, XP, AY, AZ);
            h2 = quad_pair<1, 1, 0>(q5, XP, AY, AZ);
        }
        boris(a.ah, e0, e1, e2, h0, h1, h2, u0, u1, u2);
    }
    const float g = rsqrtf(1.f + u0 * u0 + u1 * u1 + u2 * u2);
    const float nx1 = x + a.S * u0 * g, ny1 = y + a.S * u1 * g, nz1 = z + a.S * u2 * g;
    const bool dep = had && !leaves(a, nx1, ny1, nz1);
    if (had && c == 0) {
        UX[p] = u0;
        UY[p] = u1;
        UZ[p] = u2;
        X[p] = dep ? (a.per[0] ? fold(nx1, a.nx) : nx1) : -1.f;
        if (dep) {
            Y[p] = a.per[1] ? fold(ny1, a.ny) : ny1;
            Z[p] = a.per[2] ? fold(nz1, a.nz) : nz1;
        }
    }
    const float x0 = dep ? x : 0.f, y0 = dep ? y : 0.f, z0 = dep ? z : 0.f;
    const float x1 = dep ? nx1 : 0.f, y1 = dep ? ny1 : 0.f, z1 = dep ? nz1 : 0.f;
    const int base[3] = {min((int)floorf(x0), (int)floorf(x1)), min((int)floorf(y0), (int)floorf(y1)),
                         min((int)floorf(z0), (int)floorf(z1))};
    __shared__ RowLds L;
    __shared__ int4 B[PUSH_BLOCK];
    __shared__ float R[2][4][8][64];
    {
        const AxisF fy = axis_factors(y0, y1, base[1]), fz = axis_factors(z0, z1, base[2]);
        const bool yz = fy.P[0] != 0.f || fy.P[1] != 0.f || fz.P[0] != 0.f || fz.P[1] != 0.f;
        if (c == 0) {
            row_factors(L, slot, fy, fz);
            L.x[slot] = make_float2(x0, x1);
            B[slot] = make_int4(base[0], base[1], base[2], dep ? (yz ? 3 : 1) : 0);
        }
    }
    __syncthreads();
    const int4 b = B[lane];
    unsigned long long rem = __ballot(b.w & 1), small = 0;
    const bool yz = __ballot(b.w & 2) != 0ull;
    if (threadIdx.x == 0 && rem) gatomic_add(G(a.pushes) + blk, (unsigned long long)__popcll(rem));
    const int lanes = __popcll(rem);
    unsigned long long widest = 0;
    int buf = 0;
    for (int least = SPLIT_LANES;; least = SPLIT_DENSE_LANES) {
        while (rem) {
            const int leader = __ffsll((long long)rem) - 1;
            const int X0 = __builtin_amdgcn_readlane(b.x, leader) - 1;
            const int by = __builtin_amdgcn_readlane(b.y, leader);
            const int bz = __builtin_amdgcn_readlane(b.z, leader);
            const unsigned long long m =
                __ballot(b.y == by && b.z == bz && (unsigned)(b.x - X0) < (unsigned)ROW_BASES) & rem;
            rem &= ~m;
            if (__popcll(m) < least) {
                small |= m;
                continue;
            }
            if (DENSE && __popcll(m) > __popcll(widest)) widest = m;
            const unsigned own = (unsigned)(m >> (16 * wave)) & 0xffffu;
            fvec4 jx = {0.f, 0.f, 0.f, 0.f}, jyz = {0.f, 0.f, 0.f, 0.f};
            if (own) row_chunk<true>(L, 16 * wave, own, lane, X0, yz, jx, jyz);
            int waves = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) waves += ((m >> (16 * w)) & 0xffffull) != 0;
            if (waves < 3) {
                if (own) {
                    const RowOut r = row_out(a, lane, X0, by, bz);
#pragma unroll
                    for (int j = 0; j < 4; ++j) row_add(a, r, lane, j, yz, jx[j], jyz[j]);
                }
                continue;
            }
            if (own) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    R[buf][wave][j][lane] = jx[j];
                    R[buf][wave][4 + j][lane] = jyz[j];
                }
            }
            __syncthreads();
            float sx = 0.f, syz = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                if ((m >> (16 * w)) & 0xffffull) {
                    sx += R[buf][w][wave][lane];
                    syz += R[buf][w][4 + wave][lane];
                }
            row_add(a, row_out(a, lane, X0, by, bz), lane, wave, yz, sx, syz);
            buf ^= 1;
        }
        if (!DENSE || least != SPLIT_LANES || !widest || 2 * __popcll(widest) < lanes) break;
        rem = small & (~0ull >> __clzll((long long)widest)) & (~0ull << (__ffsll((long long)widest) - 1));
        small &= ~rem;
    }
    if ((small >> slot) & 1ull) quarter_deposit(a, c, base, x0, y0, z0, x1, y1, z1);
}

template <int MODE, int PX, int FIX>
__global__ __launch_bounds__(PUSH_BLOCK) void k_push_deposit(PartArgs a)
{
    push_body<MODE, PX, FIX>(a, ends_first(blockIdx.x, gridDim.x));
}

// Many simulations in one launch: workgroup b is push block own[b] & 0xffffff
// of simulation own[b] >> 24 (a table the host builds).
template <int MODE, int PX>
__global__ __launch_bounds__(PUSH_BLOCK) void k_push_deposit_batch(const PartArgs *__restrict__ args,
                                                                   const int *__restrict__ own)
{
    const int o = own[blockIdx.x];
    push_body<MODE, PX, 0>(args[o >> 24], o & 0xffffff);
}

void launch_push_deposit(const PartArgs &a, int mode, hipStream_t s)
{
    if (a.n <= 0) return;
    const int nb = (int)(((long long)a.n + PUSH_BLOCK - 1) / PUSH_BLOCK);
    // mode 2: wavefront-reduced deposit into the fixed-point current
    const bool fix = mode == 2 && a.Jq[0];
    if (mode == 0 && a.n <= SPLIT_MAX) {
        const bool dense = a.n > SPLIT_DENSE;
        if (a.per[0] && dense) hipLaunchKernelGGL((k_push_split<1, 1>), dim3(nb), dim3(256), 0, s, a);
        else if (a.per[0]) hipLaunchKernelGGL((k_push_split<1, 0>), dim3(nb), dim3(256), 0, s, a);
        else if (dense) hipLaunchKernelGGL((k_push_split<0, 1>), dim3(nb), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_push_split<0, 0>), dim3(nb), dim3(256), 0, s, a);
        return;
    }
    if (a.per[0]) {
        if (fix) hipLaunchKernelGGL((k_push_deposit<0, 1, 1>), dim3(nb), dim3(PUSH_BLOCK), 0, s, a);
        else if (mode == 1) hipLaunchKernelGGL((k_push_deposit<1, 1, 0>), dim3(nb), dim3(PUSH_BLOCK), 0, s, a);
        else hipLaunchKernelGGL((k_push_deposit<0, 1, 0>), dim3(nb), dim3(PUSH_BLOCK), 0, s, a);
    } else {
        if (fix) hipLaunchKernelGGL((k_push_deposit<0, 0, 1>), dim3(nb), dim3(PUSH_BLOCK), 0, s, a);
        else if (mode == 1) hipLaunchKernelGGL((k_push_deposit<1, 0, 0>), dim3(nb), dim3(PUSH_BLOCK), 0, s, a);
        else hipLaunchKernelGGL((k_push_deposit<0, 0, 0>), dim3(nb), dim3(PUSH_BLOCK), 0, s, a);
    }
}

// `mode` bit 0: per-lane atomics; bit 1: some simulation has a periodic x axis.
void launch_push_deposit_batch(const PartArgs *args, const int *own, int total, int mode, hipStream_t s)
{
    if (total <= 0) return;
    switch (mode & 3) {
    case 0: hipLaunchKernelGGL((k_push_deposit_batch<0, 0>), dim3(total), dim3(PUSH_BLOCK), 0, s, args, own); break;
    case 1: hipLaunchKernelGGL((k_push_deposit_batch<1, 0>), dim3(total), dim3(PUSH_BLOCK), 0, s, args, own); break;
    case 2: hipLaunchKernelGGL((k_push_deposit_batch<0, 1>), dim3(total), dim3(PUSH_BLOCK), 0, s, args, own); break;
    default: hipLaunchKernelGGL((k_push_deposit_batch<1, 1>), dim3(total), dim3(PUSH_BLOCK), 0, s, args, own); break;
    }
}

// ---------------------------------------------------------------------------
// Counting sort by cell: count (with in-cell rank), exclusive scan, scatter.
// ---------------------------------------------------------------------------

__global__ void k_fill_i32(int *p, int v, long long n)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long st = (long long)gridDim.x * blockDim.x;
    for (long long q = t; q < n; q += st) p[q] = v;
}

void launch_fill_i32(int *p, int v, long long n, hipStream_t s)
{
    if (n <= 0) return;
    long long nb = (n + 255) / 256;
    if (nb > 65536) nb = 65536;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)nb), dim3(256), 0, s, p, v, n);
}

template <bool MAX>
__device__ __forceinline__ int wave_minmax(int v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int o = __shfl_xor(v, off, 64);
        v = MAX ? max(v, o) : min(v, o);
    }
    return v;
}

// Cell key of a particle position (the lost-particle bucket ncell when it is
// not live).
// live_pos evaluated without short-circuit: every coordinate is read before
// the test, so the compiler cannot sink the loads of y and z below a branch
// on x (each sunk group would be one more round trip to memory).
__device__ __forceinline__ bool live_all(float x, float y, float z, int nx, int ny, int nz)
{
    return (x >= 0.f) & (x < (float)nx) & (y >= 0.f) & (y < (float)ny) & (z >= 0.f) & (z < (float)nz);
}

__device__ __forceinline__ int cell_key(float x, float y, float z, int nx, int ny, int nz)
{
    if (!live_all(x, y, z, nx, ny, nz)) return nx * ny * nz;
    return min((int)x, nx - 1) + nx * (min((int)y, ny - 1) + ny * min((int)z, nz - 1));
}

// Count particles per cell.  Lanes of a wavefront with the same cell (most
// of them: the particles are nearly sorted from the last sort) reserve their
// ranks with one atomic and take consecutive ones in lane order, so the
// scatter writes them to consecutive places.  The groups are found first and
// their leaders then issue all their atomics at once, so a wavefront spread
// over many cells waits for one atomic return, not one per cell.
// Each run of equal keys in the array's order also counts itself in
// runs[key] and records its start in first[key]: the scatter keeps the order
// of a key that forms a single run.  (The bunch is loaded ordered by x inside
// each cell, and under a near-uniform drift that order survives the sorts.  The
// deposit does not need it: its sums take the lanes of a row in any order.)
__device__ __forceinline__ void count_body(const SortArgs &a, int blk)
{
    __shared__ int bb[6];
    if (threadIdx.x < 6) bb[threadIdx.x] = threadIdx.x < 3 ? INT_MAX : INT_MIN;
    __syncthreads();
    const int p = blk * PBLOCK + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int pc = a.st->pcur;
    int key = a.ncell;
    int cell[3] = {INT_MAX, INT_MAX, INT_MAX};
    bool in = false;
    // lane 0 also needs the cell of particle p - 1 (the run test below):
    // its position is loaded here, with the lane's own
    float xq = -1.f, yq = -1.f, zq = -1.f;
    if (lane == 0 && p > 0 && p <= a.n) {
        xq = a.P[pc][0][p - 1];
        yq = a.P[pc][1][p - 1];
        zq = a.P[pc][2][p - 1];
    }
    if (p < a.n) {
        const float x = a.P[pc][0][p], y = a.P[pc][1][p], z = a.P[pc][2][p];
        if (live_all(x, y, z, a.nx, a.ny, a.nz)) {
            cell[0] = min((int)x, a.nx - 1);
            cell[1] = min((int)y, a.ny - 1);
            cell[2] = min((int)z, a.nz - 1);
            key = cell[0] + a.nx * (cell[1] + a.ny * cell[2]);
            in = true;
        }
    }
    unsigned long long rem = __ballot(p < a.n);
    unsigned long long group = 0;  // lanes sharing this lane's cell
    int leader = lane;
    while (rem) {
        const int l0 = __ffsll((long long)rem) - 1;
        const int k0 = __builtin_amdgcn_readlane(key, l0);
        const unsigned long long m = __ballot(((rem >> lane) & 1ull) && key == k0);
        if ((m >> lane) & 1ull) {
            group = m;
            leader = l0;
        }
        rem &= ~m;
    }
    int b = 0;
    if (p < a.n && lane == leader) b = atomicAdd(&a.counts[key], __popcll(group));
    b = __shfl(b, leader, 64);
    const int rank = b + __popcll(group & ((1ull << lane) - 1ull));
    if (p < a.n) {
        a.key[p] = key;
        a.rank[p] = rank;
    }
    // key of particle p - 1: the lane below, or for lane 0 from its position
    int kprev = __builtin_amdgcn_update_dpp(-1, key, 0x138, 0xf, 0xf, false);  // wave_shr:1
    if (lane == 0 && p > 0 && p <= a.n) kprev = cell_key(xq, yq, zq, a.nx, a.ny, a.nz);
    if (p < a.n && (p == 0 || kprev != key)) {
        atomicAdd(&a.runs[key], 1);
        a.first[key] = p;
    }
    // box of the live cells: wavefront min / max, then the workgroup's in LDS
    const bool any = __ballot(in) != 0ull;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int lo = wave_minmax<false>(in ? cell[q] : INT_MAX);
        const int hi = wave_minmax<true>(in ? cell[q] : INT_MIN);
        if (lane == 0 && any) {
            atomicMin(&bb[q], lo);
            atomicMax(&bb[3 + q], hi);
        }
    }
    __syncthreads();
    // one partial box per workgroup (global atomics from every workgroup on
    // the same six words would serialise); k_box_reduce combines them
    if (threadIdx.x < 6) a.boxpart[blk * 6 + threadIdx.x] = bb[threadIdx.x];
}

__global__ __launch_bounds__(PBLOCK) void k_sort_count(SortArgs a) { count_body(a, blockIdx.x); }

// The live-cell box from the count workgroups' partial boxes (one workgroup).
constexpr int BOX_THREADS = 1024;
__device__ __forceinline__ void box_reduce_body(const SortArgs &a, int nparts)
{
    __shared__ int red[6][BOX_THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int v[6] = {INT_MAX, INT_MAX, INT_MAX, INT_MIN, INT_MIN, INT_MIN};
    for (int w = threadIdx.x; w < nparts; w += BOX_THREADS) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            v[q] = min(v[q], a.boxpart[w * 6 + q]);
            v[3 + q] = max(v[3 + q], a.boxpart[w * 6 + 3 + q]);
        }
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        v[q] = q < 3 ? wave_minmax<false>(v[q]) : wave_minmax<true>(v[q]);
        if (lane == 0) red[q][wave] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int q = threadIdx.x;
        int r = red[q][0];
        for (int w = 1; w < BOX_THREADS / 64; ++w) r = q < 3 ? min(r, red[q][w]) : max(r, red[q][w]);
        a.box[q] = r;
    }
}

__global__ __launch_bounds__(BOX_THREADS) void k_box_reduce(SortArgs a, int nparts) { box_reduce_body(a, nparts); }

// Three-phase exclusive scan over SCAN_ITEMS * SCAN_THREADS elements per block.
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

__device__ __forceinline__ int block_exclusive_scan(int v, int *sm, int &total)
{
    // Hillis-Steele in LDS over 256 thread totals
    const int t = threadIdx.x;
    sm[t] = v;
    __syncthreads();
    for (int off = 1; off < SCAN_THREADS; off <<= 1) {
        const int add = t >= off ? sm[t - off] : 0;
        __syncthreads();
        sm[t] += add;
        __syncthreads();
    }
    total = sm[SCAN_THREADS - 1];
    const int incl = sm[t];
    __syncthreads();
    return incl - v;
}

// The keys a sort gives out: the cells of its live-cell box (the count
// kernel's), in global key order, then the lost-particle bucket (key ncell).
// Element e of that list.  The scans run over it alone: a key outside the box
// has no particle, so its offset is never read, and the offsets inside are
// those of a scan over every cell.
struct KeyDomain {
    int lo[3], w[3];
    long long cells;  // box cells; the list has cells + 1 entries
};

__device__ __forceinline__ KeyDomain key_domain(const SortArgs &a)
{
    KeyDomain D;
    D.cells = 1;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int lo = a.box[d], hi = a.box[3 + d];
        D.lo[d] = lo;
        D.w[d] = hi >= lo ? hi - lo + 1 : 0;
        D.cells *= D.w[d];
    }
    return D;
}

// Element e of the list in 32-bit unsigned arithmetic: e < cells <= ncell
// and every key below ncell fit, since ncell < 2^31 (a box exists, so its
// widths are at least 1).
__device__ __forceinline__ long long domain_key(const SortArgs &a, const KeyDomain &D, long long e)
{
    if (e >= D.cells) return a.ncell;
    const unsigned ue = (unsigned)e, w0 = (unsigned)D.w[0], w1 = (unsigned)D.w[1];
    const unsigned r = ue / w0;
    const unsigned x = ue - r * w0;
    const unsigned z = r / w1;
    const unsigned y = r - z * w1;
    return (long long)(((unsigned)D.lo[0] + x) +
                       (unsigned)a.nx * (((unsigned)D.lo[1] + y) + (unsigned)a.ny * ((unsigned)D.lo[2] + z)));
}

// Workgroups of the scan launches: a fixed grid walking the list's tiles (the
// list's length is known on the device only).
constexpr int SCAN_BLOCKS = 1024;

// Workgroup blk of nblk walking the tiles.
__device__ __forceinline__ void scan_tiles_body(const SortArgs &a, int *tile_sums, int blk, int nblk)
{
    __shared__ int sm[SCAN_THREADS];
    const KeyDomain D = key_domain(a);
    const long long n = D.cells + 1;
    for (long long b0 = (long long)blk * SCAN_TILE; b0 < n; b0 += (long long)nblk * SCAN_TILE) {
        int s = 0;
        for (int q = 0; q < SCAN_ITEMS; ++q) {
            const long long e = b0 + (long long)q * SCAN_THREADS + threadIdx.x;
            if (e < n) s += a.counts[domain_key(a, D, e)];
        }
        int total;
        block_exclusive_scan(s, sm, total);
        if (threadIdx.x == 0) tile_sums[b0 / SCAN_TILE] = total;
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_tiles(SortArgs a, int *tile_sums)
{
    scan_tiles_body(a, tile_sums, blockIdx.x, gridDim.x);
}

// One workgroup; each thread scans SCAN_ITEMS consecutive tile sums of a
// chunk serially around one block scan of the thread totals.
__device__ __forceinline__ void scan_sums_body(const SortArgs &a, int *tile_sums)
{
    __shared__ int sm[SCAN_THREADS];
    const int ntiles = (int)((key_domain(a).cells + 1 + SCAN_TILE - 1) / SCAN_TILE);
    int carry = 0;
    for (int b0 = 0; b0 < ntiles; b0 += SCAN_TILE) {
        const int first = b0 + threadIdx.x * SCAN_ITEMS;
        int v[SCAN_ITEMS];
        int s = 0;
#pragma unroll
        for (int q = 0; q < SCAN_ITEMS; ++q) {
            v[q] = first + q < ntiles ? tile_sums[first + q] : 0;
            s += v[q];
        }
        int total;
        int run = carry + block_exclusive_scan(s, sm, total);
#pragma unroll
        for (int q = 0; q < SCAN_ITEMS; ++q) {
            if (first + q < ntiles) tile_sums[first + q] = run;
            run += v[q];
        }
        carry += total;
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_sums(SortArgs a, int *tile_sums) { scan_sums_body(a, tile_sums); }

__device__ __forceinline__ void scan_apply_body(const SortArgs &a, const int *tile_sums, int blk, int nblk)
{
    __shared__ int sm[SCAN_THREADS];
    const KeyDomain D = key_domain(a);
    const long long n = D.cells + 1;
    for (long long t0 = (long long)blk * SCAN_TILE; t0 < n; t0 += (long long)nblk * SCAN_TILE) {
        // each thread owns SCAN_ITEMS consecutive entries of the tile
        const long long b0 = t0 + (long long)threadIdx.x * SCAN_ITEMS;
        long long g[SCAN_ITEMS];
        int vals[SCAN_ITEMS];
#pragma unroll
        for (int q = 0; q < SCAN_ITEMS; ++q) {
            g[q] = b0 + q < n ? domain_key(a, D, b0 + q) : -1;
            vals[q] = g[q] >= 0 ? a.counts[g[q]] : 0;
        }
        int s = 0;
#pragma unroll
        for (int q = 0; q < SCAN_ITEMS; ++q) s += vals[q];
        int total;
        int run = block_exclusive_scan(s, sm, total) + tile_sums[t0 / SCAN_TILE];
#pragma unroll
        for (int q = 0; q < SCAN_ITEMS; ++q) {
            if (g[q] >= 0) a.counts[g[q]] = run;
            run += vals[q];
        }
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_apply(SortArgs a, const int *tile_sums)
{
    scan_apply_body(a, tile_sums, blockIdx.x, gridDim.x);
}

// After the scatter: the counts and run counts of the list's keys back to 0,
// so that both arrays are 0 at every key between sorts (they start so).
__device__ __forceinline__ void sort_clear_body(const SortArgs &a, int blk, int nblk)
{
    const KeyDomain D = key_domain(a);
    const long long n = D.cells + 1;
    for (long long e = (long long)blk * blockDim.x + threadIdx.x; e < n; e += (long long)nblk * blockDim.x) {
        const long long g = domain_key(a, D, e);
        a.counts[g] = 0;
        a.runs[g] = 0;
    }
}

__global__ __launch_bounds__(SCAN_THREADS) void k_sort_clear(SortArgs a) { sort_clear_body(a, blockIdx.x, gridDim.x); }

__device__ __forceinline__ void scatter_body(const SortArgs &a, int blk)
{
    const int p = blk * PBLOCK + threadIdx.x;
    if (p >= a.n) return;
    const int pc = a.st->pcur;
    // every load first, in two rounds (the particle, its key and rank; then
    // the key's count and run), then the stores: the stores to the other
    // buffer set may alias the loads as far as the compiler knows, so a load
    // after a store would wait for it
    float v[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) v[c] = a.P[pc][c][p];
    const int id = a.id[pc][p];
    const int k = a.key[p];
    const int rk = a.rank[p];
    const int cnt = a.counts[k], runs = a.runs[k], f = a.first[k];
    const int dst = cnt + (runs == 1 ? p - f : rk);
#pragma unroll
    for (int c = 0; c < 6; ++c) a.P[pc ^ 1][c][dst] = v[c];
    a.id[pc ^ 1][dst] = id;
}

__global__ __launch_bounds__(PBLOCK) void k_sort_scatter(SortArgs a) { scatter_body(a, blockIdx.x); }

// After the scatter: the sorted set becomes current and the sort clock restarts.
__device__ __forceinline__ void done_body(const SortArgs &a)
{
    const int pc = a.st->pcur ^ 1;
    a.st->pcur = pc;
    a.st->since_sort = 0;
    for (int c = 0; c < 6; ++c) a.st->P[c] = a.P[pc][c];
}

__global__ void k_sort_done(SortArgs a)
{
    if (threadIdx.x == 0) done_body(a);
}

// ---- the sorts of many simulations in one launch per kernel ----
// Particle workgroups come from a table (member << 24 | the workgroup's index
// in that member, built by the host); each member's scans and clear get
// SORT_BATCH_BLOCKS workgroups of their own, walking its key list; the
// per-member single-workgroup kernels take one workgroup per member.
constexpr int SORT_BATCH_BLOCKS = 64;

__global__ __launch_bounds__(PBLOCK) void k_sort_count_batch(const SortArgs *__restrict__ args,
                                                             const int *__restrict__ own)
{
    const int o = own[blockIdx.x];
    count_body(args[o >> 24], o & 0xffffff);
}

__global__ __launch_bounds__(BOX_THREADS) void k_box_reduce_batch(const SortArgs *__restrict__ args)
{
    const SortArgs &a = args[blockIdx.x];
    box_reduce_body(a, (int)(((long long)a.n + PBLOCK - 1) / PBLOCK));
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_tiles_batch(const SortArgs *__restrict__ args)
{
    const SortArgs &a = args[blockIdx.x / SORT_BATCH_BLOCKS];
    scan_tiles_body(a, a.scan_tmp, blockIdx.x % SORT_BATCH_BLOCKS, SORT_BATCH_BLOCKS);
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_sums_batch(const SortArgs *__restrict__ args)
{
    const SortArgs &a = args[blockIdx.x];
    scan_sums_body(a, a.scan_tmp);
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_apply_batch(const SortArgs *__restrict__ args)
{
    const SortArgs &a = args[blockIdx.x / SORT_BATCH_BLOCKS];
    scan_apply_body(a, a.scan_tmp, blockIdx.x % SORT_BATCH_BLOCKS, SORT_BATCH_BLOCKS);
}

__global__ __launch_bounds__(PBLOCK) void k_sort_scatter_batch(const SortArgs *__restrict__ args,
                                                               const int *__restrict__ own)
{
    const int o = own[blockIdx.x];
    scatter_body(args[o >> 24], o & 0xffffff);
}

__global__ __launch_bounds__(SCAN_THREADS) void k_sort_clear_batch(const SortArgs *__restrict__ args)
{
    sort_clear_body(args[blockIdx.x / SORT_BATCH_BLOCKS], blockIdx.x % SORT_BATCH_BLOCKS, SORT_BATCH_BLOCKS);
}

__global__ void k_sort_done_batch(const SortArgs *__restrict__ args, int nmem)
{
    if (threadIdx.x < nmem) done_body(args[threadIdx.x]);
}

int scan_tmp_size(long long n) { return (int)((n + SCAN_TILE - 1) / SCAN_TILE) + 1; }

void launch_sort(const SortArgs &a, int *scan_tmp, hipStream_t s)
{
    // counts and runs are 0 at every key here (cleared at allocation and by
    // the previous sort over the keys it used)
    const int nb = (int)(((long long)a.n + PBLOCK - 1) / PBLOCK);
    if (a.n > 0) {
        hipLaunchKernelGGL(k_sort_count, dim3(nb), dim3(PBLOCK), 0, s, a);
        hipLaunchKernelGGL(k_box_reduce, dim3(1), dim3(BOX_THREADS), 0, s, a, nb);
    } else {
        launch_fill_i32(a.box, INT_MAX, 3, s);
        launch_fill_i32(a.box + 3, INT_MIN, 3, s);
    }
    // the list of keys has at most ncell + 1 entries
    const long long tiles = ((long long)a.ncell + 1 + SCAN_TILE - 1) / SCAN_TILE;
    const int grid = (int)std::min<long long>(tiles, SCAN_BLOCKS);
    hipLaunchKernelGGL(k_scan_tiles, dim3(grid), dim3(SCAN_THREADS), 0, s, a, scan_tmp);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(SCAN_THREADS), 0, s, a, scan_tmp);
    hipLaunchKernelGGL(k_scan_apply, dim3(grid), dim3(SCAN_THREADS), 0, s, a, scan_tmp);
    if (a.n > 0) hipLaunchKernelGGL(k_sort_scatter, dim3(nb), dim3(PBLOCK), 0, s, a);
    hipLaunchKernelGGL(k_sort_clear, dim3(grid), dim3(SCAN_THREADS), 0, s, a);
    hipLaunchKernelGGL(k_sort_done, dim3(1), dim3(64), 0, s, a);
}

void launch_sort_batch(const SortArgs *args, const int *own, int nown, int nmem, hipStream_t s)
{
    // every member has particles, and its counts and runs are 0 at every key
    if (nmem <= 0 || nown <= 0) return;
    const int g = nmem * SORT_BATCH_BLOCKS;
    hipLaunchKernelGGL(k_sort_count_batch, dim3(nown), dim3(PBLOCK), 0, s, args, own);
    hipLaunchKernelGGL(k_box_reduce_batch, dim3(nmem), dim3(BOX_THREADS), 0, s, args);
    hipLaunchKernelGGL(k_scan_tiles_batch, dim3(g), dim3(SCAN_THREADS), 0, s, args);
    hipLaunchKernelGGL(k_scan_sums_batch, dim3(nmem), dim3(SCAN_THREADS), 0, s, args);
    hipLaunchKernelGGL(k_scan_apply_batch, dim3(g), dim3(SCAN_THREADS), 0, s, args);
    hipLaunchKernelGGL(k_sort_scatter_batch, dim3(nown), dim3(PBLOCK), 0, s, args, own);
    hipLaunchKernelGGL(k_sort_clear_batch, dim3(g), dim3(SCAN_THREADS), 0, s, args);
    hipLaunchKernelGGL(k_sort_done_batch, dim3(1), dim3(64), 0, s, args, nmem);
}

}  // namespace pic
