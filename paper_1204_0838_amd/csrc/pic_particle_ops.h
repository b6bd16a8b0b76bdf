// Per-particle steps of the PIC cycle shared by the split kernels and the
// fused tiled kernel (identical arithmetic in both).
#pragma once

#include "pic_device.h"

namespace pic {

__device__ __forceinline__ void decompose(const Geom& g, int cell, int c[3]) {
    const int cz = cell / g.nxy;
    const int r = cell - cz * g.nxy;
    const int cy = r / g.n[0];
    c[0] = r - cy * g.n[0];
    c[1] = cy;
    c[2] = cz;
}

// Moving window: particles outside window cells [kill_lo, n - 1 - kill_hi] are
// removed (their cubic shapes would reach across the window's ends).
__device__ __forceinline__ bool window_killed(const Geom& g, int cx) {
    if (!g.window) return false;
    int xw = cx - g.origin;
    if (xw < 0) xw += g.n[0];
    return xw < g.kill_lo || xw > g.n[0] - 1 - g.kill_hi;
}

// Removed at the start of a step: in a window kill zone, or in a transverse
// cell of the absorbing layer.
__device__ __forceinline__ bool particle_killed(const Geom& g, const int c[3]) {
    if (window_killed(g, c[0])) return true;
    if (g.pml == 0) return false;
    return c[1] < g.pml || c[1] >= g.n[1] - g.pml || c[2] < g.pml || c[2] >= g.n[2] - g.pml;
}

// Shift between two cell indices along a periodic axis, mapped to (-n/2, n/2].
__device__ __forceinline__ int unwrap_shift(int di, int n) {
    if (di > n / 2) di -= n;
    if (di < -(n / 2)) di += n;
    return di;
}

// Cubic gather of the six staggered components given the per-axis node index
// offsets (already multiplied by the axis stride) of the integer (ii) and
// half-integer (ih) grids.  E_x: x half, y, z integer; E_y: y half; E_z: z half;
// B_x: y, z half; B_y: x, z half; B_z: x, y half.
__device__ __forceinline__ void gather_fields(float* const E[3], float* const B[3], const int ii[3][4],
                                              const int ih[3][4], const GatherStencil& s, float Ep[3],
                                              float Bp[3]) {
    Ep[0] = interp3(E[0], ih[0], ii[1], ii[2], s.wh[0], s.wi[1], s.wi[2]);
    Ep[1] = interp3(E[1], ii[0], ih[1], ii[2], s.wi[0], s.wh[1], s.wi[2]);
    Ep[2] = interp3(E[2], ii[0], ii[1], ih[2], s.wi[0], s.wi[1], s.wh[2]);
    Bp[0] = interp3(B[0], ii[0], ih[1], ih[2], s.wi[0], s.wh[1], s.wh[2]);
    Bp[1] = interp3(B[1], ih[0], ii[1], ih[2], s.wh[0], s.wi[1], s.wh[2]);
    Bp[2] = interp3(B[2], ih[0], ih[1], ii[2], s.wh[0], s.wh[1], s.wi[2]);
}

// Boris push, then move by dt u / gamma with carry into the cell index
// (periodic wrap in storage coordinates).  Returns device error flags.
__device__ __forceinline__ int push_move(const Geom& g, float qmh, const float E[3], const float B[3], float u[3],
                                         float off[3], int c[3]) {
    boris(u, E, B, qmh);
    const float ig = 1.0f / sqrtf(fmaf(u[0], u[0], fmaf(u[1], u[1], fmaf(u[2], u[2], 1.0f))));
    int flags = 0;
    if (!(isfinite(u[0]) && isfinite(u[1]) && isfinite(u[2]))) {
        flags |= ERR_NONFINITE;
        u[0] = u[1] = u[2] = 0.0f;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        float dc = (g.dtd[d] * u[d]) * ig;
        if (!(fabsf(dc) < 1.0f)) {   // a move of a cell or more breaks the deposit's support
            flags |= ERR_CFL;
            dc = dc > 0.0f ? 0.99f : -0.99f;
        }
        const int carry = move_carry(off[d], dc);
        c[d] = wrapi(c[d] + carry, g.n[d]);
    }
    return flags;
}

// True unless the particle kept its cell and offsets (then its current is zero).
__device__ __forceinline__ bool moved(const int c0[3], const int c1[3], const float o0[3], const float o1[3]) {
    return (c0[0] != c1[0]) | (c0[1] != c1[1]) | (c0[2] != c1[2]) | (o0[0] != o1[0]) | (o0[1] != o1[1]) |
           (o0[2] != o1[2]);
}

// Esirkepov current of one particle: for component x,
//   J_x[a][b][c] += (-q w) * P_x[a] * (M_y[b] M_z[c] + dS_y[b] dS_z[c] / 12)
// with P_x the running sum of dS_x along x and M = S0 + dS/2 (this product form
// equals dS_x (S0y S0z + dSy S0z/2 + S0y dSz/2 + dSy dSz/3) summed along x).
// Emit::add(comp, jx, jy, jz, k) receives each contribution as the int64
// k = round(2^40 (-q w) P Y), (jx, jy, jz) being union-node indices 0..4
// along x, y, z: the FP32 factor Q = 2^40 (-q w) Y is formed as
// fma((Q0 / 12) dS_y[b], dS_z[c], (Q0 M_y[b]) M_z[c]), Q0 = 2^40 (-q w), with
// the two scaled arrays of the first transverse axis computed once per
// component, and Q and P are multiplied exactly and rounded once.
// Callers skip particles that did not move (every contribution is zero).
template <class Emit>
__device__ __forceinline__ void esirkepov(const Axis5 A[3], float qw, Emit& em) {
    const float qw40 = qw * PIC_FIX_SCALE;   // exact: a power-of-two scale
    const float qw12 = qw40 * (1.0f / 12.0f);
    float M[3][5];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int j = 0; j < 5; ++j) M[d][j] = fmaf(0.5f, A[d].dS[j], A[d].S0[j]);
#pragma unroll
    for (int comp = 0; comp < 3; ++comp) {
        const int t1 = comp == 0 ? 1 : (comp == 1 ? 2 : 0);
        const int t2 = comp == 0 ? 2 : (comp == 1 ? 0 : 1);
        float P[4];
        P[0] = A[comp].dS[0];
#pragma unroll
        for (int a = 1; a < 4; ++a) P[a] = P[a - 1] + A[comp].dS[a];
        double Pd[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) Pd[a] = (double)P[a];
        const int la = A[comp].len - 1, lb = A[t1].len, lc = A[t2].len;
        float Mq[5], dSq[5];
#pragma unroll
        for (int b = 0; b < 5; ++b) {
            Mq[b] = qw40 * M[t1][b];
            dSq[b] = qw12 * A[t1].dS[b];
        }
#pragma unroll
        for (int cc = 0; cc < 5; ++cc) {
            if (cc >= lc) continue;
#pragma unroll
            for (int b = 0; b < 5; ++b) {
                if (b >= lb) continue;
                const double qy = (double)fmaf(dSq[b], A[t2].dS[cc], Mq[b] * M[t2][cc]);
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    if (a >= la) continue;
                    const long long k = fix_mul(qy, Pd[a]);
                    if (comp == 0)
                        em.add(0, a, b, cc, k);
                    else if (comp == 1)
                        em.add(1, cc, a, b, k);
                    else
                        em.add(2, b, cc, a, k);
                }
            }
        }
    }
}

// Emitter of deposit contributions into the global fixed-point accumulator.
struct GlobalEmit {
    unsigned long long* acc;
    int ncell;
    int X[5], Y[5], Z[5];
    __device__ __forceinline__ void add(int comp, int jx, int jy, int jz, long long k) const {
        atomicAdd(acc + ((size_t)comp * ncell + X[jx] + Y[jy] + Z[jz]), (unsigned long long)k);
    }
};

// One particle's move into the global accumulator.
__device__ __forceinline__ void deposit_global(const Geom& g, const int c0[3], const int c1[3], const float o0[3],
                                               const float o1[3], float wq, unsigned long long* acc) {
    const int stride[3] = {1, g.n[0], g.nxy};
    Axis5 A[3];
    GlobalEmit em;
    em.acc = acc;
    em.ncell = g.ncell;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        axis5(unwrap_shift(c1[d] - c0[d], g.n[d]), o0[d], o1[d], A[d]);
        int* dst = d == 0 ? em.X : (d == 1 ? em.Y : em.Z);
#pragma unroll
        for (int j = 0; j < 5; ++j) dst[j] = wrapi(c0[d] + A[d].base + j, g.n[d]) * stride[d];
    }
    esirkepov(A, wq, em);
}

// The same contributions in slots relative to the old cell, for the LDS
// deposits.  Along an axis transverse to the component, core slots 0..3 are
// the nodes at cell - 1 .. cell + 2 whatever the crossing, and slot 4 is the
// node that a crossing adds (cell + 3 forward, cell - 2 backward); along the
// component's own axis core slots 0..2 are cell - 1 .. cell + 1 and slot 3 is
// cell + 2 (forward) or cell - 2 (backward).  The old weights fill the core;
// the new ones sit one slot further on (forward, slot 4 the last of them) or
// back (backward, slot 4 the first).  Every sum is Axis5's and esirkepov's,
// in their order, so each node gets the same value bit for bit.
struct AxisSlots {
    float M[5], dS[5];   // S0 + dS / 2, dS; slot 4: the crossing's node
    float P[4];          // running sum of dS; slot 3: the crossing's
};

__device__ __forceinline__ void axis_slots(int di, float d0, float d1, AxisSlots& A) {
    const bool fwd = di > 0, back = di < 0;
    const float r1 = di == 0 ? d0 : (fwd ? 0.0f : 1.0f);
    const float r0 = di == 0 ? d0 : (fwd ? 1.0f : 0.0f);
    float W[4], Dn[4], Do[4];
    spline4(d0, W);
    dweight4(d1, r1, Dn);
    dweight4(r0, d0, Do);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float dn = fwd ? (j > 0 ? Dn[j - 1] : 0.0f) : (back ? (j < 3 ? Dn[j + 1] : 0.0f) : Dn[j]);
        A.dS[j] = dn + Do[j];
        A.M[j] = fmaf(0.5f, A.dS[j], W[j]);
    }
    A.dS[4] = fwd ? Dn[3] : Dn[0];
    A.M[4] = 0.5f * A.dS[4];
    A.P[0] = back ? A.dS[4] + A.dS[0] : A.dS[0];
    A.P[1] = A.P[0] + A.dS[1];
    A.P[2] = A.P[1] + A.dS[2];
    A.P[3] = back ? A.dS[4] : A.P[2] + A.dS[3];
}

// Emit::add(comp, sx, sy, sz, k) receives the contributions by slot.  A
// component's contributions over the slots [a0, a1) of its own axis and
// [b0, b1) x [c0, c1) of the next two.
template <int COMP, class Emit>
__device__ __forceinline__ void emit_slots(const AxisSlots A[3], float qw, int a0, int a1, int b0, int b1, int c0,
                                           int c1, const Emit& em) {
    constexpr int t1 = COMP == 0 ? 1 : (COMP == 1 ? 2 : 0);
    constexpr int t2 = COMP == 0 ? 2 : (COMP == 1 ? 0 : 1);
    const float qw40 = qw * PIC_FIX_SCALE;   // exact: a power-of-two scale
    const float qw12 = qw40 * (1.0f / 12.0f);
#pragma unroll
    for (int cc = 0; cc < 5; ++cc)
#pragma unroll
        for (int b = 0; b < 5; ++b) {
            if (cc < c0 || cc >= c1 || b < b0 || b >= b1) continue;   // (compile-time ranges)
            const float Mq = qw40 * A[t1].M[b], dSq = qw12 * A[t1].dS[b];
            const double qy = (double)fmaf(dSq, A[t2].dS[cc], Mq * A[t2].M[cc]);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                if (a < a0 || a >= a1) continue;
                const long long k = fix_mul(qy, (double)A[COMP].P[a]);
                if (COMP == 0)
                    em.add(0, a, b, cc, k);
                else if (COMP == 1)
                    em.add(1, cc, a, b, k);
                else
                    em.add(2, b, cc, a, k);
            }
        }
}

// The contributions of one component that involve a crossing's slot (x: which
// axes were crossed), by how many of its three axes were.
template <int COMP, class Emit>
__device__ __forceinline__ void emit_crossing(const AxisSlots A[3], float qw, const bool x[3], const Emit& em) {
    const bool xa = x[COMP], xb = x[COMP == 0 ? 1 : (COMP == 1 ? 2 : 0)], xc = x[COMP == 0 ? 2 : (COMP == 1 ? 0 : 1)];
    if (xa) emit_slots<COMP>(A, qw, 3, 4, 0, 4, 0, 4, em);
    if (xb) emit_slots<COMP>(A, qw, 0, 3, 4, 5, 0, 4, em);
    if (xc) emit_slots<COMP>(A, qw, 0, 3, 0, 4, 4, 5, em);
    if (xa && xb) emit_slots<COMP>(A, qw, 3, 4, 4, 5, 0, 4, em);
    if (xa && xc) emit_slots<COMP>(A, qw, 3, 4, 0, 4, 4, 5, em);
    if (xb && xc) {
        emit_slots<COMP>(A, qw, 0, 3, 4, 5, 4, 5, em);
        if (xa) emit_slots<COMP>(A, qw, 3, 4, 4, 5, 4, 5, em);
    }
}

}  // namespace pic
