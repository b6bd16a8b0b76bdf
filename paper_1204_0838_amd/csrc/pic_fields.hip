// FDTD field kernels: the B half step with the (optionally smoothed) curl of E,
// the E step with the standard curl of B and the current, the binomial current
// filter, and small utility kernels.
//
// Boundaries: y and z periodic, or (transverse absorbing layer) zero-valued
// beyond the y and z edges with the layer's stretched derivatives in its
// cells.  x periodic, or (moving window) a circular buffer in which the two
// planes where the window ends meet see zero-valued ghost fields across that
// seam.
//
// The layer (Section 3.1 surrounds the box transversely with a 16-layer
// PML) is the convolutional form: each transverse derivative D of a curl
// inside it is replaced by D + psi with psi <- b psi + (b - 1) D,
// b = exp(-sigma dt), sigma graded over the layer.  The two B half steps of
// a field step together are the leapfrog step of B between half-integer
// times, so the B arrays follow that recursion: the first half step of a
// step advances them with E^n, the second reads the value the next step's
// first half step will store (it sees the same E^{n+1}).
#include <algorithm>

#include "pic_internal.h"

namespace pic {

// A field value that an update leaves as it was (the pulse has not reached it)
// is not written back: wakefield run of 512x256x256 cells, B half step 264 ->
// 238 us, E update 523 -> 502 (fields that change everywhere: the same).  With
// the absorbing layer every value is written: its kernels are slower with the
// test (288x152x136 cells, a field step 279 -> 290 us).
template <bool PML>
__device__ __forceinline__ void put(float& f, float old, float v) {
    if (PML || __float_as_int(v) != __float_as_int(old)) f = v;
}

// Neighbour indices of one cell along each axis with the boundary rule.
struct Nbr {
    int i, j, k;              // cell
    int ip, im, jp, jm, kp, km;  // neighbour coordinates (wrapped)
    bool xp_ok, xm_ok;        // false when the x neighbour lies across the window seam
};

__device__ __forceinline__ Nbr neighbours(const Geom& g, int idx) {
    Nbr n;
    n.k = idx / g.nxy;
    const int r = idx - n.k * g.nxy;
    n.j = r / g.n[0];
    n.i = r - n.j * g.n[0];
    n.ip = n.i + 1 == g.n[0] ? 0 : n.i + 1;
    n.im = n.i == 0 ? g.n[0] - 1 : n.i - 1;
    n.jp = n.j + 1 == g.n[1] ? 0 : n.j + 1;
    n.jm = n.j == 0 ? g.n[1] - 1 : n.j - 1;
    n.kp = n.k + 1 == g.n[2] ? 0 : n.k + 1;
    n.km = n.k == 0 ? g.n[2] - 1 : n.k - 1;
    n.xp_ok = true;
    n.xm_ok = true;
    if (g.window) {
        int xw = n.i - g.origin;
        if (xw < 0) xw += g.n[0];
        n.xp_ok = xw != g.n[0] - 1;
        n.xm_ok = xw != 0;
    }
    return n;
}

__device__ __forceinline__ int at(const Geom& g, int i, int j, int k) { return i + g.n[0] * (j + g.n[1] * k); }

// B -= h curl' E with forward differences, curl'_x = D_y S_y E_z - D_z S_z E_y
// (cyclic), where S_axis is the transverse smoothing of the Section 2 stencil
// (identity for the Yee scheme): centre alpha_axis, +-t1 neighbours beta_t1,
// +-t2 neighbours beta_t2, the four corners gamma_{t1 t2}, t1 = axis + 1 and
// t2 = axis + 2 cyclically.  y and z are periodic; with the moving window,
// x neighbours across the window seam read as zero.
//
// A workgroup takes 64 x 8 columns and marches along z, one plane at a
// time: plane z + 1 of E (with its one-cell halo, in window coordinates, zeros
// beyond the window's two ends, or periodic images without a window) is
// staged in LDS while the values of planes z - 1 and z that the stencils need
// stay in registers.  A stencil's corner sum is the sum of its pair sums one
// plane up and down, so each new plane costs 26 LDS reads per cell for all
// twelve smoothed values; the 32x8x4-tile form it replaces read 80 (in 42
// instructions) and staged each plane twice.  The pair sums are formed and
// added in the stencil's own order: the results are the same bit for bit.
// HBM bounds it: 36 B per cell, 512x256x256 cells 327 -> 264 us (4.6 TB/s);
// with the layer, 288x152x136 cells, 84 -> 73 us.
// A grid narrower than 64 cells takes columns of 16 x 32 or 32 x 16 where they
// hold its x axis: 64 x 8 leaves most of their threads idle.  A field step, in
// tiles of 32 x 8 x 4, columns of 64 x 8, and these: 8x256x256 cells 58.5, 62.5
// and 36.3 us, with the layer 68.8, 77.2 and 42.0; 20x192x192 48.2, 49.0 and
// 34.6, with the layer 57.6, 59.1 and 43.4.
constexpr int BT_THREADS = 512;
template <int W>
struct BTile {
    static constexpr int X = W, Y = BT_THREADS / W;         // columns of a workgroup
    static constexpr int SX = X + 2, SY = Y + 2, N = SX * SY;   // staged cells of a plane
    static constexpr int PER = (N + BT_THREADS - 1) / BT_THREADS;
};
constexpr int kWide = 64;   // (the batch's columns for every member)

// Smoothed value from the centre, the sums over the +-t1 and +-t2 neighbours
// and over the four corners (in the order the terms are added).
__device__ __forceinline__ float smooth(const PDCoef& c, int axis, float ctr, float first, int t_first, float second,
                                        int t_second, float corners) {
    return fmaf(c.gam[axis], corners,
                fmaf(c.beta[t_second], second, fmaf(c.beta[t_first], first, c.alpha[axis] * ctr)));
}

// Centre value and pair sum of one stencil leg on planes z - 1 and z.
struct Leg {
    float f0, f1, s0, s1;
    __device__ __forceinline__ void push(float f, float s) {
        f0 = f1;
        s0 = s1;
        f1 = f;
        s1 = s;
    }
};

// S_x on plane z from a leg of +-y sums (order: y, z), S_y from a leg of +-x
// sums (order: z, x); f, s belong to plane z + 1.
template <bool PD>
__device__ __forceinline__ float smooth_x(const PDCoef& c, const Leg& l, float f, float s) {
    return PD ? smooth(c, 0, l.f1, l.s1, 1, f + l.f0, 2, s + l.s0) : l.f1;
}
template <bool PD>
__device__ __forceinline__ float smooth_y(const PDCoef& c, const Leg& l, float f, float s) {
    return PD ? smooth(c, 1, l.f1, f + l.f0, 2, l.s1, 0, s + l.s0) : l.f1;
}
// S_z on the staged plane itself (order: x, y).
template <bool PD>
__device__ __forceinline__ float smooth_z(const PDCoef& c, float ctr, float nx, float ny, float cr) {
    return PD ? smooth(c, 2, ctr, nx, 0, ny, 1, cr) : ctr;
}

// psi' = b psi + (b - 1) D (stored when `store`), returns D + psi'; old: the
// value of psi[q].
__device__ __forceinline__ float pml_stretch(float* __restrict__ psi, size_t q, float old, float b, float bm1, float D,
                                             bool store) {
    const float p = fmaf(b, old, bm1 * D);
    if (store) psi[q] = p;
    return D + p;
}

__device__ __forceinline__ float pml_stretch(float* __restrict__ psi, size_t q, float b, float bm1, float D,
                                             bool store) {
    return pml_stretch(psi, q, psi[q], b, bm1, D, store);
}

// Columns (bx, by), planes [z0, z1) of the B half step.
template <bool PD, bool PML, int W>
__device__ __forceinline__ void bhalf_columns(const Geom& g, const PDCoef& c, const float* __restrict__ Ex,
                                              const float* __restrict__ Ey, const float* __restrict__ Ez,
                                              float* __restrict__ Bx, float* __restrict__ By, float* __restrict__ Bz,
                                              float h, int bx, int by, int z0, int z1, float (*El)[3][BTile<W>::N],
                                              const PmlDev& P, bool store) {
    using T = BTile<W>;
    const int x0 = bx * T::X, y0 = by * T::Y;
    const int origin = g.window ? g.origin : 0;
    // the plane offsets of this thread's staged cells (the same on every plane)
    int so[T::PER];
    bool ok[T::PER];
#pragma unroll
    for (int q = 0; q < T::PER; ++q) {
        const int i = threadIdx.x + q * BT_THREADS;
        int xw = x0 - 1 + i % T::SX, y = y0 - 1 + i / T::SX;
        ok[q] = i < T::N;
        if (PML) ok[q] = ok[q] && y >= 0 && y < g.n[1];   // zero beyond the edges
        y = ((y % g.n[1]) + g.n[1]) % g.n[1];
        if (g.window)
            ok[q] = ok[q] && xw >= 0 && xw < g.n[0];
        else
            xw = ((xw % g.n[0]) + g.n[0]) % g.n[0];
        int xs = xw + origin;
        xs = xs >= g.n[0] ? xs - g.n[0] : xs;
        so[q] = ok[q] ? xs + g.n[0] * y : 0;
    }
    float v[T::PER][3];
    auto load = [&](int z) {
        const bool zok = !PML || (z >= 0 && z < g.n[2]);
        const int zw = z < 0 ? z + g.n[2] : (z >= g.n[2] ? z - g.n[2] : z);
#pragma unroll
        for (int q = 0; q < T::PER; ++q) {
            const int s = so[q] + g.nxy * zw;
            const bool in = ok[q] && zok;
            v[q][0] = in ? Ex[s] : 0.0f;
            v[q][1] = in ? Ey[s] : 0.0f;
            v[q][2] = in ? Ez[s] : 0.0f;
        }
    };
    const int x = threadIdx.x % T::X, y = threadIdx.x / T::X;
    const int xw = x0 + x, yy = y0 + y;
    const bool mine = xw < g.n[0] && yy < g.n[1];
    int xs = xw + origin;
    xs = xs >= g.n[0] ? xs - g.n[0] : xs;
    const int col = xs + g.n[0] * yy;
    constexpr int X = 1, Y = T::SX;
    const int o = (y + 1) * T::SX + (x + 1);
    // legs: S_y of E_x and E_z at y and y + 1, S_x of E_y and E_z at x and x + 1;
    // S_z of E_x and E_y on plane z
    Leg ex[2] = {}, ey[2] = {}, ezx[2] = {}, ezy[2] = {};
    float sxz = 0.0f, syz = 0.0f;
    // B and the layer's values of the plane finished next, loaded a plane ahead
    const int L2 = PML ? 2 * P.L : 0;
    const int jl = PML && mine ? pml_index(yy, g.n[1], P.L) : -1;
    float yb = 0.0f, ybm1 = 0.0f;
    if (PML && jl >= 0) {
        yb = P.coef[jl];            // axis y, B kind
        ybm1 = P.coef[L2 + jl];
    }
    const size_t yq0 = (size_t)xs + (size_t)g.n[0] * (size_t)(jl < 0 ? 0 : jl);
    const size_t yqz = (size_t)g.n[0] * (size_t)L2;
    float bn[3] = {0.0f, 0.0f, 0.0f}, pn[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto load_b = [&](int zc) {
        if (!mine || zc < z0 || zc >= z1) return;
        const int idx = col + g.nxy * zc;
        bn[0] = Bx[idx];
        bn[1] = By[idx];
        bn[2] = Bz[idx];
        if (PML) {
            if (jl >= 0) {
                pn[0] = P.y[0][yq0 + yqz * zc];
                pn[1] = P.y[1][yq0 + yqz * zc];
            }
            const int kl = pml_index(zc, g.n[2], P.L);
            if (kl >= 0) {
                const size_t q = (size_t)col + (size_t)g.nxy * kl;
                pn[2] = P.z[0][q];
                pn[3] = P.z[1][q];
            }
        }
    };
    load(z0 - 1);
    for (int z = z0 - 1, buf = 0; z <= z1; ++z, buf ^= 1) {
        float(*L)[T::N] = El[buf];
#pragma unroll
        for (int q = 0; q < T::PER; ++q) {
            const int i = threadIdx.x + q * BT_THREADS;
            if (i < T::N) {
                L[0][i] = v[q][0];
                L[1][i] = v[q][1];
                L[2][i] = v[q][2];
            }
        }
        __syncthreads();   // (the other buffer's readers are past their reads of the plane before)
        if (z < z1) load(z + 1);
        const float b0 = bn[0], b1 = bn[1], b2 = bn[2];
        const float p0 = pn[0], p1 = pn[1], p2 = pn[2], p3 = pn[3];
        load_b(z);
        if (!mine) continue;
        const int zc = z - 1;   // the plane that can be finished now
        const int idx = col + g.nxy * zc;
        const bool out = zc >= z0;
        const float* lx = L[0];
        const float* ly = L[1];
        const float* lz = L[2];
        // E_x: sums over +-x on rows y - 1, y, y + 1
        const float x00 = lx[o], x10 = lx[o + Y], xm0 = lx[o - Y];
        const float xn0 = lx[o + X] + lx[o - X], xn1 = lx[o + Y + X] + lx[o + Y - X], xnm = lx[o - Y + X] + lx[o - Y - X];
        const float sxz1 = smooth_z<PD>(c, x00, xn0, x10 + xm0, xn1 + xnm);
        // E_y
        const float y00 = ly[o], y01 = ly[o + X];
        const float yp0 = ly[o + Y], ym0 = ly[o - Y], yp1 = ly[o + Y + X], ym1 = ly[o - Y + X];
        const float yn0 = yp0 + ym0, yn1 = yp1 + ym1;
        const float syz1 = smooth_z<PD>(c, y00, y01 + ly[o - X], yn0, (yp1 + ly[o + Y - X]) + (ym1 + ly[o - Y - X]));
        // E_z
        const float z00 = lz[o], z10 = lz[o + Y], z01 = lz[o + X], z11 = lz[o + Y + X];
        const float zx0 = z01 + lz[o - X], zx1 = z11 + lz[o + Y - X];
        const float zy0 = z10 + lz[o - Y], zy1 = z11 + lz[o - Y + X];
        if (out) {
            float dyEz = (smooth_y<PD>(c, ezy[1], z10, zx1) - smooth_y<PD>(c, ezy[0], z00, zx0)) * g.inv_d[1];
            float dzEy = (syz1 - syz) * g.inv_d[2];
            float dzEx = (sxz1 - sxz) * g.inv_d[2];
            const float dxEz = (smooth_x<PD>(c, ezx[1], z01, zy1) - smooth_x<PD>(c, ezx[0], z00, zy0)) * g.inv_d[0];
            const float dxEy = (smooth_x<PD>(c, ey[1], y01, yn1) - smooth_x<PD>(c, ey[0], y00, yn0)) * g.inv_d[0];
            float dyEx = (smooth_y<PD>(c, ex[1], x10, xn1) - smooth_y<PD>(c, ex[0], x00, xn0)) * g.inv_d[1];
            if (PML) {
                if (jl >= 0) {
                    dyEz = pml_stretch(P.y[0], yq0 + yqz * zc, p0, yb, ybm1, dyEz, store);
                    dyEx = pml_stretch(P.y[1], yq0 + yqz * zc, p1, yb, ybm1, dyEx, store);
                }
                const int kl = pml_index(zc, g.n[2], P.L);
                if (kl >= 0) {
                    const size_t q = (size_t)col + (size_t)g.nxy * kl;
                    const float b = P.coef[4 * L2 + kl], bm1 = P.coef[5 * L2 + kl];  // axis z, B kind
                    dzEy = pml_stretch(P.z[0], q, p2, b, bm1, dzEy, store);
                    dzEx = pml_stretch(P.z[1], q, p3, b, bm1, dzEx, store);
                }
            }
            put<PML>(Bx[idx], b0, b0 - h * (dyEz - dzEy));
            put<PML>(By[idx], b1, b1 - h * (dzEx - dxEz));
            put<PML>(Bz[idx], b2, b2 - h * (dxEy - dyEx));
        }
        ex[0].push(x00, xn0);
        ex[1].push(x10, xn1);
        ey[0].push(y00, yn0);
        ey[1].push(y01, yn1);
        ezy[0].push(z00, zx0);
        ezy[1].push(z10, zx1);
        ezx[0].push(z00, zy0);
        ezx[1].push(z01, zy1);
        sxz = sxz1;
        syz = syz1;
    }
}

// Workgroups go round-robin over the 8 XCDs, each with its own L2: deal each
// XCD a contiguous run of workgroups (x fastest), so that neighbours' halos
// meet in one L2.  b -> position, of n.
__device__ __forceinline__ int xcd_run(int b, int n) {
    const int k = b % 8, q = n / 8, r = n % 8;
    return k * q + min(k, r) + b / 8;
}

// Planes per workgroup for `columns` workgroups side by side, `resident` of
// them on the chip at once: the shortest time in plane steps, rounds of
// workgroups times the planes that each stages (its own and two more), at most
// 16 (512x256x256 cells: 264 us with 16 planes, 288 with 64).
static int march_planes(int64_t columns, int nz, int resident) {
    int best = 1;
    int64_t cost = INT64_MAX;
    for (int z = 1; z <= 16; ++z) {
        const int64_t blocks = columns * ((nz + z - 1) / z);
        const int64_t c = (blocks + resident - 1) / resident * (z + 2);
        if (c < cost) {
            cost = c;
            best = z;
        }
    }
    return best;
}
constexpr int kMarchResident = 4 * 256;   // workgroups of 8 wavefronts: 32 wavefronts per CU

template <bool PD, bool PML, int W>
__global__ void __launch_bounds__(BT_THREADS) k_bhalf_march(Geom g, PDCoef c, const float* __restrict__ Ex,
                                                            const float* __restrict__ Ey,
                                                            const float* __restrict__ Ez, float* __restrict__ Bx,
                                                            float* __restrict__ By, float* __restrict__ Bz, float h,
                                                            int planes, PmlDev P, int store) {
    using T = BTile<W>;
    __shared__ float El[2][3][T::N];
    const int t = xcd_run(blockIdx.x, gridDim.x);
    const int tx = (g.n[0] + T::X - 1) / T::X, ty = (g.n[1] + T::Y - 1) / T::Y;
    const int bx = t % tx, by = (t / tx) % ty, z0 = (t / (tx * ty)) * planes;
    bhalf_columns<PD, PML, W>(g, c, Ex, Ey, Ez, Bx, By, Bz, h, bx, by, z0, min(z0 + planes, g.n[2]), El, P, store != 0);
}

// Where the E update takes its current from: the J planes (clearing the
// accumulator when a filter has read it); another buffer (the post-processed
// current), which it also stores to the J planes; or the fixed-point
// accumulator, which it rounds into the J planes and clears.
struct JSource {
    const float* in[3];
    unsigned long long* acc;
    float* J[3];
    double scale[3];
    int* rest_n;   // the species' rest-list counters (their passes are over): emptied on the way
};
// (Reading the accumulator here saves a read of J and a launch: 512x256x256
// cells of a wakefield run 634 -> 502 us together, 4.8 TB/s of the 72 B per
// cell that it reads, and writes where E and J are not zero.)
enum { J_PLANES = 0, J_COPY = 1, J_ACC = 2, J_CLEAR = 3 };

template <int SRC>
__device__ __forceinline__ float take_current(const JSource& s, int comp, int ncell, int idx) {
    if (SRC == J_ACC) {
        unsigned long long* a = s.acc + (size_t)comp * ncell + idx;
        const unsigned long long v = *a;
        const float j = (float)((double)(long long)v * s.scale[comp]);
        if (v) *a = 0ull;   // (vacuum and plasma at rest hold no current)
        s.J[comp][idx] = j;
        return j;
    }
    const float j = s.in[comp][idx];
    if (SRC == J_COPY) s.J[comp][idx] = j;
    if (SRC == J_CLEAR) s.acc[(size_t)comp * ncell + idx] = 0ull;
    return j;
}

// E += dt (curl B - J) with backward differences.
template <bool PML, int SRC>
__device__ __forceinline__ void efull_cell(const Geom& g, float* __restrict__ Ex, float* __restrict__ Ey,
                                           float* __restrict__ Ez, const float* __restrict__ Bx,
                                           const float* __restrict__ By, const float* __restrict__ Bz,
                                           const JSource& js, int idx, const PmlDev* P = nullptr) {
    const float jx = take_current<SRC>(js, 0, g.ncell, idx);
    const float jy = take_current<SRC>(js, 1, g.ncell, idx);
    const float jz = take_current<SRC>(js, 2, g.ncell, idx);
    const Nbr n = neighbours(g, idx);
    const float bz = Bz[idx], by = By[idx], bx = Bx[idx];
    const float bzm_x = n.xm_ok ? Bz[at(g, n.im, n.j, n.k)] : 0.0f;
    const float bym_x = n.xm_ok ? By[at(g, n.im, n.j, n.k)] : 0.0f;
    const bool ym_ok = !PML || n.j > 0, zm_ok = !PML || n.k > 0;   // zero beyond the layer's outer faces
    float dyBz = (bz - (ym_ok ? Bz[at(g, n.i, n.jm, n.k)] : 0.0f)) * g.inv_d[1];
    float dzBy = (by - (zm_ok ? By[at(g, n.i, n.j, n.km)] : 0.0f)) * g.inv_d[2];
    float dzBx = (bx - (zm_ok ? Bx[at(g, n.i, n.j, n.km)] : 0.0f)) * g.inv_d[2];
    const float dxBz = (bz - bzm_x) * g.inv_d[0];
    const float dxBy = (by - bym_x) * g.inv_d[0];
    float dyBx = (bx - (ym_ok ? Bx[at(g, n.i, n.jm, n.k)] : 0.0f)) * g.inv_d[1];
    if (PML) {
        const int L2 = 2 * P->L;
        const int jl = pml_index(n.j, g.n[1], P->L);
        if (jl >= 0) {
            const size_t q = (size_t)n.i + (size_t)g.n[0] * (size_t)(jl + L2 * n.k);
            const float b = P->coef[2 * L2 + jl], bm1 = P->coef[3 * L2 + jl];   // axis y, E kind
            dyBz = pml_stretch(P->y[2], q, b, bm1, dyBz, true);
            dyBx = pml_stretch(P->y[3], q, b, bm1, dyBx, true);
        }
        const int kl = pml_index(n.k, g.n[2], P->L);
        if (kl >= 0) {
            const size_t q = (size_t)n.i + (size_t)g.n[0] * (size_t)(n.j + g.n[1] * kl);
            const float b = P->coef[6 * L2 + kl], bm1 = P->coef[7 * L2 + kl];   // axis z, E kind
            dzBy = pml_stretch(P->z[2], q, b, bm1, dzBy, true);
            dzBx = pml_stretch(P->z[3], q, b, bm1, dzBx, true);
        }
    }
    const float ex = Ex[idx], ey = Ey[idx], ez = Ez[idx];
    put<PML>(Ex[idx], ex, ex + g.dt * ((dyBz - dzBy) - jx));
    put<PML>(Ey[idx], ey, ey + g.dt * ((dzBx - dxBz) - jy));
    put<PML>(Ez[idx], ez, ez + g.dt * ((dxBy - dyBx) - jz));
}

template <bool PML, int SRC>
__global__ void __launch_bounds__(256) k_efull(Geom g, float* __restrict__ Ex, float* __restrict__ Ey,
                                               float* __restrict__ Ez, const float* __restrict__ Bx,
                                               const float* __restrict__ By, const float* __restrict__ Bz, JSource js,
                                               PmlDev P) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= g.ncell) return;
    if (idx < kMaxSpecies) js.rest_n[idx] = 0;   // (a grid has 64 cells at least)
    efull_cell<PML, SRC>(g, Ex, Ey, Ez, Bx, By, Bz, js, idx, &P);
}

// Zero the layer's auxiliary values on storage x plane ix (the plane a
// window move turns into the new, empty leading plane).
__global__ void __launch_bounds__(256) k_clear_pml_plane(Geom g, PmlDev P, int ix) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const int L2 = 2 * P.L;
    if (t < L2 * g.n[2]) {
        const int l = t % L2, k = t / L2;
        const size_t q = (size_t)ix + (size_t)g.n[0] * (size_t)(l + L2 * k);
#pragma unroll
        for (int a = 0; a < 4; ++a) P.y[a][q] = 0.0f;
    }
    if (t < g.n[1] * L2) {
        const int j = t % g.n[1], l = t / g.n[1];
        const size_t q = (size_t)ix + (size_t)g.n[0] * (size_t)(j + g.n[1] * l);
#pragma unroll
        for (int a = 0; a < 4; ++a) P.z[a][q] = 0.0f;
    }
}

// One (1/4, 1/2, 1/4) pass along each axis, src -> dst (distinct buffers), one
// component: a thread takes one x and kBinRows rows and marches along z.  Each
// plane's x sums (kBinRows + 2 rows, three loads each) and y sums are formed
// once and kept in registers for the three planes that use them: 4.5 loads
// per value where the 27-point product stencil loaded 27, with the same sums
// in the same order (bit for bit).  288x152x136 cells: 308 -> 47 us (3.0 TB/s
// of the 24 B per cell).  y and z are periodic; x neighbours across the window
// seam read as zero.
constexpr int kBinRows = 4, kBinWaves = 4;   // a workgroup: 64 x by kBinWaves kBinRows rows

struct PlaneSource {   // an FP32 component
    const float* p;
    __device__ __forceinline__ float operator()(size_t i) const { return p[i]; }
};
struct AccSource {     // a component of the accumulator, as the read-out rounds it
    const unsigned long long* p;
    double scale;
    __device__ __forceinline__ float operator()(size_t i) const { return (float)((double)(long long)p[i] * scale); }
};

template <class Src>
__device__ __forceinline__ void binomial_march(const Geom& g, const Src& src, float* __restrict__ dst, int bx, int by,
                                               int z0, int z1) {
    const int i = bx * 64 + ((int)threadIdx.x & 63);
    const int j0 = (by * kBinWaves + ((int)threadIdx.x >> 6)) * kBinRows;
    if (i >= g.n[0] || j0 >= g.n[1]) return;
    const int ip = i + 1 == g.n[0] ? 0 : i + 1, im = i == 0 ? g.n[0] - 1 : i - 1;
    bool xp_ok = true, xm_ok = true;
    if (g.window) {
        int xw = i - g.origin;
        if (xw < 0) xw += g.n[0];
        xp_ok = xw != g.n[0] - 1;
        xm_ok = xw != 0;
    }
    int row[kBinRows + 2];
#pragma unroll
    for (int b = 0; b < kBinRows + 2; ++b) {
        int j = j0 - 1 + b;
        while (j >= g.n[1]) j -= g.n[1];   // (rows past the last wrap; they are not stored)
        row[b] = (j < 0 ? j + g.n[1] : j) * g.n[0];
    }
    float ym[kBinRows], yc[kBinRows];   // y sums of planes z - 2 and z - 1
#pragma unroll
    for (int b = 0; b < kBinRows; ++b) ym[b] = yc[b] = 0.0f;
    float v[kBinRows + 2][3];   // x - 1, x, x + 1 of each row: the next plane's, loaded a plane ahead
    auto load = [&](int z) {
        const size_t p = (size_t)g.nxy * (z < 0 ? z + g.n[2] : (z >= g.n[2] ? z - g.n[2] : z));
#pragma unroll
        for (int b = 0; b < kBinRows + 2; ++b) {
            v[b][0] = xm_ok ? src(p + row[b] + im) : 0.0f;
            v[b][1] = src(p + row[b] + i);
            v[b][2] = xp_ok ? src(p + row[b] + ip) : 0.0f;
        }
    };
    load(z0 - 1);
    for (int z = z0 - 1; z <= z1; ++z) {
        float ax[kBinRows + 2];
#pragma unroll
        for (int b = 0; b < kBinRows + 2; ++b)
            ax[b] = fmaf(0.25f, v[b][2], fmaf(0.5f, v[b][1], fmaf(0.25f, v[b][0], 0.0f)));
        if (z < z1) load(z + 1);
#pragma unroll
        for (int b = 0; b < kBinRows; ++b) {
            const float ay = fmaf(0.25f, ax[b + 2], fmaf(0.5f, ax[b + 1], fmaf(0.25f, ax[b], 0.0f)));
            if (z > z0 && j0 + b < g.n[1])
                dst[i + g.n[0] * (j0 + b) + (size_t)g.nxy * (z - 1)] =
                    fmaf(0.25f, ay, fmaf(0.5f, yc[b], fmaf(0.25f, ym[b], 0.0f)));
            ym[b] = yc[b];
            yc[b] = ay;
        }
    }
}

struct BinArgs {
    const float* s[3];
    const unsigned long long* acc;
    double scale[3];
    float* d[3];
};

template <bool ACC>
__global__ void __launch_bounds__(64 * kBinWaves) k_binomial(Geom g, BinArgs p, int planes, int chunks) {
    const int tx = (g.n[0] + 63) / 64, ty = (g.n[1] + kBinWaves * kBinRows - 1) / (kBinWaves * kBinRows);
    const int t = xcd_run(blockIdx.x, gridDim.x);   // x fastest, then y, plane chunk, component
    const int u = t / (tx * ty), comp = u / chunks, z0 = (u - comp * chunks) * planes;
    const int bx = t % tx, by = (t / tx) % ty, z1 = min(z0 + planes, g.n[2]);
    if (ACC)
        binomial_march(g, AccSource{p.acc + (size_t)comp * g.ncell, p.scale[comp]}, p.d[comp], bx, by, z0, z1);
    else
        binomial_march(g, PlaneSource{p.s[comp]}, p.d[comp], bx, by, z0, z1);
}

// Batched field kernels: grid y = member.
constexpr int kBatchPlanes = 8;   // planes per workgroup of the batched marches

// Grid x = workgroup (x fastest, then y, then plane chunk) of the member's grid.
__global__ void __launch_bounds__(BT_THREADS) k_batch_bhalf(const InstDesc* __restrict__ tab) {
    using T = BTile<kWide>;
    __shared__ float El[2][3][T::N];
    const InstDesc& d = tab[blockIdx.y];
    const Geom g = d.g;
    const int tx = (g.n[0] + T::X - 1) / T::X, ty = (g.n[1] + T::Y - 1) / T::Y;
    const int t = blockIdx.x;
    if (t >= tx * ty * ((g.n[2] + kBatchPlanes - 1) / kBatchPlanes)) return;
    const PDCoef c = d.c;
    const int bx = t % tx, by = (t / tx) % ty, z0 = (t / (tx * ty)) * kBatchPlanes;
    const int z1 = min(z0 + kBatchPlanes, g.n[2]);
    const PmlDev none{};
    if (d.pd)
        bhalf_columns<true, false, kWide>(g, c, d.f.E[0], d.f.E[1], d.f.E[2], d.f.B[0], d.f.B[1], d.f.B[2], d.hdt, bx, by,
                                   z0, z1, El, none, false);
    else
        bhalf_columns<false, false, kWide>(g, c, d.f.E[0], d.f.E[1], d.f.E[2], d.f.B[0], d.f.B[1], d.f.B[2], d.hdt, bx, by,
                                    z0, z1, El, none, false);
}

// A member without post-processing takes its current from the accumulator.
__global__ void __launch_bounds__(256) k_batch_efull(const InstDesc* __restrict__ tab) {
    const InstDesc& d = tab[blockIdx.y];
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= d.g.ncell) return;
    const Geom g = d.g;
    JSource js;
    for (int a = 0; a < 3; ++a) {
        js.in[a] = d.J[a];
        js.J[a] = d.J[a];
        js.scale[a] = d.jscale[a];
    }
    js.acc = d.acc;
    if (d.jpost)
        efull_cell<false, J_CLEAR>(g, d.f.E[0], d.f.E[1], d.f.E[2], d.f.B[0], d.f.B[1], d.f.B[2], js, idx);
    else
        efull_cell<false, J_ACC>(g, d.f.E[0], d.f.E[1], d.f.E[2], d.f.B[0], d.f.B[1], d.f.B[2], js, idx);
}

// Grid x = workgroup of the member's grid, z = component.
__global__ void __launch_bounds__(64 * kBinWaves) k_batch_binomial(const InstDesc* __restrict__ tab) {
    const InstDesc& d = tab[blockIdx.y];
    if (!d.jpost) return;
    const Geom g = d.g;
    const int tx = (g.n[0] + 63) / 64, ty = (g.n[1] + kBinWaves * kBinRows - 1) / (kBinWaves * kBinRows);
    const int t = blockIdx.x, z0 = (t / (tx * ty)) * kBatchPlanes, comp = blockIdx.z;
    if (z0 >= g.n[2]) return;
    binomial_march(g, AccSource{d.acc + (size_t)comp * g.ncell, d.jscale[comp]}, d.J[comp], t % tx, (t / tx) % ty, z0,
                   min(z0 + kBatchPlanes, g.n[2]));
}

__global__ void k_zero_u64(unsigned long long* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

template <int W>
static hipError_t launch_bhalf_w(const Geom& g, int pd, const PDCoef& c, float* const E[3], float* const B[3], float h,
                                 const PmlDev* pml, int store, hipStream_t st) {
    using T = BTile<W>;
    const int bx = (g.n[0] + T::X - 1) / T::X, by = (g.n[1] + T::Y - 1) / T::Y;
    const int planes = march_planes((int64_t)bx * by, g.n[2], kMarchResident);
    const dim3 nb(bx * by * ((g.n[2] + planes - 1) / planes));
    const PmlDev P = pml ? *pml : PmlDev{};
    auto k = pd ? (pml ? k_bhalf_march<true, true, W> : k_bhalf_march<true, false, W>)
                : (pml ? k_bhalf_march<false, true, W> : k_bhalf_march<false, false, W>);
    hipLaunchKernelGGL(k, nb, dim3(BT_THREADS), 0, st, g, c, E[0], E[1], E[2], B[0], B[1], B[2], h, planes, P, store);
    return hipGetLastError();
}

hipError_t launch_bhalf(const Geom& g, int pd, const PDCoef& c, float* const E[3], float* const B[3], float h,
                        const PmlDev* pml, int store, hipStream_t st) {
    return g.n[0] <= 16   ? launch_bhalf_w<16>(g, pd, c, E, B, h, pml, store, st)
           : g.n[0] <= 32 ? launch_bhalf_w<32>(g, pd, c, E, B, h, pml, store, st)
                          : launch_bhalf_w<kWide>(g, pd, c, E, B, h, pml, store, st);
}

hipError_t launch_efull(const Geom& g, float* const E[3], float* const B[3], float* const J[3], float* const Jcopy[3],
                        unsigned long long* acc, const double* scale, int* rest_n, const PmlDev* pml, hipStream_t st) {
    const int nb = (g.ncell + 255) / 256;
    const PmlDev P = pml ? *pml : PmlDev{};
    JSource js{};
    for (int a = 0; a < 3; ++a) {
        js.in[a] = J[a];
        js.J[a] = Jcopy ? Jcopy[a] : J[a];
        if (scale) js.scale[a] = scale[a];
    }
    js.acc = acc;
    js.rest_n = rest_n;
    auto k = acc && scale ? (pml ? k_efull<true, J_ACC> : k_efull<false, J_ACC>)
             : acc        ? (pml ? k_efull<true, J_CLEAR> : k_efull<false, J_CLEAR>)
                 : Jcopy ? (pml ? k_efull<true, J_COPY> : k_efull<false, J_COPY>)
                         : (pml ? k_efull<true, J_PLANES> : k_efull<false, J_PLANES>);
    hipLaunchKernelGGL(k, dim3(nb), dim3(256), 0, st, g, E[0], E[1], E[2], B[0], B[1], B[2], js, P);
    return hipGetLastError();
}

hipError_t launch_clear_pml_plane(const Geom& g, const PmlDev& P, int ix, hipStream_t st) {
    const int n = std::max(2 * P.L * g.n[2], 2 * P.L * g.n[1]);
    hipLaunchKernelGGL(k_clear_pml_plane, dim3((n + 255) / 256), dim3(256), 0, st, g, P, ix);
    return hipGetLastError();
}

hipError_t launch_binomial(const Geom& g, float* const src[3], const unsigned long long* acc, const double scale[3],
                           float* const dst[3], hipStream_t st) {
    const int bx = (g.n[0] + 63) / 64, by = (g.n[1] + kBinWaves * kBinRows - 1) / (kBinWaves * kBinRows);
    const int planes = march_planes(3ll * bx * by, g.n[2], 2 * kMarchResident), chunks = (g.n[2] + planes - 1) / planes;
    BinArgs p{};
    for (int a = 0; a < 3; ++a) {
        if (src) p.s[a] = src[a];
        if (scale) p.scale[a] = scale[a];
        p.d[a] = dst[a];
    }
    p.acc = acc;
    hipLaunchKernelGGL(src ? k_binomial<false> : k_binomial<true>, dim3(bx * by * 3 * chunks), dim3(64 * kBinWaves), 0,
                       st, g, p, planes, chunks);
    return hipGetLastError();
}

hipError_t launch_batch_bhalf(const InstDesc* d, int n, int max_tiles, hipStream_t st) {
    if (n <= 0 || max_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_bhalf, dim3(max_tiles, n), dim3(BT_THREADS), 0, st, d);
    return hipGetLastError();
}

int bhalf_tiles(const int n[3]) {
    using T = BTile<kWide>;
    return ((n[0] + T::X - 1) / T::X) * ((n[1] + T::Y - 1) / T::Y) * ((n[2] + kBatchPlanes - 1) / kBatchPlanes);
}

int binomial_tiles(const int n[3]) {
    return ((n[0] + 63) / 64) * ((n[1] + kBinWaves * kBinRows - 1) / (kBinWaves * kBinRows)) *
           ((n[2] + kBatchPlanes - 1) / kBatchPlanes);
}

hipError_t launch_batch_efull(const InstDesc* d, int n, int max_cells, hipStream_t st) {
    if (n <= 0 || max_cells <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_efull, dim3((max_cells + 255) / 256, n), dim3(256), 0, st, d);
    return hipGetLastError();
}

hipError_t launch_batch_binomial(const InstDesc* d, int n, int max_tiles, hipStream_t st) {
    if (n <= 0 || max_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_binomial, dim3(max_tiles, n, 3), dim3(64 * kBinWaves), 0, st, d);
    return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long* p, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t nb = (n + 255) / 256;
    hipLaunchKernelGGL(k_zero_u64, dim3((unsigned)nb), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

}  // namespace pic
