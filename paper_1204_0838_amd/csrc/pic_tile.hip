// Fused gather + push + move + deposit over cell-sorted particle tiles.
//
// One workgroup per tile of T[0] x T[1] x T[2] cells.  The workgroup stages
// E and B of the tile plus a halo of H = guard + 2 cells in LDS, zeroes an
// int64 current tile covering the tile plus guard + 2 (low) / guard + 3 (high)
// cells, and then streams its particles (coalesced SoA loads):
//   particles still within `guard` cells of the tile: gather from LDS,
//     deposit with LDS 64-bit atomics;
//   particles that drifted further since the last sort: left for a second
//     kernel (their cell index is replaced by -2 - cell and their index is
//     appended to the species' rest list, one atomic per wavefront), which
//     gathers from global memory and deposits with global atomics (the same
//     arithmetic).  Keeping that path out of the tile kernel keeps its loop
//     free of calls, so the kernel arguments stay in scalar registers.
// Finally the non-zero LDS current is added to the global fixed-point
// accumulator in one atomic pass.  The step right after a sort also does the
// sort's gather: the sort leaves each destination's source index in the
// cell array, and this kernel reads every particle through it from the
// pre-sort arrays and writes all of its arrays at the destination.  Every value goes through the same device
// functions as the split kernels, so the fused and split paths agree bit for
// bit (integer sums are order-independent).
//
// Workgroups are mapped to tiles XCD by XCD: consecutive workgroup indices go
// round-robin over the 8 XCDs, and the tiles are dealt to the XCDs in chunks
// (a row of tiles along x for one grid, 8 tiles of the concatenated list for a
// batch): XCD k takes chunks k, k + 8, k + 16, ...  Neighbouring tiles of a
// row share their halos in that XCD's L2, while a dense region (the wake on
// the axis) is spread over all XCDs instead of loading one of them.
#include <algorithm>

#include "pic_internal.h"
#include "pic_particle_ops.h"

namespace pic {

// LDS current tile, addressed by slots relative to the particle's old cell
// (AxisSlots): `base` is the lane's node at its old cell - 1 along each axis
// (slot 0, component 0), and every core slot is base plus an offset that is a
// compile-time constant for the compiled tile shapes (the whole core stencil
// of all three components lies within the 16-bit immediate offset of
// ds_add_u64), so lanes in distinct cells stay in distinct banks whether or
// not, and which way, they crossed a cell face.
struct LdsCore {
    unsigned long long* base;
    int jx, jpl, jr;                // row, plane and component strides
    __device__ __forceinline__ void add(int comp, int sx, int sy, int sz, long long k) const {
        atomicAdd(base + (comp * jr + sx + sy * jx + sz * jpl), (unsigned long long)k);
    }
};

// The same with a crossing's slots, which take a per-lane correction: they are
// written as the forward node (slot 4 = old cell + 3, or along the
// component's own axis slot 3 = old cell + 2) and moved to old cell - 2 for a
// backward crossing.
struct LdsCrossing {
    unsigned long long* base;
    int jx, jpl, jr;
    int dxm, dym, dzm;              // backward corrections of the transverse extra slot (elements)
    int dxp, dyp, dzp;              // ... and of the own-axis extra slot
    __device__ __forceinline__ void add(int comp, int sx, int sy, int sz, long long k) const {
        const int off = comp * jr + sx + sy * jx + sz * jpl;
        int corr = 0;
        if (comp == 0 ? sx == 3 : sx == 4) corr += comp == 0 ? dxp : dxm;
        if (comp == 1 ? sy == 3 : sy == 4) corr += comp == 1 ? dyp : dym;
        if (comp == 2 ? sz == 3 : sz == 4) corr += comp == 2 ? dzp : dzm;
        atomicAdd(base + (off + corr), (unsigned long long)k);
    }
};

// Tile of workgroup b when chunks of `chunk` consecutive tiles are dealt
// round-robin to the 8 XCDs (>= ntiles: no tile; grid = xcd_blocks).
// v mod n in [0, n) for any v; a single compare when v is already inside
// (the staging and flush loops wrap only at the domain's faces).
__device__ __forceinline__ int wrap_any(int v, int n) {
    return (unsigned)v < (unsigned)n ? v : ((v % n) + n) % n;
}

__device__ __forceinline__ int xcd_tile(int b, int ntiles, int chunk) {
    const int k = b % 8, j = b / 8;
    const int c = k + 8 * (j / chunk);
    const long long tile = (long long)c * chunk + j % chunk;
    return tile < ntiles ? (int)tile : ntiles;
}

static __host__ __device__ int xcd_blocks(int ntiles, int chunk) {
    const int nchunks = (ntiles + chunk - 1) / chunk;
    return 8 * ((nchunks + 7) / 8) * chunk;
}

constexpr int kBatchChunk = 8;

// One particle (index p, cell coordinates c) through global memory: gather,
// push, move, store, deposit with global atomics.  Returns error flags.
__device__ __forceinline__ int push_deposit_global(const Geom& g, const FieldPtrs& f, const SpeciesDev& s, int p,
                                                const int c[3], unsigned long long* acc) {
    const int gstride[3] = {1, g.n[0], g.nxy};
    float o[3] = {s.off[0][p], s.off[1][p], s.off[2][p]};
    const float o0[3] = {o[0], o[1], o[2]};
    float u[3] = {s.u[0][p], s.u[1][p], s.u[2][p]};
    GatherStencil st;
    gather_stencil(o, st);
    int ii[3][4], ih[3][4];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            ii[d][a] = wrapi(c[d] - 1 + a, g.n[d]) * gstride[d];
            ih[d][a] = wrapi(c[d] + st.hb[d] + a, g.n[d]) * gstride[d];
        }
    float E[3], B[3];
    gather_fields(f.E, f.B, ii, ih, st, E, B);
    int c1[3] = {c[0], c[1], c[2]};
    const int errs = push_move(g, s.qmh, E, B, u, o, c1);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        s.u[d][p] = u[d];
        s.off[d][p] = o[d];
    }
    s.cell[p] = c1[0] + g.n[0] * (c1[1] + g.n[1] * c1[2]);
    if (moved(c, c1, o0, o)) deposit_global(g, c, c1, o0, o, s.mq * s.w[p], acc);
    return errs;
}

// Plane (z) strides of the two LDS regions, padded so that one z step moves
// the address by 8 banks: fields in 4-byte words mod 32, current in 8-byte
// words mod 16.  The sort stores a tile's cells as 8x2x4 bricks (x, then 4 z,
// then 2 y), so at 8 particles per cell the lanes of one LDS pass (32 for
// the b32 field reads, 16 for the int64 atomics) sit in 8 x-cells of 4 (or
// 2) successive z-planes and address disjoint banks.
__host__ __device__ constexpr int pad_plane(int p, int m) { return p + ((8 - p % m) + m) % m; }
__host__ __device__ constexpr int field_plane(int fx, int fy) { return pad_plane(fx * fy, 32); }
__host__ __device__ constexpr int cur_plane(int jx, int jy) { return pad_plane(jx * jy, 16); }

// Load particle pn of the tile's range.  With GATHER the step runs right
// after a sort that left only each destination's source index in s.cell:
// the particle is read from src at that index, and w and id, which the step
// does not change, are written to the destination at once (the step writes
// the other arrays), so the sort needs no copy pass of its own.
template <bool GATHER>
__device__ __forceinline__ void load_particle(const SpeciesDev& s, const SpeciesDev& src, int pn, int& cell,
                                              float o[3], float u[3], float& w) {
    if (GATHER) {
        const int ps = s.cell[pn];
        cell = src.cell[ps];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            o[d] = src.off[d][ps];
            u[d] = src.u[d][ps];
        }
        w = src.w[ps];
        s.w[pn] = w;
        s.id[pn] = src.id[ps];
    } else {
        cell = s.cell[pn];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            o[d] = s.off[d][pn];
            u[d] = s.u[d][pn];
        }
        w = s.w[pn];
    }
}

// Offsets and momenta of particle p written unchanged (a gathering step's
// particles that it does not push here still need them at their new place).
template <bool GATHER>
__device__ __forceinline__ void keep_particle(const SpeciesDev& s, int p, const float o[3], const float u[3]) {
    if (GATHER) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            s.off[d][p] = o[d];
            s.u[d][p] = u[d];
        }
    }
}

// Add the non-zero LDS current of a tile at t0 (its region starting `lo`
// cells before it) to the global accumulator.
template <int NT>
__device__ __forceinline__ void flush_current(const Geom& g, const int t0[3], int lo, int jx, int jpl, int jr,
                                              const unsigned long long* Jl, unsigned long long* __restrict__ acc) {
    for (int i = threadIdx.x; i < 3 * jr; i += NT) {
        const unsigned long long v = Jl[i];
        if (v == 0ull) continue;   // (the padding of each plane stays zero)
        const int comp = i / jr;
        const int k = i - comp * jr;
        const int lz = k / jpl;
        const int rr = k - lz * jpl;
        const int ly = rr / jx;
        const int lx = rr - ly * jx;
        int gx = t0[0] - lo + lx, gy = t0[1] - lo + ly, gz = t0[2] - lo + lz;
        gx = wrap_any(gx, g.n[0]);
        gy = wrap_any(gy, g.n[1]);
        gz = wrap_any(gz, g.n[2]);
        atomicAdd(acc + ((size_t)comp * g.ncell + gx + g.n[0] * (gy + g.n[1] * gz)), v);
    }
}

// Deposit into a tile's LDS region, one particle per lane, in two parts.  The
// core part (3 x 48 contributions, `core`) is every moving particle's.  The
// contributions that a cell crossing adds (up to 156 more) concern a third of
// the particles at most, but nearly every wavefront has a lane among them,
// and a wavefront that runs them for a few lanes pays for all 64.  So `cross`
// only queues the crossing lanes' particles, in five registers per lane (old
// offsets, index, cell and crossings; moved there by ds_permute), and their
// contributions are added when 64 are waiting, and at the tile's end
// (`finish`); new offsets and weights are read back from s, where they are
// stored by then.  (Kept in the queue as well, eight registers, they made the
// 1024-thread kernels spill up to 11: two steps of a 512x256x256 wakefield
// 26.46 ms against 26.03.)  Sums are integers: the order does not matter.
// Every lane of the wavefront calls cross and finish.
// An LDS atomic costs a wavefront 6 cycles however few lanes are active, 8
// with two-way bank conflicts.  Measured against running the crossings with the
// rest (tile launch, 512 threads): wakefield 256x120x120 cells 2596 -> 2341 us,
// warm plasma of 5.7e6 particles 824 -> 781.
struct TileDeposit {
    unsigned long long* Jl;
    int guard, jx, jpl, jr;
    float q[3];    // the queued particle of this lane: old offsets
    int qp;        // its index
    int qkey;      // its local cell (+ guard, 5 bits per axis) and crossings (+ 1, 2 bits per axis)
    int waiting;   // queued particles: lanes 0 .. waiting - 1 (the same in every lane)

    __device__ __forceinline__ void init(unsigned long long* lds, int g, int row, int plane, int region) {
        Jl = lds;
        guard = g;
        jx = row;
        jpl = plane;
        jr = region;
        waiting = 0;
        qkey = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) q[k] = 0.0f;
        qp = 0;
    }

    // lc: old cell relative to the tile; di: cells crossed (-1, 0, 1)
    __device__ __forceinline__ void core(const int lc[3], const int di[3], const float o0[3], const float o1[3],
                                         float wq) const {
        AxisSlots A[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) axis_slots(di[d], o0[d], o1[d], A[d]);
        const LdsCore em{Jl + ((lc[0] + guard + 1) + (lc[1] + guard + 1) * jx + (lc[2] + guard + 1) * jpl), jx, jpl,
                         jr};
        emit_slots<0>(A, wq, 0, 3, 0, 4, 0, 4, em);
        emit_slots<1>(A, wq, 0, 3, 0, 4, 0, 4, em);
        emit_slots<2>(A, wq, 0, 3, 0, 4, 0, 4, em);
    }

    // (the lanes' stores of new offsets and weights come before the reads: a
    // workgroup's stores and loads go through one L1)
    __device__ __forceinline__ void extra(const SpeciesDev& s) const {
        AxisSlots A[3];
        int di[3], lc[3];
        bool x[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lc[d] = (qkey >> (5 * d)) & 31;
            di[d] = ((qkey >> (15 + 2 * d)) & 3) - 1;
            x[d] = di[d] != 0;
            axis_slots(di[d], q[d], s.off[d][qp], A[d]);
        }
        LdsCrossing em;
        em.base = Jl + ((lc[0] + 1) + (lc[1] + 1) * jx + (lc[2] + 1) * jpl);
        em.jx = jx;
        em.jpl = jpl;
        em.jr = jr;
        em.dxm = di[0] < 0 ? -5 : 0;
        em.dxp = di[0] < 0 ? -4 : 0;
        em.dym = di[1] < 0 ? -5 * jx : 0;
        em.dyp = di[1] < 0 ? -4 * jx : 0;
        em.dzm = di[2] < 0 ? -5 * jpl : 0;
        em.dzp = di[2] < 0 ? -4 * jpl : 0;
        const float wq = s.mq * s.w[qp];
        emit_crossing<0>(A, wq, x, em);
        emit_crossing<1>(A, wq, x, em);
        emit_crossing<2>(A, wq, x, em);
    }

    // Queue the lanes with `crossed`; when the queue fills, add its 64.
    __device__ __forceinline__ void cross(const SpeciesDev& s, bool crossed, const int lc[3], const int di[3],
                                          const float o0[3], int p) {
        const unsigned long long m = __ballot(crossed);
        if (m == 0ull) return;
        const int lane = __lane_id(), k = __popcll(m);
        const unsigned long long below = (1ull << lane) - 1ull;
        // crossing lanes go to places waiting, waiting + 1, ... (mod 64), the others to the rest
        const int to = (waiting + (crossed ? __popcll(m & below) : k + __popcll(~m & below))) & 63;
        float r[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) r[d] = __int_as_float(__builtin_amdgcn_ds_permute(to << 2, __float_as_int(o0[d])));
        const int rp = __builtin_amdgcn_ds_permute(to << 2, p);
        int key = 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) key |= ((lc[d] + guard) << (5 * d)) | ((di[d] + 1) << (15 + 2 * d));
        const int rkey = __builtin_amdgcn_ds_permute(to << 2, key);
        int end = waiting + k;
        take(lane >= waiting && lane < end, r, rp, rkey);
        if (end >= 64) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            extra(s);
            end -= 64;
            take(lane < end, r, rp, rkey);
        }
        waiting = end;
    }

    __device__ __forceinline__ void finish(const SpeciesDev& s) const {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        if ((int)__lane_id() < waiting) extra(s);
    }

  private:
    __device__ __forceinline__ void take(bool mine, const float r[3], int rp, int rkey) {
#pragma unroll
        for (int k = 0; k < 3; ++k) q[k] = mine ? r[k] : q[k];
        qp = mine ? rp : qp;
        qkey = mine ? rkey : qkey;
    }
};

// Body of the fused step for one tile (the whole workgroup cooperates).
// TX, TY, TZ > 0 and GD >= 0 fix the tile shape and guard at compile time:
// every LDS stride is then a constant and each particle's current atomics
// and field reads address LDS as one base register plus immediate offsets.
// 0 (-1 for GD) takes them from t and guard_rt.
template <int NT, int TX = 0, int TY = 0, int TZ = 0, int GD = -1, bool GATHER = false>
__device__ __forceinline__ void tile_body(const Geom& g, const TileGeom& t, int guard_rt, const FieldPtrs& f,
                                          const SpeciesDev& s, const SpeciesDev& src, const int* __restrict__ toff,
                                          unsigned long long* __restrict__ acc, int* __restrict__ d_err,
                                          int* __restrict__ rest_n, int* __restrict__ rest_idx,
                                          unsigned long long* lds_u64, int tile, int part = 0, int parts = 1) {
    int pb = toff[tile], n = toff[tile + 1] - pb;
    if (parts > 1) {   // this workgroup's share of the tile's particles, in whole wavefronts
        const int share = ((n + parts - 1) / parts + 63) & ~63;
        pb += part * share;
        n = min(n - part * share, share);
    }
    if (n <= 0) return;
    const int T[3] = {TX > 0 ? TX : t.T[0], TY > 0 ? TY : t.T[1], TZ > 0 ? TZ : t.T[2]};
    const int guard = GD >= 0 ? GD : guard_rt;
    const int tz = tile / (t.nt[0] * t.nt[1]);
    const int tr = tile - tz * t.nt[0] * t.nt[1];
    const int ty = tr / t.nt[0];
    const int tx = tr - ty * t.nt[0];
    const int t0[3] = {tx * T[0], ty * T[1], tz * T[2]};
    int te[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) te[d] = min(T[d], g.n[d] - t0[d]);
    const int H = guard + 2;
    // LDS geometry (region sizes use the full tile size T, ragged tiles use part of it)
    const int fx = T[0] + 2 * H, fy = T[1] + 2 * H, fz = T[2] + 2 * H;
    const int fpl = field_plane(fx, fy);
    const int fr = fpl * fz;
    const int jx = T[0] + 2 * guard + 5, jy = T[1] + 2 * guard + 5, jz = T[2] + 2 * guard + 5;
    const int jpl = cur_plane(jx, jy);
    const int jr = jpl * jz;
    unsigned long long* Jl = lds_u64;
    float* Fl = reinterpret_cast<float*>(lds_u64 + 3 * jr);

    for (int i = threadIdx.x; i < 3 * jr; i += NT) Jl[i] = 0ull;
    // stage E, B (tile + halo, periodic wrap in storage coordinates); note
    // whether any staged value is other than +0
    unsigned int bits = 0u;
    for (int i = threadIdx.x; i < fx * fy * fz; i += NT) {
        const int lz = i / (fx * fy);
        const int rr = i - lz * fx * fy;
        const int ly = rr / fx;
        const int lx = rr - ly * fx;
        int gx = t0[0] - H + lx, gy = t0[1] - H + ly, gz = t0[2] - H + lz;
        gx = wrap_any(gx, g.n[0]);
        gy = wrap_any(gy, g.n[1]);
        gz = wrap_any(gz, g.n[2]);
        const int gi = gx + g.n[0] * (gy + g.n[1] * gz);
        const int li = lz * fpl + rr;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float e = f.E[c][gi], b = f.B[c][gi];
            Fl[c * fr + li] = e;
            Fl[(3 + c) * fr + li] = b;
            bits |= __float_as_uint(e) | __float_as_uint(b);
        }
    }
    // A cold tile: every staged field value is +0 (ahead of the laser).  There a
    // particle with u = +0 gathers E = B = +0, and the push, move and deposit
    // leave it exactly as it is (u stays +0, the offsets and the cell do not
    // change, nothing moves so nothing is deposited): it is skipped.
    const bool cold_tile = __syncthreads_or(bits != 0u) == 0;

    float* const El[3] = {Fl, Fl + fr, Fl + 2 * fr};
    float* const Bl[3] = {Fl + 3 * fr, Fl + 4 * fr, Fl + 5 * fr};
    const int fstride[3] = {1, fx, fpl};
    int errs = 0;
    TileDeposit dep;
    dep.init(Jl, guard, jx, jpl, jr);
    // software pipeline: the next particle's SoA loads are issued before the
    // current particle is processed (not in the 1024-thread launch right
    // after a sort, whose loads go through the source index: measured slower
    // there with it).  A wavefront stays whole through the loop (the deposit's
    // queue needs every lane): `go` marks the lanes with a particle to push.
    constexpr bool kAhead = NT < 1024 || !GATHER;
    int celln = -1;
    float on[3] = {0.f, 0.f, 0.f}, un[3] = {0.f, 0.f, 0.f}, wn = 0.f;
    if (kAhead && (int)threadIdx.x < n) load_particle<GATHER>(s, src, pb + (int)threadIdx.x, celln, on, un, wn);
    const int q_first = __builtin_amdgcn_readfirstlane((int)threadIdx.x & ~63);
    for (int q0 = q_first; q0 < n; q0 += NT) {
        const int q = q0 + (int)__lane_id(), p = pb + q;
        bool go = q < n;
        if (!kAhead && go) load_particle<GATHER>(s, src, p, celln, on, un, wn);
        const int cell = celln;
        float o[3] = {on[0], on[1], on[2]};
        float u[3] = {un[0], un[1], un[2]};
        const float wq = s.mq * wn;
        if (kAhead && q + NT < n) load_particle<GATHER>(s, src, p + NT, celln, on, un, wn);
        int c[3] = {0, 0, 0}, lc[3] = {0, 0, 0}, di[3] = {0, 0, 0};
        if (go && (unsigned)cell >= (unsigned)g.ncell) {   // (a sort drops these)
            if (GATHER) s.cell[p] = cell;
            keep_particle<GATHER>(s, p, o, u);
            go = false;
        }
        if (go) {
            decompose(g, cell, c);
            if (particle_killed(g, c)) {
                s.cell[p] = -1;
                keep_particle<GATHER>(s, p, o, u);
                go = false;
            }
        }
        if (go) {
            bool inside = true;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                int l = c[d] - t0[d];
                if (l >= te[d] + guard) l -= g.n[d];
                if (l < -guard) l += g.n[d];
                lc[d] = l;
                inside = inside && l >= -guard && l < te[d] + guard;
            }
            if (!inside) {   // beyond the guard: the rest pass takes it
                s.cell[p] = -2 - cell;
                keep_particle<GATHER>(s, p, o, u);
                const unsigned long long m = __ballot(1);   // the lanes in this branch
                const int lane = __lane_id(), leader = __ffsll((long long)m) - 1;
                int base = 0;
                if (lane == leader) base = atomicAdd(rest_n, __popcll(m));
                base = __shfl(base, leader);
                rest_idx[base + __popcll(m & ((1ull << lane) - 1ull))] = p;
                go = false;
            }
        }
        if (go && cold_tile && (__float_as_uint(u[0]) | __float_as_uint(u[1]) | __float_as_uint(u[2])) == 0u) {
            if (GATHER) {   // the particle still moves to its sorted place
                s.cell[p] = cell;
                keep_particle<GATHER>(s, p, o, u);
            }
            go = false;
        }
        const float o0[3] = {o[0], o[1], o[2]};
        if (go) {
            GatherStencil st;
            gather_stencil(o, st);
            float E[3], B[3];
            {
                int ii[3][4], ih[3][4];
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        ii[d][a] = (lc[d] + H - 1 + a) * fstride[d];
                        ih[d][a] = (lc[d] + H + st.hb[d] + a) * fstride[d];
                    }
                gather_fields(El, Bl, ii, ih, st, E, B);
            }
            int c1[3] = {c[0], c[1], c[2]};
            errs |= push_move(g, s.qmh, E, B, u, o, c1);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                s.u[d][p] = u[d];
                s.off[d][p] = o[d];
                di[d] = unwrap_shift(c1[d] - c[d], g.n[d]);
            }
            s.cell[p] = c1[0] + g.n[0] * (c1[1] + g.n[1] * c1[2]);
            // a particle that did not move contributes zeros only
            if (moved(c, c1, o0, o)) dep.core(lc, di, o0, o, wq);
        }
        dep.cross(s, (di[0] | di[1] | di[2]) != 0, lc, di, o0, p);
    }
    dep.finish(s);
    if (errs) atomicOr(d_err, errs);
    __syncthreads();
    flush_current<NT>(g, t0, guard + 2, jx, jpl, jr, Jl, acc);
}

// WAVES: wavefronts per SIMD that the kernel leaves registers for (see tile_packed).
template <int NT, int WAVES, int TX = 0, int TY = 0, int TZ = 0, int GD = -1, bool GATHER = false>
__global__ void __launch_bounds__(NT, WAVES) k_pic_tile(Geom g, TileGeom t, int guard, FieldPtrs f, SpeciesDev s,
                                                 SpeciesDev src, const int* __restrict__ toff,
                                                 unsigned long long* __restrict__ acc, int* __restrict__ d_err,
                                                 int* __restrict__ rest_n, int* __restrict__ rest_idx) {
    extern __shared__ unsigned long long lds_u64[];
    const int tile = xcd_tile(blockIdx.x, t.ntiles, t.nt[0]);
    if (tile >= t.ntiles) return;
    tile_body<NT, TX, TY, TZ, GD, GATHER>(g, t, guard, f, s, src, toff, acc, d_err, rest_n, rest_idx, lds_u64, tile,
                                          blockIdx.y, gridDim.y);
}

// Batched form: the work list is the concatenation of every member's tiles
// (member m owns flat tiles [tile_begin[m], tile_begin[m+1])), mapped XCD by
// XCD like the single-instance launch.  TX..GD > 0 (>= 0): every member has
// that tile shape and guard (the compile-time body of the single launch).
template <int NT, int WAVES, int TX = 0, int TY = 0, int TZ = 0, int GD = -1>
__global__ void __launch_bounds__(NT, WAVES) k_batch_tile(const InstDesc* __restrict__ tab,
                                                   const int* __restrict__ tile_begin, int n, int total) {
    extern __shared__ unsigned long long lds_u64[];
    const int ft = xcd_tile(blockIdx.x, total, kBatchChunk);
    if (ft >= total) return;
    int lo = 0, hi = n - 1;   // last member whose range starts at or before ft
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tile_begin[mid] <= ft) lo = mid; else hi = mid - 1;
    }
    const InstDesc& d = tab[lo];
    const Geom g = d.g;
    const TileGeom t = d.t;
    const FieldPtrs f = d.f;
    const SpeciesDev s = step_arrays(d);
    // a member that sorted this step gathers its particles from the pre-sort set
    if (d.sorting)
        tile_body<NT, TX, TY, TZ, GD, true>(g, t, d.guard, f, s, d.s, d.toff, d.acc, d.err, d.rest_n, d.rank, lds_u64,
                                            ft - tile_begin[lo]);
    else
        tile_body<NT, TX, TY, TZ, GD>(g, t, d.guard, f, s, s, d.toff, d.acc, d.err, d.rest_n, d.rank, lds_u64,
                                      ft - tile_begin[lo]);
}

// Deposit of the split path, tile by tile.  The particles stay in the
// caller's memory order; `list` names each tile's particles by their old
// cells (so the LDS region needs no guard: 8x8x8 cells, 57 KB, two
// workgroups per CU).  A particle's 144-300 contributions go to LDS, and the
// tile's region to the global accumulator once: global 64-bit atomics, which
// bound the one-thread-per-particle form (k_deposit), drop from ~200 to ~3
// per particle at 4 particles per cell (75x50x44 cells, 6.6e5 particles of a
// warm plasma: 2880 us -> 119 with the index list; atomics and deposit
// arithmetic in LDS bound it now).  Moves of more than one cell, which the
// region does not hold, are added straight to the accumulator after the loop;
// kept out of it, they cost it no registers (162 with them, 128 for two
// workgroups per CU: staged step of two species 729 us against 711).
constexpr int kDepTile = 8, kDepThreads = 512;

// A tile of up to kWhole list entries (8 particles per cell) is one workgroup's.
// Of a larger one its own workgroup takes the first kWindow + 1 .. 2 kWindow,
// and one more workgroup per kWindow entries of the whole list takes those
// that start at its multiple of kWindow if their tile's own workgroup does not
// reach them: the tiles that hold a beam are shared by many workgroups.
// Smaller windows fill the chip for a smaller beam; splitting ordinary tiles
// stages their fields twice.  75x50x44 cells, 3.3e5 particles within some cells
// (normal, 1.5 cells): deposit 907 us with windows of 4096, 572 with 2048, 367
// with 1024; 64x64x64 cells, 6 per cell in level order: gather 140 us with whole
// tiles, 168 with them split at 2048.
constexpr int kWhole = 4608, kWindow = 1024;

struct TileWindow {
    int tile, begin, n;   // list entries [begin, begin + n) are particles of this tile
};

__device__ __forceinline__ bool tile_window(const TileGeom& t, const TileList& l, TileWindow& w) {
    const int* __restrict__ off = l.off;
    const int own = xcd_blocks(t.ntiles, t.nt[0]);
    // entries of a tile [a, e) from here on are not its own workgroup's
    auto reach = [](int a, int e) {
        return e - a <= kWhole ? (unsigned)e : min((unsigned)e, ((unsigned)a / kWindow + 2) * kWindow);
    };
    if ((int)blockIdx.x < own) {
        w.tile = xcd_tile(blockIdx.x, t.ntiles, t.nt[0]);
        if (w.tile >= t.ntiles) return false;
        w.begin = off[w.tile * t.tcells];
        w.n = (int)reach(w.begin, off[(w.tile + 1) * t.tcells]) - w.begin;
        return w.n > 0;
    }
    const int64_t begin = (int64_t)((int)blockIdx.x - own) * kWindow;
    if (begin >= off[t.ntiles * t.tcells]) return false;
    w.begin = (int)begin;
    // last tile that starts at or before the window, which holds the window's start (64 tiles compared at a time)
    int lo = 0, count = t.ntiles;
    while (count > 1) {
        const int step = (count + 63) / 64, k = (int)__lane_id() * step;
        const int last = 63 - __clzll(__ballot(k < count && off[(lo + k) * t.tcells] <= w.begin));
        lo += last * step;
        count = min(step, count - last * step);
    }
    const int a = off[lo * t.tcells], e = off[(lo + 1) * t.tcells];
    w.tile = lo;
    w.n = min(e - w.begin, kWindow);
    return (unsigned)w.begin >= reach(a, e);
}

static int list_blocks(const TileGeom& t, const TileList& l) {
    return xcd_blocks(t.ntiles, t.nt[0]) + l.max_count / kWindow + 1;
}

// More than one cell along some axis.
__device__ __forceinline__ bool far_move(const int di[3]) {
    return max(max(abs(di[0]), abs(di[1])), abs(di[2])) > 1;
}

__global__ void __launch_bounds__(kDepThreads, 4) k_deposit_tiles(Geom g, TileGeom t, SpeciesDev s, PrevDev prev,
                                                                  const TileList l,
                                                                  unsigned long long* __restrict__ acc) {
    constexpr int jx = kDepTile + 5, jpl = cur_plane(jx, jx), jr = jpl * jx;
    __shared__ unsigned long long Jl[3 * jr];
    TileWindow w;
    if (!tile_window(t, l, w)) return;
    const int n = w.n;
    const int tz = w.tile / (t.nt[0] * t.nt[1]);
    const int tr = w.tile - tz * t.nt[0] * t.nt[1];
    const int ty = tr / t.nt[0];
    const int t0[3] = {(tr - ty * t.nt[0]) * t.T[0], ty * t.T[1], tz * t.T[2]};
    for (int i = threadIdx.x; i < 3 * jr; i += kDepThreads) Jl[i] = 0ull;
    // A crowded tile's entries are in cell order: lane k takes the k-th of 64
    // runs of them, so that the lanes of an atomic are in different cells
    const bool crowded = crowded_tile(l.off + w.tile * t.tcells, t.tcells);   // (the barrier after the clearing)
    const int* __restrict__ list = (crowded ? l.plain : l.level) + w.begin;
    const int run = (n + 63) / 64, longer = n - 64 * (run - 1), lane = __lane_id();
    const int first = crowded ? (lane < longer ? lane * run : longer * run + (lane - longer) * (run - 1)) : 0;
    TileDeposit dep;
    dep.init(Jl, 0, jx, jpl, jr);
    bool far = false;
    const int q_first = __builtin_amdgcn_readfirstlane((int)threadIdx.x & ~63);
    for (int q0 = q_first; q0 < n; q0 += kDepThreads) {
        const int q = q0 + (int)__lane_id();
        int lc[3] = {0, 0, 0}, di[3] = {0, 0, 0};
        int p = 0;
        float o0[3] = {0.f, 0.f, 0.f}, o1[3] = {0.f, 0.f, 0.f}, wq = 0.f;
        if (q < n) {
            p = list[crowded ? first + (q0 >> 6) : q];
            const int cell0 = prev.cell[p], cell1 = s.cell[p];   // (cell0 is valid: it has a key)
            int c0[3], c1[3];
            decompose(g, cell0, c0);
            decompose(g, cell1, c1);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                o0[d] = prev.off[d][p];
                o1[d] = s.off[d][p];
            }
            wq = s.mq * s.w[p];
            if ((unsigned)cell1 < (unsigned)g.ncell && moved(c0, c1, o0, o1)) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    lc[d] = c0[d] - t0[d];
                    di[d] = unwrap_shift(c1[d] - c0[d], g.n[d]);
                }
                if (far_move(di)) {
                    far = true;
                    di[0] = di[1] = di[2] = 0;
                } else {
                    dep.core(lc, di, o0, o1, wq);
                }
            }
        }
        dep.cross(s, (di[0] | di[1] | di[2]) != 0, lc, di, o0, p);
    }
    dep.finish(s);
    // (a push moves a particle into a neighbouring cell at most; a caller may have
    // moved it further since)
    if (__syncthreads_or(far))
        for (int q = threadIdx.x; q < n; q += kDepThreads) {
            const int p = list[q], cell1 = s.cell[p];
            int c0[3], c1[3], di[3];
            decompose(g, prev.cell[p], c0);
            decompose(g, cell1, c1);
#pragma unroll
            for (int d = 0; d < 3; ++d) di[d] = unwrap_shift(c1[d] - c0[d], g.n[d]);
            if ((unsigned)cell1 >= (unsigned)g.ncell || !far_move(di)) continue;
            const float o0[3] = {prev.off[0][p], prev.off[1][p], prev.off[2][p]};
            const float o1[3] = {s.off[0][p], s.off[1][p], s.off[2][p]};
            deposit_global(g, c0, c1, o0, o1, s.mq * s.w[p], acc);
        }
    flush_current<kDepThreads>(g, t0, 2, jx, jpl, jr, Jl, acc);
}

// Gather and push of the split path, tile by tile as k_deposit_tiles (the
// list by the current cells): E and B of the tile and its two-cell halo in
// LDS (48 KB, three workgroups per CU).  The one-thread-per-particle form
// (k_gather_push) reads its 384 field values from global memory, where the
// particles' memory order decides how many lines a wavefront's load touches.
// 75x50x44 cells, 3.3e5 particles of a warm plasma: 205 -> 131 us with its
// list; the particles' scattered loads and stores bound it now.
__global__ void __launch_bounds__(kDepThreads) k_gather_tiles(Geom g, TileGeom t, FieldPtrs f, SpeciesDev s,
                                                              PrevDev prev, const TileList l,
                                                              int* __restrict__ d_err) {
    constexpr int fx = kDepTile + 4, fpl = field_plane(fx, fx), fr = fpl * fx;
    __shared__ float Fl[6 * fr];
    TileWindow w;
    if (!tile_window(t, l, w)) return;
    const int tz = w.tile / (t.nt[0] * t.nt[1]);
    const int tr = w.tile - tz * t.nt[0] * t.nt[1];
    const int ty = tr / t.nt[0];
    const int t0[3] = {(tr - ty * t.nt[0]) * t.T[0], ty * t.T[1], tz * t.T[2]};
    for (int i = threadIdx.x; i < fx * fx * fx; i += kDepThreads) {
        const int lz = i / (fx * fx), rr = i - lz * fx * fx, ly = rr / fx, lx = rr - ly * fx;
        const int gi = wrap_any(t0[0] - 2 + lx, g.n[0]) +
                       g.n[0] * (wrap_any(t0[1] - 2 + ly, g.n[1]) + g.n[1] * wrap_any(t0[2] - 2 + lz, g.n[2]));
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            Fl[c * fr + lz * fpl + rr] = f.E[c][gi];
            Fl[(3 + c) * fr + lz * fpl + rr] = f.B[c][gi];
        }
    }
    const bool crowded = crowded_tile(l.off + w.tile * t.tcells, t.tcells);   // (the barrier after the staging)
    const int* __restrict__ list = (crowded ? l.plain : l.level) + w.begin;
    float* const El[3] = {Fl, Fl + fr, Fl + 2 * fr};
    float* const Bl[3] = {Fl + 3 * fr, Fl + 4 * fr, Fl + 5 * fr};
    constexpr int fstride[3] = {1, fx, fpl};
    int errs = 0;
    for (int q = threadIdx.x; q < w.n; q += kDepThreads) {
        const int p = list[q], cell = s.cell[p];
        int c[3];
        decompose(g, cell, c);
        float o[3] = {s.off[0][p], s.off[1][p], s.off[2][p]};
        float u[3] = {s.u[0][p], s.u[1][p], s.u[2][p]};
        const bool killed = particle_killed(g, c);
        prev.cell[p] = killed ? -1 : cell;
#pragma unroll
        for (int d = 0; d < 3; ++d) prev.off[d][p] = o[d];
        if (killed) {
            s.cell[p] = -1;
            continue;
        }
        GatherStencil st;
        gather_stencil(o, st);
        int ii[3][4], ih[3][4];
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                ii[d][a] = (c[d] - t0[d] + 1 + a) * fstride[d];
                ih[d][a] = (c[d] - t0[d] + 2 + st.hb[d] + a) * fstride[d];
            }
        float E[3], B[3];
        gather_fields(El, Bl, ii, ih, st, E, B);
        errs |= push_move(g, s.qmh, E, B, u, o, c);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            s.u[d][p] = u[d];
            s.off[d][p] = o[d];
        }
        s.cell[p] = c[0] + g.n[0] * (c[1] + g.n[1] * c[2]);
    }
    if (errs) atomicOr(d_err, errs);
}

// Before it: the particles that are in no tile (removed ones; an index outside
// the grid is invalid input, removed and reported).
__global__ void __launch_bounds__(256) k_gather_invalid(int ncell, int* cell, int* prev_cell,
                                                        const int* __restrict__ d_count, int* __restrict__ d_err) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= *d_count) return;
    const int c = cell[p];
    if ((unsigned)c < (unsigned)ncell) return;
    if (c >= 0) {
        atomicOr(d_err, ERR_OVERFLOW);
        cell[p] = -1;
    }
    prev_cell[p] = c < 0 ? c : -1;
}

hipError_t launch_gather_invalid(const Geom& g, const SpeciesDev& s, const PrevDev& prev, const int* d_count,
                                 int max_count, int* d_err, hipStream_t st) {
    hipLaunchKernelGGL(k_gather_invalid, dim3((max_count + 255) / 256), dim3(256), 0, st, g.ncell, s.cell, prev.cell,
                       d_count, d_err);
    return hipGetLastError();
}

hipError_t launch_gather_tiles(const Geom& g, const TileGeom& t, const FieldPtrs& f, const SpeciesDev& s,
                               const PrevDev& prev, const TileList& l, int* d_err, hipStream_t st) {
    hipLaunchKernelGGL(k_gather_tiles, dim3(list_blocks(t, l)), dim3(kDepThreads), 0, st, g, t, f, s,
                       prev, l, d_err);
    return hipGetLastError();
}

TileGeom deposit_tiling(const int n[3]) {
    TileGeom t;
    for (int a = 0; a < 3; ++a) {
        t.T[a] = std::min(kDepTile, n[a]);
        t.nt[a] = (n[a] + t.T[a] - 1) / t.T[a];
    }
    t.ntiles = t.nt[0] * t.nt[1] * t.nt[2];
    t.tcells = t.T[0] * t.T[1] * t.T[2];
    return t;
}

hipError_t launch_deposit_tiles(const Geom& g, const TileGeom& t, const SpeciesDev& s, const PrevDev& prev,
                                const TileList& l, unsigned long long* acc, hipStream_t st) {
    hipLaunchKernelGGL(k_deposit_tiles, dim3(list_blocks(t, l)), dim3(kDepThreads), 0, st, g, t, s, prev,
                       l, acc);
    return hipGetLastError();
}

// The rest pass, after the tile kernel: the particles on the species' rest
// list (marked by the tile kernel with cell -2 - c) and those appended after
// the last sort (index >= sorted, in no tile range) take the same step
// through global memory.  Item i < n_rest is list entry i, item n_rest + j
// is particle sorted + j.
__device__ __forceinline__ void rest_item(const Geom& g, const FieldPtrs& f, const SpeciesDev& s, int i, int nrest,
                                          int sorted, const int* __restrict__ rest_idx,
                                          unsigned long long* acc, int* d_err) {
    int p, c[3];
    if (i < nrest) {
        p = rest_idx[i];
        decompose(g, -2 - s.cell[p], c);   // the tile kernel already applied the window cut
    } else {
        p = sorted + (i - nrest);
        const int cell = s.cell[p];
        if ((unsigned)cell >= (unsigned)g.ncell) return;
        decompose(g, cell, c);
        if (particle_killed(g, c)) {
            s.cell[p] = -1;
            return;
        }
    }
    const int errs = push_deposit_global(g, f, s, p, c, acc);
    if (errs) atomicOr(d_err, errs);
}

constexpr int kRestThreads = 256;

__global__ void __launch_bounds__(kRestThreads) k_tile_rest(Geom g, FieldPtrs f, SpeciesDev s,
                                                            const int* __restrict__ d_sorted,
                                                            const int* __restrict__ d_count,
                                                            const int* __restrict__ rest_n,
                                                            const int* __restrict__ rest_idx,
                                                            unsigned long long* __restrict__ acc,
                                                            int* __restrict__ d_err) {
    const int nrest = *rest_n, sorted = *d_sorted;
    const int total = nrest + max(0, *d_count - sorted);
    for (int i = blockIdx.x * kRestThreads + threadIdx.x; i < total; i += gridDim.x * kRestThreads)
        rest_item(g, f, s, i, nrest, sorted, rest_idx, acc, d_err);
}

__global__ void __launch_bounds__(kRestThreads) k_batch_rest(const InstDesc* __restrict__ tab) {
    const InstDesc& d = tab[blockIdx.y];
    const Geom g = d.g;
    const FieldPtrs f = d.f;
    const SpeciesDev s = step_arrays(d);
    const int nrest = *d.rest_n, sorted = *d.sorted;
    const int total = nrest + max(0, *d.count - sorted);
    for (int i = blockIdx.x * kRestThreads + threadIdx.x; i < total; i += gridDim.x * kRestThreads)
        rest_item(g, f, s, i, nrest, sorted, d.rank, d.acc, d.err);
}

// Empty the species' rest lists (a kernel, not a memset, so that a captured
// step stays valid).
__global__ void k_zero_rest(int* rest_n) { rest_n[threadIdx.x] = 0; }

__global__ void k_batch_zero_rest(const InstDesc* __restrict__ tab, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) *tab[i].rest_n = 0;
}

size_t tile_lds_bytes(const TileGeom& t, int guard) {
    const int H = guard + 2;
    const size_t fr = (size_t)field_plane(t.T[0] + 2 * H, t.T[1] + 2 * H) * (t.T[2] + 2 * H);
    const size_t jr = (size_t)cur_plane(t.T[0] + 2 * guard + 5, t.T[1] + 2 * guard + 5) * (t.T[2] + 2 * guard + 5);
    return 3 * jr * 8 + 6 * fr * 4;
}

// Tiles so small that more than two wavefronts per SIMD fit by their LDS take
// the general body in 128 registers, four wavefronts per SIMD; in larger
// ones, one workgroup per CU, that limit would only spill.  Measured, two steps
// of 64x64x64 cells, 2.1e6 particles of a warm plasma, 4x4x4 tiles (61 KB), 512
// threads: 812 us, 1118 with the 172 registers it takes otherwise (one
// workgroup per CU); batch of 3 96x64x64 members, 8x8x4 tiles (109 KB), 512
// threads: 3957 us without the limit, 4093 with it.
static bool tile_packed(int threads, size_t lds) { return (int)(kLdsBytes / lds) * threads / 256 > 2; }

// Threads per workgroup where the caller leaves them to the library (0).
// 1024: also where a share holds few particles, the staging, clearing and flush
// of the tile's LDS gain from them (12 tiles of 1050 particles in four parts: 72
// us a step, 73 with 512, 84 with 256; 7200 tiles of 4096: 4.60 ms per two
// steps, 5.05 with 512, 7.5 with 256).  512 where two workgroups fit a CU by
// their LDS, whose phases then overlap (the 4x4x4 tiles above: 812 us, 1103 with
// 1024, 939 with 256; as a batch of 3 96x64x64: 4.45 ms, 6.67, 5.39).
static int tile_threads(int threads, size_t lds) { return threads > 0 ? threads : (2 * lds <= kLdsBytes ? 512 : 1024); }

// One tile launch: parts workgroups of NT threads per tile.
struct TileLaunch {
    const Geom& g;
    const TileGeom& t;
    int guard, parts;
    const FieldPtrs& f;
    const SpeciesDev& s;
    const SpeciesDev* src;
    const int* toff;
    unsigned long long* acc;
    int *d_err, *rest_n, *rest_idx;
    hipStream_t st;
};

template <int NT, int WAVES, int TX, int TY, int TZ, int GD, bool GATHER>
static hipError_t launch_tile_k(const TileLaunch& L) {
    const size_t lds = tile_lds_bytes(L.t, L.guard);
    const int nb = xcd_blocks(L.t.ntiles, L.t.nt[0]);
    hipError_t e = hipFuncSetAttribute((const void*)k_pic_tile<NT, WAVES, TX, TY, TZ, GD, GATHER>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_pic_tile<NT, WAVES, TX, TY, TZ, GD, GATHER>), dim3(nb, L.parts), dim3(NT), lds, L.st, L.g, L.t,
                       L.guard, L.f, L.s, GATHER ? *L.src : L.s, L.toff, L.acc, L.d_err, L.rest_n, L.rest_idx);
    return hipGetLastError();
}

template <int NT, int WAVES, int TX = 0, int TY = 0, int TZ = 0, int GD = -1>
static hipError_t launch_tile_nt(const TileLaunch& L) {
    if (L.src) return launch_tile_k<NT, WAVES, TX, TY, TZ, GD, true>(L);
    return launch_tile_k<NT, WAVES, TX, TY, TZ, GD, false>(L);
}

// Tile shapes with a compile-time specialisation (the library default and
// the autotuner's usual picks); every other shape runs the general body.
template <int NT>
static hipError_t launch_tile_shape(const TileLaunch& L) {
    const int* T = L.t.T;
    constexpr int W = NT / 256;
    if (T[0] == 8 && T[1] == 8 && T[2] == 8) {
        if (L.guard == 1) return launch_tile_nt<NT, W, 8, 8, 8, 1>(L);
        if (L.guard == 0) return launch_tile_nt<NT, W, 8, 8, 8, 0>(L);
    }
    if (T[0] == 8 && T[1] == 8 && T[2] == 4 && L.guard == 1) return launch_tile_nt<NT, W, 8, 8, 4, 1>(L);
    if (tile_packed(NT, tile_lds_bytes(L.t, L.guard))) return launch_tile_nt<NT, 4>(L);
    return launch_tile_nt<NT, W>(L);
}

// Workgroups that share a tile.  A tile's LDS leaves room for one or two
// workgroups per CU, so a grid of fewer tiles than CUs shares each tile's
// particles between workgroups (each stages the fields and adds its own
// current: sums are integers, so J is the same), as long as each gets kPartMin
// particles on average.  Measured, 128 tiles of 4096 particles: 113 us per launch
// with one part, 67 with two; 12 tiles of 1050: 48 us, 21 with four.
constexpr int kCUs = 256, kPartMin = 256;

static int tile_parts(int ntiles, int64_t count) {
    const int64_t fill = kCUs / ntiles, most = count / ((int64_t)ntiles * kPartMin);
    return (int)std::max<int64_t>(1, std::min(fill, most));
}

hipError_t launch_pic_tile(const Geom& g, const TileGeom& t, int guard, int threads, int max_count,
                           const FieldPtrs& f, const SpeciesDev& s, const SpeciesDev* src, const int* toff,
                           unsigned long long* acc, int* d_err, int* rest_n, int* rest_idx, hipStream_t st) {
    const int parts = tile_parts(t.ntiles, max_count);
    const TileLaunch L{g, t, guard, parts, f, s, src, toff, acc, d_err, rest_n, rest_idx, st};
    switch (tile_threads(threads, tile_lds_bytes(t, guard))) {
        case 256: return launch_tile_shape<256>(L);
        case 1024: return launch_tile_shape<1024>(L);
        default: return launch_tile_shape<512>(L);
    }
}

template <int NT, int WAVES, int TX = 0, int TY = 0, int TZ = 0, int GD = -1>
static hipError_t launch_batch_tile_k(const InstDesc* d, const int* tile_begin, int n, int total, size_t lds,
                                      hipStream_t st) {
    const int nb = xcd_blocks(total, kBatchChunk);
    hipError_t e = hipFuncSetAttribute((const void*)k_batch_tile<NT, WAVES, TX, TY, TZ, GD>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_batch_zero_rest, dim3((n + 63) / 64), dim3(64), 0, st, d, n);
    hipLaunchKernelGGL((k_batch_tile<NT, WAVES, TX, TY, TZ, GD>), dim3(nb), dim3(NT), lds, st, d, tile_begin, n, total);
    return hipGetLastError();
}

template <int NT>
static hipError_t launch_batch_tile_nt(const InstDesc* d, const int* tile_begin, int n, int total, size_t lds,
                                       bool all_888g1, hipStream_t st) {
    constexpr int W = NT / 256;
    if (all_888g1) return launch_batch_tile_k<NT, W, 8, 8, 8, 1>(d, tile_begin, n, total, lds, st);
    if (tile_packed(NT, lds)) return launch_batch_tile_k<NT, 4>(d, tile_begin, n, total, lds, st);
    return launch_batch_tile_k<NT, W>(d, tile_begin, n, total, lds, st);
}

hipError_t launch_batch_tile(const InstDesc* d, const int* tile_begin, int n, int total_tiles, int threads,
                             size_t lds_bytes, bool all_888g1, hipStream_t st) {
    if (n <= 0 || total_tiles <= 0) return hipSuccess;
    switch (tile_threads(threads, lds_bytes)) {
        case 256: return launch_batch_tile_nt<256>(d, tile_begin, n, total_tiles, lds_bytes, all_888g1, st);
        case 1024: return launch_batch_tile_nt<1024>(d, tile_begin, n, total_tiles, lds_bytes, all_888g1, st);
        default: return launch_batch_tile_nt<512>(d, tile_begin, n, total_tiles, lds_bytes, all_888g1, st);
    }
}

// Rest pass grids: a fixed number of blocks walking the items (list entries
// plus appended particles, a small share of the species in a step).
hipError_t launch_batch_rest(const InstDesc* d, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_rest, dim3(std::max(1, 1024 / n), n), dim3(kRestThreads), 0, st, d);
    return hipGetLastError();
}

hipError_t launch_zero_rest(int* rest_n, int n, hipStream_t st) {
    hipLaunchKernelGGL(k_zero_rest, dim3(1), dim3(n), 0, st, rest_n);
    return hipGetLastError();
}

hipError_t launch_tile_rest(const Geom& g, const FieldPtrs& f, const SpeciesDev& s, const int* d_sorted,
                            const int* d_count, const int* rest_n, const int* rest_idx, unsigned long long* acc,
                            int* d_err, bool few, hipStream_t st) {
    hipLaunchKernelGGL(k_tile_rest, dim3(few ? 64 : 1024), dim3(kRestThreads), 0, st, g, f, s, d_sorted, d_count,
                       rest_n, rest_idx, acc, d_err);
    return hipGetLastError();
}

}  // namespace pic
