// Learned current denoiser: the convolution layers of the network described
// in pic_dn_common.h and its output stage J' = B(J + sigma curl(y)).
// Inference runs layers 1, 2 (relu epilogues) and 3 (y), then the output
// stage; training reuses the same layer shapes for the gradient of the loss
// with respect to the activations (a transposed convolution is a
// convolution with the taps mirrored and the channel roles swapped) with a
// relu-mask epilogue, and the output stage with the loss.
#include <algorithm>

#include "pic_dn_common.h"

namespace pic {

// 32 output channels: EPI 0 = bf16 relu(acc + bias), 1 = bf16 acc where the
// mask activation is > 0.  The weights are the first operand of the MFMAs, so
// that lane (m, q) = (l & 15, l >> 4) holds channels 8 q + 4 h + j (dn_co) of
// cell m of each row block: 16 consecutive bytes of one cell, stored straight
// from the registers, four lanes to a cell's 64 bytes (the mask is read the
// same way).  Staging the output tile through LDS instead, with its two
// barriers and 32 two-byte stores per lane, took 336 us for layer 1 on
// 384x192x160 cells; this takes 307.
template <int EPI>
__device__ __forceinline__ void dn_store32(const DnArgs& a, const int t0[3], const f32x4 acc[4][2],
                                           const float bias[2][4]) {
    const int l = threadIdx.x & 63, lz = threadIdx.x >> 6;
    const int m = l & 15, q = l >> 4;
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
        const int cell = dn_out_cell(a, t0, lz, blk, m);
        if (cell < 0) continue;
        bf16x8 v;
        if (EPI == 0) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j) v[4 * h + j] = (__bf16)fmaxf(acc[blk][h][j] + bias[h][j], 0.0f);
        } else {
            const bf16x8 mk = reinterpret_cast<const bf16x8*>(a.mask)[(size_t)cell * 4 + q];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[4 * h + j] = (float)mk[4 * h + j] > 0.0f ? (__bf16)acc[blk][h][j] : (__bf16)0.0f;
        }
        reinterpret_cast<bf16x8*>(a.act_out)[(size_t)cell * 4 + q] = v;
    }
}

// The biases of this lane's channels (see dn_store32).
__device__ __forceinline__ void dn_bias32(const float* __restrict__ bias, float b[2][4]) {
    const int q = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 4; ++j) b[h][j] = bias[8 * q + 4 * h + j];
}

// 4-channel input (3 used), 32 output channels.  K = tap * 4 + channel
// (channel 3 and taps 27..31 zero), 4 K-steps of 32; lane chunk q of step s
// covers taps 8s + 2q and 8s + 2q + 1.  IN 0: the current J_d / s_d (FP32,
// rounded to bf16 here; a.Jcopy, if given, takes the current as it is); IN 1:
// a bf16 [cell][4] array.
template <int IN, int EPI>
__global__ void __launch_bounds__(DN_THREADS) k_dn_c4(DnArgs a) {
    constexpr int WROW = 272;              // bytes of a weight row (256, padded: 16 rows in different banks)
    __shared__ __attribute__((aligned(16))) char lds[DN_HCELLS * 8 + 32 * WROW];
    char* xin = lds;                       // [halo cell][4] bf16
    char* wl = lds + DN_HCELLS * 8;        // [co][128] bf16
    const int3 tile = dn_walk();
    const int t0[3] = {tile.x * DN_TX, tile.y * DN_TY, tile.z * DN_TZ};
    {
        const uint4* src = reinterpret_cast<const uint4*>(a.w);
        for (int g = threadIdx.x; g < 32 * 16; g += DN_THREADS)
            *reinterpret_cast<uint4*>(wl + (g >> 4) * WROW + (g & 15) * 16) = src[g];
    }
    {
        // a thread takes one (x, y) of the halo in planes pz, pz + 4, pz + 8
        // (as DnLane: only the plane changes between its loads); every global
        // load first, then the LDS stores
        constexpr int PL = DN_HX * DN_HY, PER = (DN_HZ + 3) / 4;
        static_assert(4 * PL <= DN_THREADS, "four planes at a time");
        const int pz = threadIdx.x / PL, c = threadIdx.x % PL, hx = c % DN_HX, hy = c / DN_HX;
        const int x = t0[0] - 1 + hx, y = t0[1] - 1 + hy;
        const int xs = dn_axis(x, a.n[0], a.bc[0], a.origin), ys = dn_axis(y, a.n[1], a.bc[1], 0);
        const bool in = pz < 4 && hx < DN_TX + 2 && xs >= 0 && ys >= 0;
        const bool own = IN == 0 && a.Jcopy[0] && in && hx >= 1 && hx <= DN_TX && hy >= 1 && hy <= DN_TY &&
                         x < a.n[0] && y < a.n[1];
        const int at = xs + a.n[0] * ys;
        float j[IN == 0 ? PER : 1][3];
        bf16x4 v[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int hz = pz + 4 * k, z = dn_axis(t0[2] - 1 + hz, a.n[2], a.bc[2], 0);
            const bool ok = in && hz < DN_HZ && z >= 0;
            const int s = ok ? at + a.n[0] * a.n[1] * z : 0;
            if constexpr (IN == 0) {
#pragma unroll
                for (int d = 0; d < 3; ++d) j[k][d] = ok ? a.J[d][s] : 0.0f;
            } else {
                v[k] = bf16x4{(__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f};
                if (ok) v[k] = reinterpret_cast<const bf16x4*>(a.c4_in)[s];
            }
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int hz = pz + 4 * k, z = t0[2] - 1 + hz;
            if constexpr (IN == 0) {
#pragma unroll
                for (int d = 0; d < 3; ++d) v[k][d] = (__bf16)(j[k][d] * a.inv_scale[d]);
                v[k][3] = (__bf16)0.0f;
                if (own && hz >= 1 && hz <= DN_TZ && z < a.n[2])
#pragma unroll
                    for (int d = 0; d < 3; ++d) a.Jcopy[d][at + a.n[0] * a.n[1] * z] = j[k][d];
            }
            if (pz < 4 && hz < DN_HZ) *reinterpret_cast<bf16x4*>(xin + (hz * PL + c) * 8) = v[k];
        }
    }
    __syncthreads();
    const int l = threadIdx.x & 63, lz = threadIdx.x >> 6;
    const int m = l & 15, q = l >> 4;
    float bias[2][4] = {};
    if (EPI == 0) dn_bias32(a.bias, bias);
    f32x4 acc[4][2];
#pragma unroll
    for (int blk = 0; blk < 4; ++blk)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[blk][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        bf16x8 B[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            B[h] = *reinterpret_cast<const bf16x8*>(wl + dn_co(m, h) * WROW + s * 64 + q * 16);
        const int ta = 8 * s + 2 * q;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk) {
            bf16x8 A;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int tap = ta + half;
                bf16x4 v = {(__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f, (__bf16)0.0f};
                if (tap < 27) {
                    const int dz = tap / 9, dy = (tap / 3) % 3, dx = tap % 3;
                    const int c = ((lz + dz) * DN_HY + (blk + dy)) * DN_HX + (m + dx);
                    v = *reinterpret_cast<const bf16x4*>(xin + c * 8);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) A[half * 4 + e] = v[e];
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
                acc[blk][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B[h], A, acc[blk][h], 0, 0, 0);
        }
    }
    dn_store32<EPI>(a, t0, acc, bias);
}

// Layers with a 32-channel input and output (KIND 0: relu(acc + b), 1: mask
// epilogue).  Persistent: one workgroup per compute unit walks its tiles; the
// next tile's input halo is loaded into registers while the current tile's
// matrix work runs.  A wavefront takes 16 of the output channels and two
// planes, with its weights (27 operands) in registers for the whole walk: 72
// LDS reads for 216 matrix instructions, where one plane, 32 channels and the
// weights in LDS took 108.  384x192x160 cells: 746 -> 663 us (980 TFLOP/s,
// the clock falling to 1.7 GHz under the matrix load; a large matrix product
// reaches 1184), of which half is the halo's addresses (DnLane, and planes
// inside the box by addition) and the order of stores and waits.
template <int KIND>
__global__ void __launch_bounds__(DN_THREADS) k_dn_conv32(DnArgs a) {
    extern __shared__ __attribute__((aligned(16))) char act[];
    const int m = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
    const int h = (__builtin_amdgcn_readfirstlane(threadIdx.x) >> 6) & 1;
    const int lz = (__builtin_amdgcn_readfirstlane(threadIdx.x) >> 7) * 2;
    int ntx, nty;
    const int ntiles = dn_ntiles(a.n, &ntx, &nty);
    bf16x8 W[27];
#pragma unroll
    for (int t = 0; t < 27; ++t) W[t] = reinterpret_cast<const bf16x8*>(a.w)[(t * 32 + 16 * h + m) * 4 + q];
    // XCD-aware walk (workgroups go round-robin over the 8 XCDs): the
    // workgroups of one XCD share a contiguous range of tiles and walk it
    // together, so the halos they share stay in that XCD's L2
    int tile, stride, end;
    if (gridDim.x % 8 == 0) {
        const int per = (ntiles + 7) / 8, k = blockIdx.x % 8;
        tile = k * per + blockIdx.x / 8;
        stride = gridDim.x / 8;
        end = min(ntiles, (k + 1) * per);
    } else {
        tile = blockIdx.x;
        stride = gridDim.x;
        end = ntiles;
    }
    int t0[3];
    const DnLane lane = dn_lane();
    const DnBox box = dn_box(a);
    float bias[4] = {};
    if (KIND == 0)
#pragma unroll
        for (int j = 0; j < 4; ++j) bias[j] = a.bias[16 * h + 4 * q + j];
    uint4 v[DN_ACT_PER];
    bf16x4 mk[2][4] = {};
    f32x4 acc[2][4];
    int cur[3] = {0, 0, 0};
    // f(p, r, byte offset of the row, of the lane's 4 channels in it) for the tile's output rows (p, r) inside the box
    const size_t rstep = (size_t)a.n[0] * 64, pstep = rstep * a.n[1];
    auto rows = [&](auto&& f) {
        const int x = cur[0] + m;
        if (x >= a.n[0]) return;
        const size_t at = (size_t)dn_axis_sel(x, a.n[0], a.bc[0], a.origin) * 64 + (4 * h + q) * 8;
        const size_t base = rstep * cur[1] + pstep * (cur[2] + lz);
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (cur[1] + r < a.n[1] && cur[2] + lz + p < a.n[2]) f(p, r, base + r * rstep + p * pstep, at);
    };
    bool have = false;
    unsigned out = 0;
    if (tile >= end) return;
    dn_tile_of(tile, ntx, nty, t0);
    out = dn_load_act(a.act_in, box, t0, lane, v);
    // The last tile's outputs are stored after the next halo has been taken
    // from the registers: the wait for the loads would wait for stores issued
    // in between as well (one counter).  After the last tile v holds nothing
    // new, and the halo stored is not read.
    for (;;) {
        __syncthreads();   // the previous tile's LDS reads are done (first pass: nothing)
        dn_zero_planes(v, out);
        dn_store_act(v, lane, act);
        if (have) {
            rows([&](int p, int r, size_t row, size_t at) {
                bf16x4 o;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    o[j] = KIND == 0 ? (__bf16)fmaxf(acc[p][r][j] + bias[j], 0.0f)
                                     : ((float)mk[p][r][j] > 0.0f ? (__bf16)acc[p][r][j] : (__bf16)0.0f);
                *reinterpret_cast<bf16x4*>(reinterpret_cast<char*>(a.act_out) + row + at) = o;
            });
        }
        if (tile >= end) return;
        __syncthreads();   // halo staged
#pragma unroll
        for (int d = 0; d < 3; ++d) cur[d] = t0[d];
        if (KIND == 1)
            rows([&](int p, int r, size_t row, size_t at) {
                mk[p][r] = *reinterpret_cast<const bf16x4*>(reinterpret_cast<const char*>(a.mask) + row + at);
            });
        tile += stride;
        if (tile < end) {
            dn_tile_of(tile, ntx, nty, t0);
            out = dn_load_act(a.act_in, box, t0, lane, v);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[p][r] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        dn_mma32(act, W, acc);
        have = true;
    }
}

// The 32 -> 3 layer, y = conv(a2, W3) + b3 as FP32 components into a.Jout.
// A row of 16 cells x 32 channels is 1 KB of HBM in exactly the order of an
// MFMA's second operand, so no LDS is needed: a wavefront takes 16 columns
// and 4 rows and marches along z, each input plane's 6 rows loaded once into
// registers, two planes ahead.  The first operand holds the weights of one
// (dz, dy): row 4 dx + c for x-tap dx and channel c, 9 operands in registers
// for the whole march.  The x-taps' partial sums lie in three lane groups,
// one column apart, and are added with two lane exchanges per value at the
// end: 14 of the 16 columns are outputs.  Bound by the loads (64 B read, 12
// written per cell, halos included 1.9 times that from L2).  On 384x192x160
// cells this takes 266 us; 16x4x8 tiles in LDS, every row read once per x-tap
// and the weights by every wavefront, took 588, and a single plane ahead,
// moved between buffers, 371 (the moves wait for the loads).
constexpr int L3_X = 14, L3_Y = 4, L3_WAVES = 4;

__global__ void __launch_bounds__(64 * L3_WAVES, 2) k_dn_l3(DnArgs a, int zrun) {
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = l & 15, q = l >> 4;
    const int3 t = dn_walk();
    const int x0 = t.x * L3_X, y0 = (t.y * L3_WAVES + w) * L3_Y, z0 = t.z * zrun;
    if (y0 >= a.n[1]) return;
    const int z1 = min(z0 + zrun, a.n[2]);
    bf16x8 W[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) W[k] = reinterpret_cast<const bf16x8*>(a.w)[(k * 16 + m) * 4 + q];
    const float b[3] = {a.bias[0], a.bias[1], a.bias[2]};
    // column m is window cell x0 - 1 + m (past the right edge of the box: not needed)
    const int xw = x0 - 1 + m;
    const int xs = xw <= a.n[0] ? dn_axis_sel(xw, a.n[0], a.bc[0], a.origin) : -1;
    // a column outside the box loads some cell of its row; its partial sums are dropped below
    const size_t lane = (size_t)(xs >= 0 ? xs : min(m, a.n[0] - 1)) * 64 + q * 16;
    const bool ok0 = __shfl(xs, (m + 15) & 15, 64) >= 0, ok2 = __shfl(xs, (m + 1) & 15, 64) >= 0;
    int row[L3_Y + 2];   // storage row of y0 - 1 + r, or -1
#pragma unroll
    for (int r = 0; r < L3_Y + 2; ++r) {
        const int y = y0 - 1 + r;
        row[r] = y <= a.n[1] ? dn_axis_sel(y, a.n[1], a.bc[1], 0) : -1;
    }
    auto load = [&](int z, bf16x8 (&P)[L3_Y + 2]) {
        const int zs = dn_axis_sel(z, a.n[2], a.bc[2], 0);
#pragma unroll
        for (int r = 0; r < L3_Y + 2; ++r) {
            const char* p = reinterpret_cast<const char*>(a.act_in) +
                            (size_t)a.n[0] * 64 * ((size_t)max(row[r], 0) + (size_t)a.n[1] * max(zs, 0));
            P[r] = *reinterpret_cast<const bf16x8*>(p + lane);
        }
        if (zs < 0 || row[0] < 0 || row[L3_Y + 1] < 0) {   // a row outside an open box
#pragma unroll
            for (int r = 0; r < L3_Y + 2; ++r)
                if (zs < 0 || row[r] < 0) P[r] = __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
        }
    };
    const int from0 = ((m + 15) & 15) << 2, from2 = (32 + ((m + 1) & 15)) << 2;   // lanes of dx = 0, 2
    const bool mine = q == 1 && m >= 1 && m <= L3_X && xw < a.n[0];
    using Plane = bf16x8[L3_Y + 2];
    // plane z of the output from the input planes z - 1 .. z + 1, with the load of z + 3 started first
    auto plane = [&](int z, const Plane& A, const Plane& B, const Plane& C, Plane& N) {
        if (z + 2 < z1) load(z + 3, N);
        f32x4 acc[L3_Y];
#pragma unroll
        for (int r = 0; r < L3_Y; ++r) acc[r] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int r = 0; r < L3_Y; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        W[dz * 3 + dy], dz == 0 ? A[r + dy] : (dz == 1 ? B[r + dy] : C[r + dy]), acc[r], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < L3_Y; ++r) {
            float o[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const float v0 = __int_as_float(__builtin_amdgcn_ds_bpermute(from0, __float_as_int(acc[r][j])));
                const float v2 = __int_as_float(__builtin_amdgcn_ds_bpermute(from2, __float_as_int(acc[r][j])));
                o[j] = (((ok0 ? v0 : 0.0f) + acc[r][j]) + (ok2 ? v2 : 0.0f)) + b[j];
            }
            if (y0 + r < a.n[1]) {
                const size_t c0 = (size_t)a.n[0] * (row[r + 1] + (size_t)a.n[1] * z);
                if (mine)
#pragma unroll
                    for (int j = 0; j < 3; ++j) (a.Jout[j] + c0)[(unsigned)xs] = o[j];
            }
        }
    };
    Plane P0, P1, P2, P3, P4;
    load(z0 - 1, P0);
    load(z0, P1);
    load(z0 + 1, P2);
    if (z0 + 1 < z1) load(z0 + 2, P3);
    // five buffers take turns (no register moves): two planes' loads stay in flight
    for (int z = z0;; ++z) {
        plane(z, P0, P1, P2, P4);
        if (++z >= z1) return;
        plane(z, P1, P2, P3, P0);
        if (++z >= z1) return;
        plane(z, P2, P3, P4, P1);
        if (++z >= z1) return;
        plane(z, P3, P4, P0, P2);
        if (++z >= z1) return;
        plane(z, P4, P0, P1, P3);
        if (z + 1 >= z1) return;
    }
}

// The 32 -> 3 layer for training: every output is one chain of sums over the
// taps (dz, dx, dy), as gradients have been computed so far.  (k_dn_l3 adds
// the x-taps' sums at the end, which moves y by 1e-7; the loss gradient is
// rounded to bf16, where that shows as up to 3e-5 in the weight gradients of a
// small crop.)  Row 4 blk + c (c < 3) of one MFMA holds output channel c of
// row block blk: halo row r of a tap column (dz, dx) is multiplied by the
// operand (zx, r) whose row (blk, c) carries the weight of tap (dz, r - blk,
// dx), zero where r - blk is not a tap.  Persistent, as k_dn_conv32; weights
// and halo in LDS (152 KB).
constexpr int L3T_ROWS = 9 * DN_HY * 16;   // packed weight rows of 64 B

__global__ void __launch_bounds__(DN_THREADS) k_dn_l3_train(DnArgs a) {
    extern __shared__ __attribute__((aligned(16))) char act[];
    char* wl = act + DN_ACT_LDS;
    // 16-byte chunks of a weight row rotated so that 16 rows spread over the banks
    auto chunk = [](int r, int c) { return r * 64 + (((c + (((r >> 1) ^ (r >> 2)) & 3)) & 3) << 4); };
    for (int g = threadIdx.x; g < L3T_ROWS * 4; g += DN_THREADS)
        *reinterpret_cast<uint4*>(wl + chunk(g >> 2, g & 3)) = reinterpret_cast<const uint4*>(a.w)[g];
    int ntx, nty;
    const int ntiles = dn_ntiles(a.n, &ntx, &nty);
    int tile, stride, end;   // (the walk of k_dn_conv32)
    if (gridDim.x % 8 == 0) {
        const int per = (ntiles + 7) / 8, k = blockIdx.x % 8;
        tile = k * per + blockIdx.x / 8;
        stride = gridDim.x / 8;
        end = min(ntiles, (k + 1) * per);
    } else {
        tile = blockIdx.x;
        stride = gridDim.x;
        end = ntiles;
    }
    if (tile >= end) return;
    const DnLane lane = dn_lane();
    const DnBox box = dn_box(a);
    const float b[3] = {a.bias[0], a.bias[1], a.bias[2]};
    const int l = threadIdx.x & 63, lz = threadIdx.x >> 6, m = l & 15, q = l >> 4;
    const char* abase = act + (lz * DN_HY * DN_HX + m) * DN_ROWB + q * 16;
    const char* wbase = wl + chunk(m, q);
    uint4 v[DN_ACT_PER];
    int t0[3];
    dn_tile_of(tile, ntx, nty, t0);
    unsigned out = dn_load_act(a.act_in, box, t0, lane, v);
    while (tile < end) {
        __syncthreads();   // the previous tile's LDS reads are done (first pass: nothing)
        dn_zero_planes(v, out);
        dn_store_act(v, lane, act);
        __syncthreads();   // halo (and, first pass, weights) staged
        const int cur[3] = {t0[0], t0[1], t0[2]};
        tile += stride;
        if (tile < end) {
            dn_tile_of(tile, ntx, nty, t0);
            out = dn_load_act(a.act_in, box, t0, lane, v);
        }
        f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int zx = 0; zx < 9; ++zx)
#pragma unroll
            for (int r = 0; r < DN_HY; ++r) {
                const bf16x8 A =
                    *reinterpret_cast<const bf16x8*>(abase + ((zx / 3 * DN_HY + r) * DN_HX + zx % 3) * DN_ROWB);
                const bf16x8 B = *reinterpret_cast<const bf16x8*>(wbase + (zx * DN_HY + r) * 1024);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B, A, acc, 0, 0, 0);
            }
        const int cell = dn_out_cell(a, cur, lz, q, m);   // lane (m, q): cell m of row block q
        if (cell >= 0)
#pragma unroll
            for (int j = 0; j < 3; ++j) a.Jout[j][cell] = acc[j] + b[j];
    }
}

__device__ __forceinline__ float dn_at(const float* __restrict__ F, int s) { return s >= 0 ? F[s] : 0.0f; }

constexpr int DO_TX = 32, DO_TY = 8, DO_TZ = 4, DO_THREADS = DO_TX * DO_TY * DO_TZ;   // (adjoint stage)

__device__ __forceinline__ int do_src(const DnCombine& c, int x, int y, int z) {
    const int sx = dn_axis(x, c.n[0], c.bc[0], c.origin);
    const int sy = dn_axis(y, c.n[1], c.bc[1], 0);
    const int sz = dn_axis(z, c.n[2], c.bc[2], 0);
    if (sx < 0 || sy < 0 || sz < 0) return -1;
    return sx + c.n[0] * (sy + c.n[1] * sz);
}

// Binomial filter (27-point product stencil, x innermost) of an LDS region of
// rows SX and planes SX x SY, at the cells (lx .. lx + 2, ly .. , lz ..).
template <int SX, int SY>
__device__ __forceinline__ float do_binomial(const float* F, int lx, int ly, int lz) {
    const float w[3] = {0.25f, 0.5f, 0.25f};
    float acc = 0.0f;
#pragma unroll
    for (int zc = 0; zc < 3; ++zc) {
        float ay = 0.0f;
#pragma unroll
        for (int yb = 0; yb < 3; ++yb) {
            float ax = 0.0f;
            const int row = ((lz + zc) * SY + (ly + yb)) * SX + lx;
#pragma unroll
            for (int xa = 0; xa < 3; ++xa) ax = fmaf(w[xa], F[row + xa], ax);
            ay = fmaf(w[yb], ax, ay);
        }
        acc = fmaf(w[zc], ay, acc);
    }
    return acc;
}

// Output stage J' = B(t), t = J + sigma curl(y), curl(y)_a =
// (y_{a+2} - y_{a+2}[-e_{a+1}]) / d_{a+1} - (y_{a+1} - y_{a+1}[-e_{a+2}]) / d_{a+2},
// t zero outside the box.  A workgroup takes a column of 29 x 13 cells and
// marches along z: a thread owns one (x, y) of the column with the halo that
// the stencils need (2 below, 1 above: 32 x 16) and keeps the planes below in
// registers; neighbours along x come from the next lane, along y from LDS, one
// barrier per plane (the y planes are stored one ahead, both in two buffers).
// The loads of a plane are in flight for one (y) or two (J) planes.  LOSS: J' is
// compared with the target (one FP64 atomic per workgroup) and dst takes the
// loss gradient.  Tiles of 32x8x4 with the 27-point filter taken from LDS
// needed 532 vector instructions a cell: 384x192x160 cells 215 -> 125 us (HBM: 425 MB, 87 us at the copy rate).
constexpr int OM_X = 32, OM_Y = 16, OM_TX = OM_X - 3, OM_TY = OM_Y - 3, OM_THREADS = OM_X * OM_Y;

// Value of lane - 1 / lane + 1 (the lanes at a row's ends take part in no output).
__device__ __forceinline__ float lane_below(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, false));   // wave_shr:1
}
__device__ __forceinline__ float lane_above(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, false));   // wave_shl:1
}

template <bool LOSS>
__global__ void __launch_bounds__(OM_THREADS, 6) k_dn_output(DnCombine c, int zrun) {
    __shared__ float ysh[2][2][OM_THREADS];   // y_x, y_z
    __shared__ float xsh[2][3][OM_THREADS];   // x-filtered t
    const int3 tile = dn_walk();
    const int i = threadIdx.x, hx = i % OM_X, hy = i / OM_X;
    const int x = tile.x * OM_TX - 2 + hx, y = tile.y * OM_TY - 2 + hy;
    const int z0 = tile.z * zrun, z1 = min(z0 + zrun, c.n[2]);
    const int sx = dn_axis(x, c.n[0], c.bc[0], c.origin), sy = dn_axis(y, c.n[1], c.bc[1], 0);
    const bool in = sx >= 0 && sy >= 0;
    const int at = in ? sx + c.n[0] * sy : 0;
    const bool mine = hx >= 2 && hx < OM_X - 1 && hy >= 2 && hy < OM_Y - 1 && x < c.n[0] && y < c.n[1];
    const int below = max(i - OM_X, 0), above = min(i + OM_X, OM_THREADS - 1);
    const size_t plane = (size_t)c.n[0] * c.n[1];
    // a plane of three fields at this (x, y); zero outside the box
    auto load = [&](const float* const F[3], int z, float v[3]) {
        const int sz = dn_axis(z, c.n[2], c.bc[2], 0);
        const size_t p = plane * max(sz, 0);
        const bool ok = in && sz >= 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) v[d] = ok ? (F[d] + p)[at] : 0.0f;
    };
    const float w0 = 0.25f, w1 = 0.5f;
    float a0[3] = {}, a1[3] = {};
    double part = 0.0;
    // Plane z: t from y (z - 1, z, the neighbours of z in buffer b) and J; y of
    // z + 1 goes to the other buffer; J of z + 2 and y of z + 2 are requested.
    auto step = [&](int z, int b, const float (&Yp)[3], const float (&Y)[3], const float (&Yn)[3], float (&Yf)[3],
                    const float (&J)[3], float (&Jf)[3]) {
        if (z + 1 < z1) {
            load(c.y, z + 2, Yf);
            load(c.src, z + 2, Jf);
        }
        const bool inz = in && dn_axis(z, c.n[2], c.bc[2], 0) >= 0;
        const float yx_y = ysh[b][0][below], yz_y = ysh[b][1][below];
        const float cu0 = (Y[2] - yz_y) * c.inv_d[1] - (Y[1] - Yp[1]) * c.inv_d[2];
        const float cu1 = (Y[0] - Yp[0]) * c.inv_d[2] - (Y[2] - lane_below(Y[2])) * c.inv_d[0];
        const float cu2 = (Y[1] - lane_below(Y[1])) * c.inv_d[0] - (Y[0] - yx_y) * c.inv_d[1];
        const float t[3] = {inz ? fmaf(c.sigma, cu0, J[0]) : 0.0f, inz ? fmaf(c.sigma, cu1, J[1]) : 0.0f,
                            inz ? fmaf(c.sigma, cu2, J[2]) : 0.0f};
        b ^= 1;
        float ax[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            ax[d] = fmaf(w0, lane_above(t[d]), fmaf(w1, t[d], fmaf(w0, lane_below(t[d]), 0.0f)));
            xsh[b][d][i] = ax[d];
        }
        ysh[b][0][i] = Yn[0];
        ysh[b][1][i] = Yn[2];
        __syncthreads();
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float ay = fmaf(w0, xsh[b][d][above], fmaf(w1, ax[d], fmaf(w0, xsh[b][d][below], 0.0f)));
            const float o = fmaf(w0, ay, fmaf(w1, a1[d], fmaf(w0, a0[d], 0.0f)));
            a0[d] = a1[d];
            a1[d] = ay;
            if (z > z0 && mine) {
                float* out = c.dst[d] + plane * (z - 1);
                if (LOSS) {
                    const float e = (o - (c.T[d] + plane * (z - 1))[at]) * c.inv_scale[d];
                    part += (double)e * (double)e;
                    out[at] = c.grad_scale * e * c.inv_scale[d];
                } else {
                    out[at] = o;
                }
            }
        }
    };
    float Y0[3], Y1[3], Y2[3], Y3[3], J0[3], J1[3], J2[3], J3[3];
    load(c.y, z0 - 2, Y0);
    load(c.y, z0 - 1, Y1);
    load(c.src, z0 - 1, J1);
    load(c.y, z0, Y2);
    load(c.src, z0, J2);
    ysh[0][0][i] = Y1[0];
    ysh[0][1][i] = Y1[2];
    __syncthreads();
    for (int z = z0 - 1;; ++z) {   // (four buffers take turns: no register moves, which would wait for the loads)
        step(z, 0, Y0, Y1, Y2, Y3, J1, J3);
        if (++z > z1) break;
        step(z, 1, Y1, Y2, Y3, Y0, J2, J0);
        if (++z > z1) break;
        step(z, 0, Y2, Y3, Y0, Y1, J3, J1);
        if (++z > z1) break;
        step(z, 1, Y3, Y0, Y1, Y2, J0, J2);
        if (z + 1 > z1) break;
    }
    if (LOSS) {
        __shared__ double ws[OM_THREADS / 64];
        for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
        if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = part;
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int k = 0; k < OM_THREADS / 64; ++k) sum += ws[k];
            unsafeAtomicAdd(c.loss, sum * (0.5 * (double)c.grad_scale));
        }
    }
}

// Adjoint of the output stage for training (B is symmetric): dy = sigma
// curl^T(B src), the forward-difference curl
// dy_a = sigma [(b_{a+2}(p + e_{a+1}) - b_{a+2}(p)) / d_{a+1} - (b_{a+1}(p + e_{a+2}) - b_{a+1}(p)) / d_{a+2}],
// b = B src, as bf16 [cell][4] with channel 3 zero: src staged on cells
// -1 .. T + 1, b on 0 .. T (zero outside the box).
constexpr int DA_GX = DO_TX + 3, DA_GY = DO_TY + 3, DA_GZ = DO_TZ + 3;   // src: cells -1 .. T + 1
constexpr int DA_BX = DO_TX + 1, DA_BY = DO_TY + 1, DA_BZ = DO_TZ + 1;   // b: cells 0 .. T

__global__ void __launch_bounds__(DO_THREADS) k_dn_output_adjoint(DnCombine c) {
    __shared__ float gs[3][DA_GZ * DA_GY * DA_GX];
    __shared__ float bs[3][DA_BZ * DA_BY * DA_BX];
    const int3 tile = dn_walk();
    const int t0[3] = {tile.x * DO_TX, tile.y * DO_TY, tile.z * DO_TZ};
    constexpr int NG = DA_GZ * DA_GY * DA_GX, PG = (NG + DO_THREADS - 1) / DO_THREADS;
    constexpr int NB = DA_BZ * DA_BY * DA_BX;
    float v[PG][3];
#pragma unroll
    for (int q = 0; q < PG; ++q) {
        const int i = (int)threadIdx.x + q * DO_THREADS;
        const int hx = i % DA_GX, r = i / DA_GX, hy = r % DA_GY, hz = r / DA_GY;
        const int s = i < NG ? do_src(c, t0[0] - 1 + hx, t0[1] - 1 + hy, t0[2] - 1 + hz) : -1;
#pragma unroll
        for (int d = 0; d < 3; ++d) v[q][d] = dn_at(c.src[d], s);
    }
#pragma unroll
    for (int q = 0; q < PG; ++q) {
        const int i = (int)threadIdx.x + q * DO_THREADS;
        if (i < NG)
#pragma unroll
            for (int d = 0; d < 3; ++d) gs[d][i] = v[q][d];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < NB; i += DO_THREADS) {
        const int hx = i % DA_BX, r = i / DA_BX, hy = r % DA_BY, hz = r / DA_BY;
        const bool in = do_src(c, t0[0] + hx, t0[1] + hy, t0[2] + hz) >= 0;
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) bs[comp][i] = in ? do_binomial<DA_GX, DA_GY>(gs[comp], hx, hy, hz) : 0.0f;
    }
    __syncthreads();
    const int lx = threadIdx.x % DO_TX, ly = (threadIdx.x / DO_TX) % DO_TY, lz = threadIdx.x / (DO_TX * DO_TY);
    const int x = t0[0] + lx, y = t0[1] + ly, z = t0[2] + lz;
    if (x >= c.n[0] || y >= c.n[1] || z >= c.n[2]) return;
    const int b = (lz * DA_BY + ly) * DA_BX + lx;
    const int up[3] = {b + 1, b + DA_BX, b + DA_BX * DA_BY};
    bf16x4 out;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int a1 = (a + 1) % 3, a2 = (a + 2) % 3;
        const float w = (bs[a2][up[a1]] - bs[a2][b]) * c.inv_d[a1] - (bs[a1][up[a2]] - bs[a1][b]) * c.inv_d[a2];
        out[a] = (__bf16)(c.sigma * w);
    }
    out[3] = (__bf16)0.0f;
    reinterpret_cast<bf16x4*>(c.dy)[do_src(c, x, y, z)] = out;
}

static dim3 do_grid(const DnCombine& c) {
    return dim3((c.n[0] + DO_TX - 1) / DO_TX, (c.n[1] + DO_TY - 1) / DO_TY, (c.n[2] + DO_TZ - 1) / DO_TZ);
}

hipError_t launch_dn_output(const DnCombine& c, bool loss, hipStream_t st) {
    // planes per march: 16 (3 more are loaded), fewer where that leaves the
    // chip with less than four workgroups per compute unit.  384x192x160
    // cells: 122 us with 8, 125 with 16, 140 with 32; 128x64x64: 32 with 16
    // (100 workgroups), 16 with 4
    const int tx = (c.n[0] + OM_TX - 1) / OM_TX, ty = (c.n[1] + OM_TY - 1) / OM_TY;
    int zrun = 16;
    while (zrun > 4 && (long long)tx * ty * ((c.n[2] + zrun - 1) / zrun) < 1024) zrun /= 2;
    hipLaunchKernelGGL(loss ? k_dn_output<true> : k_dn_output<false>, dim3(tx, ty, (c.n[2] + zrun - 1) / zrun),
                       dim3(OM_THREADS), 0, st, c, zrun);
    return hipGetLastError();
}

hipError_t launch_dn_output_adjoint(const DnCombine& c, hipStream_t st) {
    hipLaunchKernelGGL(k_dn_output_adjoint, do_grid(c), dim3(DO_THREADS), 0, st, c);
    return hipGetLastError();
}

template <class K>
static hipError_t dn_launch(K kern, const DnArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(kern, dn_grid(a.n), dim3(DN_THREADS), 0, st, a);
    return hipGetLastError();
}

// Persistent layers: one workgroup per compute unit (their LDS allows one),
// never more than there are tiles.
template <class K>
static hipError_t dn_launch_persistent(K kern, size_t lds, const DnArgs& a, hipStream_t st) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int dev = 0, ncu = 0;
    e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const dim3 g = dn_grid(a.n);
    const long long ntiles = (long long)g.x * g.y * g.z;
    long long nb = std::max(1LL, std::min<long long>(ntiles, ncu > 0 ? ncu : 256));
    if (nb >= 8) nb -= nb % 8;   // a multiple of the 8 XCDs: the XCD-aware walk
    hipLaunchKernelGGL(kern, dim3((unsigned)nb), dim3(DN_THREADS), lds, st, a);
    return hipGetLastError();
}

hipError_t launch_dn_layer(int kind, const DnArgs& a, hipStream_t st) {
    switch (kind) {
        case DN_L1_J_ACT: return dn_launch(k_dn_c4<0, 0>, a, st);
        case DN_L1_C4_MASK: return dn_launch(k_dn_c4<1, 1>, a, st);
        case DN_L2_ACT: return dn_launch_persistent(k_dn_conv32<0>, DN_ACT_LDS, a, st);
        case DN_L2_MASK: return dn_launch_persistent(k_dn_conv32<1>, DN_ACT_LDS, a, st);
        case DN_L3_TRAIN: return dn_launch_persistent(k_dn_l3_train, DN_ACT_LDS + L3T_ROWS * 64, a, st);
        case DN_L3_Y: {
            const int tx = (a.n[0] + L3_X - 1) / L3_X, ty = (a.n[1] + L3_Y * L3_WAVES - 1) / (L3_Y * L3_WAVES);
            // planes per wavefront: 16 (2 halo planes loaded), fewer where that leaves the chip with less
            // than two workgroups per compute unit.  384x192x160 cells: 266 us with 16, 301 with 8;
            // 128x64x64 cells: 27 with 16 (160 workgroups), 20 with 8 or 4.
            int zrun = 16;
            while (zrun > 4 && (long long)tx * ty * ((a.n[2] + zrun - 1) / zrun) < 512) zrun /= 2;
            const int tz = (a.n[2] + zrun - 1) / zrun;
            hipLaunchKernelGGL(k_dn_l3, dim3(tx, ty, tz), dim3(64 * L3_WAVES), 0, st, a, zrun);
            return hipGetLastError();
        }
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_denoise(const Geom& g, const int bc[3], const DenoiseWeights& w, float* const Jin[3],
                          float* const Jout[3], float* const Jcopy[3], __bf16* h1, __bf16* h2, hipStream_t st) {
    DnArgs a{};
    for (int d = 0; d < 3; ++d) {
        a.n[d] = g.n[d];
        a.bc[d] = bc[d];
        a.J[d] = Jin[d];
        a.Jcopy[d] = Jcopy ? Jcopy[d] : nullptr;
        a.inv_scale[d] = 1.0f / w.scale[d];
    }
    a.origin = g.window ? g.origin : 0;
    a.act_out = h1;
    a.w = w.w1;
    a.bias = w.b1;
    hipError_t e = launch_dn_layer(DN_L1_J_ACT, a, st);
    if (e != hipSuccess) return e;
    a.act_in = h1;
    a.act_out = h2;
    a.w = w.w2;
    a.bias = w.b2;
    e = launch_dn_layer(DN_L2_ACT, a, st);
    if (e != hipSuccess) return e;
    // y (3 FP32 components) reuses the first activation buffer
    const size_t N = (size_t)g.ncell;
    float* y = reinterpret_cast<float*>(h1);
    a.act_in = h2;
    a.act_out = nullptr;
    a.w = w.w3;
    a.bias = w.b3;
    for (int d = 0; d < 3; ++d) a.Jout[d] = y + d * N;
    e = launch_dn_layer(DN_L3_Y, a, st);
    if (e != hipSuccess) return e;
    // J' = B(J + sigma curl(y)) in one pass (Jout must not alias the J that
    // it reads: columns read their neighbours' J)
    DnCombine c{};
    for (int d = 0; d < 3; ++d) {
        c.n[d] = g.n[d];
        c.bc[d] = bc[d];
        c.src[d] = Jcopy ? Jcopy[d] : Jin[d];
        c.y[d] = y + d * N;
        c.dst[d] = Jout[d];
        c.inv_d[d] = w.inv_d[d];
    }
    c.origin = a.origin;
    c.sigma = w.sigma;
    return launch_dn_output(c, false, st);
}

}  // namespace pic
