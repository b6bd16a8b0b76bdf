// Building blocks of the learned current denoiser's convolutions (inference
// and training): three 3x3x3 convolution layers on the deposited current, as
// implicit GEMMs on the bf16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32
// accumulation).
//
//   x  = bf16(J_d / s_d)                    layer 1: 3 (padded to 4) -> 32 channels
//   a1 = bf16(relu(conv(x, W1) + b1))
//   a2 = bf16(relu(conv(a1, W2) + b2))      layer 2: 32 -> 32 (84 % of the work)
//   J'_d = J_d + s_d (conv(a2, W3) + b3)_d  layer 3: 32 -> 3 (3 x-taps x 4 weight rows)
//
// conv is the "same"-size 3x3x3 cross-correlation; y and z are periodic, x is
// periodic or (moving window) zero beyond the window's two ends, or zero
// outside the box on any axis (training crops).  Activations live in HBM
// channels-last as bf16 [cell][32] (64 B per cell).
//
// Layers 1 and 2: one workgroup of 8 wavefronts computes a tile of 16 x 4 x 8
// cells (x, y, z) in window coordinates: it stages the tile's input halo (18 x
// 6 x 10 cells, rows padded to 20) in LDS.  Layer 1: each wavefront takes one
// z-plane, 4 rows of 16 cells, and all 32 output channels; layer 2: two planes
// and 16 channels, accumulated over the 27 taps x 32 input channels (one MFMA
// K-step of 32 per tap).  Layer 3 streams its input from HBM straight into the
// MFMA operands (k_dn_l3); training keeps one chain of sums per output there
// (k_dn_l3_train).
//
// MFMA operand layout (16x16x32): lane l holds row l%16 of the first operand,
// K elements 8(l/16)..8(l/16)+7, and column l%16 of the second with the same K
// elements; the result holds column l%16, rows 4(l/16)..4(l/16)+3.  Rows =
// output channels (the weights), K = input channels, columns = cells, so that
// a lane's results are neighbouring channels of one cell.  (A and B below
// name the cells' and the weights' fragments.)
//
// The input halo's cell rows are padded to 80 B (8 consecutive cells, one
// 16-byte read each, fall in disjoint bank quadruples), so every read of a
// wavefront is one base address plus a constant per tap.
#pragma once

#include "pic_internal.h"

namespace pic {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int DN_TX = 16, DN_TY = 4, DN_TZ = 8;        // output tile
constexpr int DN_HX = 20, DN_HY = DN_TY + 2, DN_HZ = DN_TZ + 2;   // halo tile (x padded)
constexpr int DN_HCELLS = DN_HX * DN_HY * DN_HZ;
constexpr int DN_THREADS = 512;
constexpr int DN_ROWB = 80;                               // LDS bytes per halo cell row
constexpr int DN_ACT_LDS = DN_HCELLS * DN_ROWB;

// Storage index along one axis of window/box coordinate v, or -1 when the
// neighbour reads as zero.  bc: 0 periodic, 1 zero outside [0, n), 2 moving
// window (zero outside [0, n), storage = (v + origin) mod n).
__device__ __forceinline__ int dn_axis(int v, int n, int bc, int origin) {
    if (bc == 0) return v < 0 ? v + n : (v >= n ? (v == n ? 0 : -1) : v);   // (no output needs v > n)
    if (v < 0 || v >= n) return -1;
    if (bc == 2) {
        v += origin;
        return v >= n ? v - n : v;
    }
    return v;
}

struct DnArgs {
    int n[3];
    int bc[3];
    int origin;
    const float* J[3];        // layer 1 input
    float* Jcopy[3];          // (or null) layer 1 writes its J here as well
    float* Jout[3];           // layer 3 output
    const __bf16* act_in;     // 32-channel input [cell][32]
    __bf16* act_out;          // 32-channel output [cell][32]
    const __bf16* w;          // packed weights (see the host packing)
    const float* bias;
    float inv_scale[3];
    // training
    const __bf16* c4_in;      // 4-channel input [cell][4] (output gradient of layer 3)
    const __bf16* mask;       // relu mask source [cell][32] (an activation: > 0 passes)
};

// Kernel variants: input of the 4-channel-input shape, and epilogues.
// DN_L3_* write y = conv(a2, W3) + b3 as FP32 components into Jout.
enum { DN_L1_J_ACT = 0, DN_L1_C4_MASK, DN_L2_ACT, DN_L2_MASK, DN_L3_Y, DN_L3_TRAIN };

// Output stage J' = B(J + sigma curl(y)) (backward-difference curl, binomial
// filter B), and for training the loss against a target and the gradient.
struct DnCombine {
    int n[3];
    int bc[3];
    int origin;
    const float* src[3];    // J (adjoint: dL/dJ')
    const float* y[3];
    float* dst[3];          // J' (or the loss gradient)
    float sigma;
    float inv_d[3];
    // training
    const float* T[3];
    float inv_scale[3];
    float grad_scale;       // 2 / (3 N)
    double* loss;
    __bf16* dy;             // sigma curl^T(src) as bf16 [cell][4]
};

// dst = B(src + sigma curl(y)); with loss: J' = that against T, dst = dL/dJ' = grad_scale (J' - T) / s^2
hipError_t launch_dn_output(const DnCombine& c, bool loss, hipStream_t st);
// dy = sigma curl^T(B src)
hipError_t launch_dn_output_adjoint(const DnCombine& c, hipStream_t st);

// Output tiles of a box of n cells.
inline dim3 dn_grid(const int n[3]) {
    return dim3((n[0] + DN_TX - 1) / DN_TX, (n[1] + DN_TY - 1) / DN_TY, (n[2] + DN_TZ - 1) / DN_TZ);
}

hipError_t launch_dn_layer(int kind, const DnArgs& a, hipStream_t st);

// Tile of this workgroup in a grid of (nx, ny, nz) tiles.  Workgroups go
// round-robin over the 8 XCDs; each XCD takes a contiguous run of tiles, x
// fastest, then 4 rows of tiles along y, then z, so that the halo along z is
// read while the rows that it shares are still in that XCD's L2.
__device__ __forceinline__ int3 dn_walk(int nx, int ny, int nz, int nb, int id) {
    const int k = id % 8, per = nb / 8, rem = nb % 8;
    const int t = k * per + min(k, rem) + id / 8;
    const int band = nx * 4 * nz, yb = t / band, r = t - yb * band;
    const int rows = min(4, ny - 4 * yb), z = r / (nx * rows), q = r - z * (nx * rows);
    return make_int3(q % nx, 4 * yb + q / nx, z);
}

__device__ __forceinline__ int3 dn_walk() {
    const int id = (int)(blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
    return dn_walk((int)gridDim.x, (int)gridDim.y, (int)gridDim.z, (int)(gridDim.x * gridDim.y * gridDim.z), id);
}

// A 32-channel bf16 activation halo in two phases: every global load of the
// thread into registers (they can stay in flight while the previous tile's
// matrix work runs), then the LDS stores.  A thread takes one 16-byte chunk of
// one (x, y) of the halo (DnLane) in all of its planes, so that only the
// plane, which is uniform, changes between its loads: with the chunks dealt
// linearly the coordinates of every load were computed per lane, which was
// two thirds of the layer's vector instructions.
constexpr int DN_ACT_PER = DN_HZ;
static_assert(DN_HX * DN_HY * 4 <= DN_THREADS, "a thread per chunk of a halo plane");

struct DnLane {
    int hx, hy, chunk;
    bool read;   // reads a cell (x padding is stored as zero)
};

__device__ __forceinline__ DnLane dn_lane() {
    DnLane t;
    const int c = min((int)(threadIdx.x >> 2), DN_HX * DN_HY - 1);   // (the threads over repeat the last cell)
    t.chunk = threadIdx.x & 3;
    t.hx = c % DN_HX;
    t.hy = c / DN_HX;
    t.read = t.hx < DN_TX + 2;
    return t;
}

// Grid and boundary of a layer held in registers for the halo loads.
struct DnBox {
    int n[3], bc[3], origin;
};

__device__ __forceinline__ DnBox dn_box(const DnArgs& a) {
    DnBox b;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        b.n[d] = a.n[d];
        b.bc[d] = a.bc[d];
    }
    b.origin = a.origin;
    return b;
}

// dn_axis without branches (v >= -1).
__device__ __forceinline__ int dn_axis_sel(int v, int n, int bc, int origin) {
    const bool out = v < 0 || v >= n;
    const int w = v < 0 ? v + n : (v >= n ? 0 : v);
    int x = v + origin;
    x = x >= n ? x - n : x;
    const int r = bc == 0 ? w : (bc == 2 ? x : v);
    return (bc != 0 && out) || v > n ? -1 : r;
}

// Starts the loads; returns the planes that lie outside the box (bit k), which
// dn_zero_planes clears once the loads have arrived.
__device__ __forceinline__ unsigned dn_load_act(const __bf16* __restrict__ act, const DnBox& b, const int t0[3],
                                            const DnLane& t, uint4 v[DN_ACT_PER]) {
    const int x = dn_axis_sel(t0[0] - 1 + t.hx, b.n[0], b.bc[0], b.origin);
    const int y = dn_axis_sel(t0[1] - 1 + t.hy, b.n[1], b.bc[1], 0);
    const bool ok = t.read && x >= 0 && y >= 0;
    const uint4* src = reinterpret_cast<const uint4*>(act) + ((size_t)x + (size_t)b.n[0] * y) * 4 + t.chunk;
    const size_t plane = (size_t)b.n[0] * b.n[1] * 4;
#pragma unroll
    for (int k = 0; k < DN_ACT_PER; ++k) v[k] = make_uint4(0u, 0u, 0u, 0u);
    unsigned out = 0;
    size_t at[DN_ACT_PER];
    if (t0[2] >= 1 && t0[2] - 1 + DN_HZ <= b.n[2]) {   // every plane inside the box
        at[0] = plane * (t0[2] - 1);
#pragma unroll
        for (int k = 1; k < DN_ACT_PER; ++k) at[k] = at[k - 1] + plane;
    } else {
#pragma unroll
        for (int k = 0; k < DN_ACT_PER; ++k) {
            const int z = dn_axis_sel(t0[2] - 1 + k, b.n[2], b.bc[2], 0);
            at[k] = plane * max(z, 0);
            out |= z < 0 ? 1u << k : 0u;
        }
    }
    if (ok)
#pragma unroll
        for (int k = 0; k < DN_ACT_PER; ++k) v[k] = src[at[k]];
    return out;
}

__device__ __forceinline__ void dn_zero_planes(uint4 v[DN_ACT_PER], unsigned out) {
    if (out == 0) return;
#pragma unroll
    for (int k = 0; k < DN_ACT_PER; ++k)
        if ((out >> k) & 1) v[k] = make_uint4(0u, 0u, 0u, 0u);
}

__device__ __forceinline__ void dn_store_act(const uint4 v[DN_ACT_PER], const DnLane& t, char* lds) {
    char* p = lds + (t.hy * DN_HX + t.hx) * DN_ROWB + t.chunk * 16;
#pragma unroll
    for (int k = 0; k < DN_ACT_PER; ++k) *reinterpret_cast<uint4*>(p + k * (DN_HX * DN_HY * DN_ROWB)) = v[k];
}

// Output tiles of the box and the origin of tile t (x fastest).
__device__ __forceinline__ int dn_ntiles(const int n[3], int* ntx, int* nty) {
    *ntx = (n[0] + DN_TX - 1) / DN_TX;
    *nty = (n[1] + DN_TY - 1) / DN_TY;
    return *ntx * *nty * ((n[2] + DN_TZ - 1) / DN_TZ);
}

__device__ __forceinline__ void dn_tile_of(int t, int ntx, int nty, int t0[3]) {
    const int bx = t % ntx, r = t / ntx;
    t0[0] = bx * DN_TX;
    t0[1] = (r % nty) * DN_TY;
    t0[2] = (r / nty) * DN_TZ;
}

// Storage cell of output row block `blk` (y row), lane row m, plane lz; -1 outside the box.
__device__ __forceinline__ int dn_out_cell(const DnArgs& a, const int t0[3], int lz, int blk, int m) {
    const int x = t0[0] + m, y = t0[1] + blk, z = t0[2] + lz;
    if (x >= a.n[0] || y >= a.n[1] || z >= a.n[2]) return -1;
    const int xs = a.bc[0] == 2 ? (x + a.origin >= a.n[0] ? x + a.origin - a.n[0] : x + a.origin) : x;
    return xs + a.n[0] * (y + a.n[1] * z);
}

// Output channel of weight operand row r (0..15) of half h: the four rows of
// lane group q (4 q ..) of both halves together are channels 8 q .. 8 q + 7.
__device__ __forceinline__ int dn_co(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// Accumulate the 27 taps x 32 input channels for 16 output channels of 2
// planes x 4 rows of 16 cells: per halo plane and x-tap the wavefront reads the
// 6 halo rows once and uses each for up to 3 dy taps and both output planes,
// 72 reads for 216 matrix instructions.  All taps are unrolled, so every LDS
// address is the lane's base plus a constant.
__device__ __forceinline__ void dn_mma32(const char* act, const bf16x8 W[27], f32x4 acc[2][4]) {
    const int l = threadIdx.x & 63, lz = (threadIdx.x >> 7) * 2;
    const int m = l & 15, q = l >> 4;
    const char* abase = act + (lz * DN_HY * DN_HX + m) * DN_ROWB + q * 16;
#pragma unroll
    for (int pz = 0; pz < 4; ++pz)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            bf16x8 A[DN_HY];
#pragma unroll
            for (int r = 0; r < DN_HY; ++r)
                A[r] = *reinterpret_cast<const bf16x8*>(abase + ((pz * DN_HY + r) * DN_HX + dx) * DN_ROWB);
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const int dz = pz - p;
                    if (dz < 0 || dz > 2) continue;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[p][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[dz * 9 + dy * 3 + dx], A[r + dy],
                                                                            acc[p][r], 0, 0, 0);
                }
        }
}

}  // namespace pic
