// spx_net.hip -- the learned GNEB initial-path corrector: a 4-layer 3^3
// convolution network (10 -> 16 -> 16 -> 16 -> 3 channels, zero padding,
// SiLU between layers) with hand-written FP32 forward, backward and Adam
// kernels.  Input per image: the geodesic guess S_g, the two end images S_A,
// S_B and the reaction coordinate t (10 channels); output u (3 channels) is
// projected on the tangent plane of S_g and applied by the exponential map
// S_hat = exp_{S_g}(P u) (the retraction of the Methods' minimum-energy-path
// section).  Training loss: mean over images and sites of |S_hat - S*|^2.
//
// Activations are [batch][channel][z][y][x] FP32.  Convolutions are direct
// sums on the FP32 matrix cores: a 256-thread block takes boxes of at most 256
// sites in turn (conv_box), stages a box and its one-cell halo for every input
// channel in LDS (SiLU applied on load) and keeps the layer's weights there
// over all its boxes.  The input gradient is the same convolution with
// transposed, flipped weights; weight gradients are sums over the sites on the
// FP64 matrix cores, one partial per block in registers over its boxes, then a
// fixed-order reduction over the blocks (deterministic).
//
// A layer may be dilated by d (tap k reads offset (k - 1) d per axis, which
// widens the receptive field of the four layers from 9 to 1 + 2 (d1 + d2 +
// d3 + d4) cells).  The sites of one phase (px, py, pz) in [0, d)^3, at
// (px + d sx, py + d sy, pz + d sz), only read each other, so a dilated
// layer runs as the same 3^3 tiles over every phase's sub-grid of
// ceil(L / d) sites per axis: tiles stay in sub-grid coordinates and only
// the global addressing is strided.
//
// Inference may instead run every layer as a BF16 implicit GEMM on the
// matrix cores (spx_net_set_precision): for 16 output sites x 16 output
// channels (inputs and outputs padded to 16 channels), K runs over pairs of
// taps x 16 input channels, 14 v_mfma_f32_16x16x32_bf16 per layer with FP32
// accumulation.  The activations between layers are stored as BF16 with the
// channels innermost (32 bytes per site), each layer's epilogue applying
// the next layer's SiLU, so a tile is staged in LDS by 16-byte copies and a
// lane's operand fragment (8 channels of one site and tap) is one 16-byte
// read; the weight fragments of a layer are packed from the FP32 parameters
// by a small kernel before the layer runs.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "spx_device.hpp"
#include "spx_ext.hpp"

namespace spx {
namespace {

constexpr int kTXn = 8, kTYn = 8, kTZn = 4;  // output tile
constexpr int kHX = kTXn + 2, kHY = kTYn + 2, kHZ = kTZn + 2;
constexpr int kNT = 256;

__device__ __forceinline__ float silu(float z) { return z / (1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_grad(float z) {
    const float s = 1.0f / (1.0f + __expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

struct NetDims {
    int Lx, Ly, Lz;
    int64_t P;
    int dil;         // dilation of the layer
    int Sx, Sy, Sz;  // sub-grid extents ceil(L / dil)
};

// Tile of this block: origin (x0, y0, z0) in sub-grid coordinates and the
// phase (px, py, pz).  blockIdx.x = bx + nbx (by + nby (px + dil py)),
// blockIdx.y = bz + nbz pz.
struct NetTile {
    int x0, y0, z0, px, py, pz;
};
__device__ __forceinline__ NetTile tile_origin_at(const NetDims &d, int bx, int by) {
    const int nbx = (d.Sx + kTXn - 1) / kTXn, nby = (d.Sy + kTYn - 1) / kTYn, nbz = (d.Sz + kTZn - 1) / kTZn;
    NetTile t;
    int r = bx;
    t.x0 = (r % nbx) * kTXn;
    r /= nbx;
    t.y0 = (r % nby) * kTYn;
    r /= nby;
    t.px = r % d.dil;
    t.py = r / d.dil;
    t.z0 = (by % nbz) * kTZn;
    t.pz = by / nbz;
    return t;
}
// ---------------------------------------------------------------- FP32 matrix-core form
// Tiles of the FP32 layers: a box of bx x by x bz <= 256 sub-grid sites whose
// one-cell halo holds at most kBoxHalo sites, chosen per layer on the host
// (conv_box) for the fewest tiles.  An 8 x 8 x 4 box fills only 42% of its
// sites on the 6^3 sub-grids of dilation 8 at 48^3 and 56% on the 12^3 of
// dilation 4; 6 x 6 x 6 fills 84% of both.  Blocks are persistent over the
// tiles (tile index = box, then phase, then image).
constexpr int kBoxSites = 256, kBoxHalo = 640;
constexpr int kConvBlocks = 512;  // two per CU: what the registers and LDS of either kernel admit

struct NetBox {
    int bx, by, bz;     // box
    int nx, ny, nz;     // boxes per axis of one phase's sub-grid
    int hx, hy, halo;   // halo row, rows per halo plane, halo sites
    int px, py, pz;     // phases per axis, min(dil, L)
    int vol;            // bx by bz
    int64_t tiles;      // nx ny nz px py pz batch
};

struct BoxTile {
    int x0, y0, z0;  // lattice coordinates of box site (0, 0, 0)
    int image;
};
__device__ __forceinline__ BoxTile box_tile(const NetDims &d, const NetBox &b, int64_t t) {
    // at most one tile per site: 32 bits hold an image's tiles
    const uint32_t per_image = (uint32_t)b.nx * b.ny * b.nz * b.px * b.py * b.pz;
    BoxTile o;
    o.image = (int)(t / per_image);
    uint32_t r = (uint32_t)(t - (int64_t)o.image * per_image);
    const uint32_t px = r % (uint32_t)b.px;  // phases innermost: they share cache lines
    r /= (uint32_t)b.px;
    const uint32_t py = r % (uint32_t)b.py;
    r /= (uint32_t)b.py;
    const uint32_t ix = r % (uint32_t)b.nx;
    r /= (uint32_t)b.nx;
    const uint32_t iy = r % (uint32_t)b.ny;
    r /= (uint32_t)b.ny;
    const uint32_t iz = r % (uint32_t)b.nz;
    const uint32_t pz = r / (uint32_t)b.nz;
    o.x0 = (int)px + d.dil * b.bx * (int)ix;
    o.y0 = (int)py + d.dil * b.by * (int)iy;
    o.z0 = (int)pz + d.dil * b.bz * (int)iz;
    return o;
}

// First tile of this block when workgroups are dealt to the 8 XCDs in turn:
// blocks of one XCD take consecutive tiles, so the halos that neighbouring
// tiles share meet in one L2.
__device__ __forceinline__ int64_t first_tile() {
    const uint32_t T = gridDim.x, b = blockIdx.x, q = T / 8, r = T % 8, k = b % 8;
    return (int64_t)(k * q + (k < r ? k : r) + b / 8);
}

// The halo sites that a thread stages, (x, y, z) packed by 10 bits, -1 past the end.
constexpr int kSlots = (kBoxHalo + kNT - 1) / kNT;
__device__ __forceinline__ void halo_slots(const NetBox &b, int slot[kSlots]) {
#pragma unroll
    for (int q = 0; q < kSlots; ++q) {
        const int r = (int)threadIdx.x + q * kNT;
        const int x = r % b.hx, yz = r / b.hx, y = yz % b.hy, z = yz / b.hy;
        slot[q] = r < b.halo ? x | (y << 10) | (z << 20) : -1;
    }
}
// lattice index of a packed halo site of a tile, -1 outside the lattice
__device__ __forceinline__ int64_t halo_site(const NetDims &d, const BoxTile &t, int slot) {
    const int x = t.x0 + d.dil * ((slot & 1023) - 1), y = t.y0 + d.dil * (((slot >> 10) & 1023) - 1),
              z = t.z0 + d.dil * ((slot >> 20) - 1);
    const bool in = x >= 0 && y >= 0 && z >= 0 && x < d.Lx && y < d.Ly && z < d.Lz;
    return in ? x + (int64_t)d.Lx * (y + (int64_t)d.Ly * z) : -1;
}
// box site s = threadIdx.x of a tile: its coordinates packed likewise (-1 past the box)
__device__ __forceinline__ int box_slot(const NetBox &b, int s) {
    const int x = s % b.bx, yz = s / b.bx, y = yz % b.by, z = yz / b.by;
    return s < b.vol ? (x + 1) | ((y + 1) << 10) | ((z + 1) << 20) : -1;
}

// out[co] = bias[co] + sum_ci sum_k W[co][ci][k] a[ci](p + (k - 1) d)   (bias may be NULL)
// MUL_GRAD: the result is multiplied by silu'(zmul) (input-gradient pass).
//
// Each wavefront takes 64 sites of the box as four groups of 16, all 16
// output channels (COUT < 16: zero weights) and K = 27 CIN in steps of four:
// v_mfma_f32_16x16x4_f32 with the sites as rows and W[co][kk], kk = 27 ci +
// k, as columns.  That instruction adds its four products to the accumulator
// one after another, each a fused multiply-add with FP32 rounding (checked
// bit for bit against fmaf, subnormals included), and kk runs in the order of
// the sum above, so a result is the same chain of FMAs, bit for bit, as one
// thread per site doing them in turn on the vector ALU.  The weights of the
// block stay in LDS and the 27 tap offsets of a lane in registers over all its
// tiles; kk + 108 is the same tap four channels on.
// Bound by the matrix cores' FP32 rate with the staging of the next block's
// tile beside it: 16 -> 16 channels on 16 images of 48^3 (24.5 GFLOP) took
// 908 us on the vector ALUs.
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int CIN, int COUT, bool SILU_IN, bool MUL_GRAD>
__global__ __launch_bounds__(kNT, 2) void k_conv(const float *__restrict__ in, const float *__restrict__ W,
                                                 const float *__restrict__ bias, const float *__restrict__ zmul,
                                                 float *__restrict__ out, NetDims d, NetBox bx) {
    constexpr int K = 27 * CIN, NS = (K + 3) / 4;
    constexpr int kOt = kBoxSites + 4;      // floats per channel row of the output staging
    constexpr int kTile = CIN * kBoxHalo > COUT * kOt ? CIN * kBoxHalo : COUT * kOt;
    __shared__ __attribute__((aligned(16))) float tile[kTile + 1];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, row = lane & 15, quad = lane >> 4;
    // weight fragments: lane l of step i reads W[co = l % 16][4 i + l / 16]
    __shared__ float wl[NS * 64];
    for (int q = t; q < NS * 64; q += kNT) {
        const int co = q & 15, kk = 4 * (q >> 6) + ((q >> 4) & 3);
        wl[q] = (co < COUT && kk < K) ? W[co * K + kk] : 0.0f;
    }
    const float bco = (bias && row < COUT) ? bias[row] : 0.0f;
    int off[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) {
        const int kk = 4 * i + quad, ci = kk / 27, k = kk - 27 * ci;
        off[i] = ci * kBoxHalo + k % 3 + bx.hx * ((k / 3) % 3 + bx.hy * (k / 9));
    }
    int base[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const int s = 16 * (4 * wave + m) + row;
        const int q = s < bx.vol ? s : 0;
        base[m] = q % bx.bx + bx.hx * ((q / bx.bx) % bx.by + bx.hy * (q / (bx.bx * bx.by)));
    }
    int slot[kSlots];
    halo_slots(bx, slot);
    const int own = box_slot(bx, t);
    for (int64_t tl = first_tile(); tl < bx.tiles; tl += gridDim.x) {
        const BoxTile o = box_tile(d, bx, tl);
        const float *src = in + (int64_t)o.image * CIN * d.P;
#pragma unroll
        for (int q = 0; q < kSlots; ++q) {
            if (slot[q] < 0) continue;
            const int64_t p = halo_site(d, o, slot[q]);
            float v[CIN];
#pragma unroll
            for (int ci = 0; ci < CIN; ++ci) v[ci] = p >= 0 ? src[ci * d.P + p] : 0.0f;
#pragma unroll
            for (int ci = 0; ci < CIN; ++ci)
                tile[ci * kBoxHalo + t + q * kNT] = SILU_IN ? (p >= 0 ? silu(v[ci]) : 0.0f) : v[ci];
        }
        if (K % 4 != 0 && t == 0) tile[kTile] = 0.0f;  // read by the lanes past K in the last step
        __syncthreads();
        f32x4 acc[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[m] = f32x4{bco, bco, bco, bco};
        auto step = [&](int i, int r, int ch) __attribute__((always_inline)) {
            const float wv = wl[i * 64 + lane];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                int at = base[m] + off[r] + ch * kBoxHalo;
                if (K % 4 != 0 && i == NS - 1) at = 4 * i + quad < K ? at : kTile;
                acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(tile[at], wv, acc[m], 0, 0, 0);
            }
        };
        // four channels are 27 steps; the loop over them stays rolled and its
        // 108 tile addresses are made in it (held over the tiles they spill)
#pragma unroll 1
        for (int c4 = 0; c4 < NS / 27; ++c4) {
#pragma unroll
            for (int m = 0; m < 4; ++m) asm volatile("" : "+v"(base[m]));
#pragma unroll
            for (int r = 0; r < 27; ++r) step(27 * c4 + r, r, 4 * c4);
        }
#pragma unroll
        for (int i = NS / 27 * 27; i < NS; ++i) step(i, i % 27, i / 27 * 4);
        __syncthreads();  // every wavefront is done with the tile
        // accumulator j of a lane: site 16 (4 wave + m) + 4 quad + j, channel row
        if (row < COUT) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
                *reinterpret_cast<f32x4 *>(tile + row * kOt + 16 * (4 * wave + m) + 4 * quad) = acc[m];
        }
        __syncthreads();
        const int64_t p = own >= 0 ? halo_site(d, o, own) : -1;
        if (p >= 0) {
            float *dst = out + (int64_t)o.image * COUT * d.P + p;
            const float *zm = MUL_GRAD ? zmul + (int64_t)o.image * COUT * d.P + p : nullptr;
#pragma unroll
            for (int co = 0; co < COUT; ++co) {
                float v = tile[co * kOt + t];
                if (MUL_GRAD) v *= silu_grad(zm[co * d.P]);
                dst[co * d.P] = v;
            }
        }
        __syncthreads();  // the next tile is staged over the outputs
    }
}

// Wt[ci][co][k] = W[co][ci][26 - k]: weights of the input-gradient convolution.
__global__ void k_transpose_flip(const float *__restrict__ W, float *__restrict__ Wt, int cin, int cout) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cin * cout * 27) return;
    const int k = i % 27, co = (i / 27) % cout, ci = i / (27 * cout);
    Wt[i] = W[(co * cin + ci) * 27 + (26 - k)];
}

// Weight and bias gradients of a layer, one partial per block (and site half):
//   dW[co][ci][k] = sum_p g[co](p) a[ci](p + (k - 1) d),  db[co] = sum_p g[co](p).
// FP64 accumulation: the product of two floats is exact in double, so the
// sums carry no FP32 rounding of their own.  v_mfma_f64_16x16x4_f64 contracts
// four sites at a time: the 16 channels of one field (rows, the box alone)
// against channel and tap of the other (columns, with halo), flattened so
// that 10 channels fill 17 column tiles of 16 and 3 channels 6.
//   SWAP = false: rows g, columns a (CC = cin); true (3 outputs): rows a,
//   columns g (CC = cout), whose tap k is a's tap 26 - k.
// The column tiles are dealt to 4 / WS wavefronts, the sites to WS groups of
// them; the accumulators live in registers over all tiles of the block, so a
// block writes one partial (before: one per tile, 6912 of 55 kB for a 16 ->
// 16 layer of 16 images of 48^3, which one thread per weight then summed).
// Bound by the FP64 matrix rate; the vector ALUs took 3792 us for that layer
// and the sum 4054 us.
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int CC, bool SWAP, bool SILU_A, int WS>
__global__ __launch_bounds__(kNT, 2) void k_conv_wgrad(const float *__restrict__ in, const float *__restrict__ g,
                                                       double *__restrict__ partial, NetDims d, NetBox bx) {
    constexpr int NC = 27 * CC, NT = (NC + 15) / 16, NWV = 4 / WS, NJ = (NT + NWV - 1) / NWV;
    constexpr int PC = CC | 1, PR = 17;  // odd pitches: staging writes and fragment reads spread over the banks
    constexpr int COUT = SWAP ? CC : 16, CIN = SWAP ? 16 : CC;
    constexpr int nw = COUT * CIN * 27 + COUT;
    __shared__ float hal[kBoxHalo * PC];
    __shared__ float rows[kBoxSites * PR];
    __shared__ int hb[kBoxSites];
    __shared__ double red[kNT / 64][COUT];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, row = lane & 15, quad = lane >> 4;
    const int wv = wave % NWV, ws = wave / NWV;
    int coff[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int n = 16 * (wv + NWV * j) + row;
        const int k = n < NC ? n / CC : 0, c = n < NC ? n - CC * (n / CC) : 0;
        coff[j] = PC * (k % 3 + bx.hx * ((k / 3) % 3 + bx.hy * (k / 9))) + c;
    }
    {
        const int q = t < bx.vol ? t : 0;
        hb[t] = PC * (q % bx.bx + bx.hx * ((q / bx.bx) % bx.by + bx.hy * (q / (bx.bx * bx.by))));
    }
    int slot[kSlots];
    halo_slots(bx, slot);
    const int own = box_slot(bx, t);
    f64x4 acc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[j] = f64x4{0.0, 0.0, 0.0, 0.0};
    double sb[COUT];
#pragma unroll
    for (int c = 0; c < COUT; ++c) sb[c] = 0.0;
    // groups of four sites, at most 64 (54 for a box of 6 x 6 x 6); the last turn
    // below may pass them but stays below 64, where rows are zero and hb valid
    const int groups = (bx.vol + 3) / 4;
    for (int64_t tl = first_tile(); tl < bx.tiles; tl += gridDim.x) {
        const BoxTile o = box_tile(d, bx, tl);
        const float *csrc = (SWAP ? g : in) + (int64_t)o.image * CC * d.P;
        const float *rsrc = (SWAP ? in : g) + (int64_t)o.image * 16 * d.P;
        __syncthreads();  // the previous tile's reads are done (and hb is written)
#pragma unroll
        for (int q = 0; q < kSlots; ++q) {
            if (slot[q] < 0) continue;
            const int64_t p = halo_site(d, o, slot[q]);
            float v[CC];
#pragma unroll
            for (int c = 0; c < CC; ++c) v[c] = p >= 0 ? csrc[c * d.P + p] : 0.0f;
#pragma unroll
            for (int c = 0; c < CC; ++c)
                hal[(t + q * kNT) * PC + c] = (!SWAP && SILU_A) ? (p >= 0 ? silu(v[c]) : 0.0f) : v[c];
        }
        {
            const int64_t p = own >= 0 ? halo_site(d, o, own) : -1;
            float v[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) v[c] = p >= 0 ? rsrc[c * d.P + p] : 0.0f;
#pragma unroll
            for (int c = 0; c < 16; ++c)
                rows[t * PR + c] = (SWAP && SILU_A) ? (p >= 0 ? silu(v[c]) : 0.0f) : v[c];
            if constexpr (!SWAP) {
#pragma unroll
                for (int c = 0; c < COUT; ++c) sb[c] += (double)v[c];
            } else if (p >= 0) {
#pragma unroll
                for (int c = 0; c < COUT; ++c) sb[c] += (double)csrc[c * d.P + p];
            }
        }
        __syncthreads();
        // four groups of four sites a turn (rows past the box are zero)
        for (int q0 = ws; q0 < groups; q0 += 4 * WS) {
            int h[4];
            double a[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int sq = 4 * (q0 + e * WS) + quad;
                h[e] = hb[sq];
                a[e] = (double)rows[sq * PR + row];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], (double)hal[h[e] + coff[j]], acc[j], 0, 0, 0);
        }
    }
    // accumulator i of a lane: row 4 i + quad, column lane % 16 of the tile
    double *dst = partial + ((size_t)blockIdx.x * WS + ws) * nw;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int n = 16 * (wv + NWV * j) + row;
        if (n >= NC) continue;
        const int k = n / CC, c = n - CC * k;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * i + quad;
            dst[SWAP ? (c * CIN + r) * 27 + 26 - k : (r * CIN + c) * 27 + k] = acc[j][i];
        }
    }
#pragma unroll
    for (int c = 0; c < COUT; ++c) {
        const double v = wave_sum(sb[c]);
        if (lane == 0) red[wave][c] = v;
    }
    __syncthreads();
    if (t < COUT) {
        double v = 0.0;
        for (int q = 0; q < kNT / 64; ++q) v += red[q][t];
        double *db = partial + (size_t)blockIdx.x * WS * nw + COUT * CIN * 27 + t;
        db[0] = v;
        for (int q = 1; q < WS; ++q) db[(size_t)q * nw] = 0.0;
    }
}

// Fixed-order FP64 sum of n_part partial vectors of length nw, rounded to
// float once: 32 weights per block, eight interleaved runs of partials each.
constexpr int kSumW = 32;
__global__ __launch_bounds__(kNT) void k_sum_partials(const double *__restrict__ partial, int n_part, int nw,
                                                      float *__restrict__ out) {
    __shared__ double red[kNT / kSumW][kSumW];
    const int c = threadIdx.x % kSumW, r = threadIdx.x / kSumW, i = blockIdx.x * kSumW + c;
    double s = 0.0;
    if (i < nw) {
#pragma unroll 8
        for (int b = r; b < n_part; b += kNT / kSumW) s += partial[(size_t)b * nw + i];
    }
    red[r][c] = s;
    __syncthreads();
    if (r == 0 && i < nw) {
        for (int q = 1; q < kNT / kSumW; ++q) s += red[q][c];
        out[i] = (float)s;
    }
}

// Network input: channels (S_g, S_A, S_B, t) as FP32.
// ab_stride: 3P for per-image end images, 0 when all images share them.
__global__ void k_net_input(const double *__restrict__ Sg, const double *__restrict__ SA,
                            const double *__restrict__ SB, const float *__restrict__ t, float *__restrict__ x,
                            int64_t P, int64_t ab_stride) {
    const int64_t p = (int64_t)blockIdx.x * kNT + threadIdx.x;
    const int b = blockIdx.y;
    if (p >= P) return;
    float *xb = x + (int64_t)b * 10 * P;
    const int64_t o = (int64_t)b * 3 * P, oab = (int64_t)b * ab_stride;
    for (int c = 0; c < 3; ++c) {
        xb[c * P + p] = (float)Sg[o + c * P + p];
        xb[(3 + c) * P + p] = (float)SA[oab + c * P + p];
        xb[(6 + c) * P + p] = (float)SB[oab + c * P + p];
    }
    xb[9 * P + p] = t[b];
}

// S_hat = exp_{S_g}(P_perp u) (FP64); with S* also the loss partial per block
// and d loss / d u for the backward pass (loss = mean over batch and sites).
__global__ __launch_bounds__(kNT) void k_net_head(const float *__restrict__ u, const double *__restrict__ Sg,
                                                  const double *__restrict__ Sstar, double *__restrict__ Shat,
                                                  float *__restrict__ gu, double *__restrict__ loss_part, int64_t P,
                                                  double inv_count) {
    __shared__ double red[kNT / 64];
    const int64_t p = (int64_t)blockIdx.x * kNT + threadIdx.x;
    const int b = blockIdx.y;
    double l = 0.0;
    if (p < P) {
        const int64_t o = (int64_t)b * 3 * P;
        double s[3], r[3];
        for (int c = 0; c < 3; ++c) {
            s[c] = Sg[o + c * P + p];
            r[c] = (double)u[o + c * P + p];
        }
        const double rs = r[0] * s[0] + r[1] * s[1] + r[2] * s[2];
        double w[3] = {r[0] - rs * s[0], r[1] - rs * s[1], r[2] - rs * s[2]};
        const double th = sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
        double sinc, c2;  // sin(th)/th, (cos th - sinc)/th^2 with series near 0
        if (th < 1e-4) {
            const double t2 = th * th;
            sinc = 1.0 - t2 / 6.0 + t2 * t2 / 120.0;
            c2 = -1.0 / 3.0 + t2 / 30.0;
        } else {
            sinc = sin(th) / th;
            c2 = (cos(th) - sinc) / (th * th);
        }
        const double ct = cos(th);
        double h[3] = {ct * s[0] + sinc * w[0], ct * s[1] + sinc * w[1], ct * s[2] + sinc * w[2]};
        normalise3(h);
        if (Shat)
            for (int c = 0; c < 3; ++c) Shat[o + c * P + p] = h[c];
        if (Sstar) {
            double gs[3];
            for (int c = 0; c < 3; ++c) {
                const double dlt = h[c] - Sstar[o + c * P + p];
                l += dlt * dlt;
                gs[c] = 2.0 * dlt * inv_count;
            }
            const double ug = w[0] * gs[0] + w[1] * gs[1] + w[2] * gs[2];
            const double sg = s[0] * gs[0] + s[1] * gs[1] + s[2] * gs[2];
            double gw[3];
            for (int c = 0; c < 3; ++c) gw[c] = sinc * gs[c] + c2 * ug * w[c] - sinc * sg * w[c];
            const double gws = gw[0] * s[0] + gw[1] * s[1] + gw[2] * s[2];
            for (int c = 0; c < 3; ++c) gu[o + c * P + p] = (float)(gw[c] - gws * s[c]);
        }
    }
    if (loss_part) {
        const double t = wave_sum(l);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
        __syncthreads();
        if (threadIdx.x == 0) {
            double a = 0.0;
            for (int w = 0; w < kNT / 64; ++w) a += red[w];
            loss_part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = a;
        }
    }
}

// The loss: a fixed-order sum of the block partials by one block.
__global__ __launch_bounds__(kNT) void k_loss_final(const double *__restrict__ part, int n, double scale,
                                                    double *__restrict__ loss) {
    __shared__ double red[kNT / 64];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += kNT) s += part[i];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0;
        for (int q = 0; q < kNT / 64; ++q) a += red[q];
        *loss = a * scale;
    }
}

// ---------------------------------------------------------------- BF16 MFMA form
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kTapPairs = 14;  // 27 taps in pairs, the last padded

// v_mfma_f32_16x16x32_bf16, one wavefront: lane l holds A[l % 16][8 (l / 16) + j]
// and B[8 (l / 16) + j][l % 16], j = 0..7; accumulator i of lane l is
// D[4 (l / 16) + i][l % 16].
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Weight fragments of one layer: frag[tp][lane][j] = W[co][ci][tap] with
// co = lane % 16, tap = 2 tp + (lane / 32), ci = 8 ((lane / 16) & 1) + j
// (zero for co >= cout, ci >= cin or tap 27), rounded to BF16.
__global__ void k_wfrag(const float *__restrict__ W, int cin, int cout, bf16x8 *__restrict__ frag) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kTapPairs * 64) return;
    const int tp = i / 64, lane = i % 64;
    const int co = lane % 16, tap = 2 * tp + (lane >> 5), ci0 = 8 * ((lane >> 4) & 1);
    bf16x8 v;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int ci = ci0 + j;
        const float w = (co < cout && ci < cin && tap < 27) ? W[(co * cin + ci) * 27 + tap] : 0.0f;
        v[j] = (__bf16)w;
    }
    frag[i] = v;
}

// The BF16 form keeps each layer's input as BF16 activations with the 16
// channels innermost, a[b][p][16] (32 bytes per site; layer 0: the 10 input
// channels and six zeros), so that staging a tile is a copy of 32 bytes per
// halo site.  Each layer's epilogue writes the next layer's input,
// BF16(SiLU(z)); the last writes its FP32 pre-activation u [b][3][p] for the
// head.

// layer-0 input: (S_g, S_A, S_B, t) rounded to float, then to BF16
__global__ void k_net_input_bf16(const double *__restrict__ Sg, const double *__restrict__ SA,
                                 const double *__restrict__ SB, const float *__restrict__ t,
                                 bf16x8 *__restrict__ xa, int64_t P, int64_t ab_stride) {
    const int64_t p = (int64_t)blockIdx.x * kNT + threadIdx.x;
    const int b = blockIdx.y;
    if (p >= P) return;
    const int64_t o = (int64_t)b * 3 * P, oab = (int64_t)b * ab_stride;
    float v[16];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        v[c] = (float)Sg[o + c * P + p];
        v[3 + c] = (float)SA[oab + c * P + p];
        v[6 + c] = (float)SB[oab + c * P + p];
    }
    v[9] = t[b];
#pragma unroll
    for (int c = 10; c < 16; ++c) v[c] = 0.0f;
    bf16x8 lo, hi;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        lo[j] = (__bf16)v[j];
        hi[j] = (__bf16)v[8 + j];
    }
    bf16x8 *dst = xa + ((int64_t)b * P + p) * 2;
    dst[0] = lo;
    dst[1] = hi;
}

// Workgroups are dealt to the 8 XCDs in turn by linear id (x fastest).  This
// renumbering gives each XCD one contiguous range of the grid instead, so the
// d^3 phase tiles of one region, consecutive in x, run on one XCD: the
// strided halo rows they read and the partial cache lines they write meet in
// its L2.  The grid holds fewer than 2^31 blocks.
struct GridBlock {
    int x, y, z;
};
__device__ __forceinline__ GridBlock xcd_grid_block() {
    const uint32_t gx = gridDim.x, gy = gridDim.y, T = gx * gy * gridDim.z;
    const uint32_t b = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
    const uint32_t q = T / 8, r = T % 8, k = b % 8;
    const uint32_t l = k * q + (k < r ? k : r) + b / 8;
    return GridBlock{(int)(l % gx), (int)((l / gx) % gy), (int)(l / (gx * gy))};
}

// The BF16 halo tile in LDS: 32 bytes per site (16 channels), x rows of 10
// sites (320 bytes).  The two 16-byte halves of a site are stored swapped
// where bit 2 of its halo x is set, so that the 8 lanes (x = 0..7) that read
// one half each in an A-operand load cover eight different 16-byte bank
// groups instead of four (measured: 36% fewer bank-conflict cycles; the
// layer's time is set elsewhere and did not move).
constexpr int kRowB = kHX * 32, kPlaneB = kHY * kRowB, kTileB = kHZ * kPlaneB;
__host__ __device__ constexpr int swz(int hx) { return (hx >> 2) & 1; }

// byte offset of the y and z parts of tap (kx, ky, kz) = (tap % 3, tap / 3 %
// 3, tap / 9) in the tile, and its kx; the padded tap 27 reads offset 0 (its
// weights are zero)
constexpr int tap_bytes(int tap) { return tap >= 27 ? 0 : kRowB * ((tap / 3) % 3) + kPlaneB * (tap / 9); }
constexpr int tap_kx(int tap) { return tap >= 27 ? 0 : tap % 3; }

// SiLU with the hardware reciprocal: its result is rounded to BF16 next
__device__ __forceinline__ float silu_bf16(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// out[co] = bias[co] + sum_ci sum_k W[co][ci][k] a[ci](p + (k - 1) d), BF16
// operands, FP32 accumulation; the block's 8 x 8 x 4 tile is 16 groups of 16
// sites (two y rows of one z plane), four per wavefront.  LAST: write the
// FP32 pre-activation of the COUT channels to u [b][COUT][p]; otherwise
// BF16(SiLU) of all 16 channels to the next activation buffer.  Either goes
// through LDS first, site-major, so that each thread then writes one site.
template <int COUT, bool LAST>
__global__ __launch_bounds__(kNT) void k_conv_mfma(const bf16x8 *__restrict__ in, const bf16x8 *__restrict__ frag,
                                                   const float *__restrict__ bias, void *__restrict__ out,
                                                   NetDims d) {
    static_assert(kHX == 10 && kHY * kHZ == 60 && kNT >= 240, "staging map assumes the 10 x 10 x 6 halo");
    static_assert(kTileB >= kNT * 32, "the epilogue reuses the tile");
    __shared__ __attribute__((aligned(16))) char lds[kTileB];
    const GridBlock g = xcd_grid_block();
    const NetTile tl = tile_origin_at(d, g.x, g.y);
    const int t = threadIdx.x;
    // staging: thread t < 240 copies the 16-byte chunk c = t % 20 (halo x =
    // c / 2, channels 8 (c % 2) .. + 7) of halo rows t / 20 + 12 k, k = 0..4
    // (row = hy + kHY hz); sites outside the lattice are zero
    if (t < 240) {
        const int c = t % 20, hx = c >> 1, half = c & 1, r0 = t / 20;
        const int gx = tl.px + d.dil * (tl.x0 + hx - 1);
        const bool okx = gx >= 0 && gx < d.Lx;
        const bf16x8 *src = in + (int64_t)g.z * d.P * 2 + half;
        bf16x8 v[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const int hr = r0 + 12 * k, hy = hr % kHY, hz = hr / kHY;
            const int gy = tl.py + d.dil * (tl.y0 + hy - 1), gz = tl.pz + d.dil * (tl.z0 + hz - 1);
            const bool ok = okx && gy >= 0 && gy < d.Ly && gz >= 0 && gz < d.Lz;
            const int64_t o = ok ? (gx + (int64_t)d.Lx * (gy + (int64_t)d.Ly * gz)) * 2 : 0;
            v[k] = src[o];
            if (!ok) v[k] = bf16x8{};
        }
#pragma unroll
        for (int k = 0; k < 5; ++k)
            *reinterpret_cast<bf16x8 *>(lds + (r0 + 12 * k) * kRowB + 32 * hx + 16 * (half ^ swz(hx))) = v[k];
    }
    __syncthreads();
    const int lane = t & 63, wave = t >> 6, row = lane & 15, grp = lane >> 4;
    // lane's A operand: site (x, y, z) = (row % 8, row / 8 + 2 m, wave) of
    // group m, channels 8 (grp % 2) .. + 7; lanes 32..63 take the pair's
    // second tap.  abx[kx]: the byte address of that half at tap offset kx
    // in x (the y and z offsets of a tap add to it)
    int abx[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int hx = (row & 7) + k;
        abx[k] = 32 * hx + kRowB * (row >> 3) + kPlaneB * wave + 16 * ((grp & 1) ^ swz(hx));
    }
    const bool second = grp >= 2;
    f32x4 acc[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[m] = f32x4{};
#pragma unroll
    for (int tp = 0; tp < kTapPairs; ++tp) {
        const bf16x8 b = frag[tp * 64 + lane];
        const int a = second ? abx[tap_kx(2 * tp + 1)] + tap_bytes(2 * tp + 1) : abx[tap_kx(2 * tp)] + tap_bytes(2 * tp);
#pragma unroll
        for (int m = 0; m < 4; ++m)
            acc[m] = mfma16(*reinterpret_cast<const bf16x8 *>(lds + a + 2 * kRowB * m), b, acc[m]);
    }
    // accumulator i of lane l: site 16 mb + 4 grp + i of the tile (mb = 4
    // wave + m), channel co = l % 16
    const int co = lane & 15;
    __syncthreads();  // every wavefront is done with the tile
    // thread t then writes site t: group mb = t / 16, r = t % 16
    const int mb = t >> 4, r = t & 15;
    const int x = tl.px + d.dil * (tl.x0 + (r & 7)), y = tl.py + d.dil * (tl.y0 + 2 * (mb & 3) + (r >> 3)),
              z = tl.pz + d.dil * (tl.z0 + (mb >> 2));
    const bool inside = x < d.Lx && y < d.Ly && z < d.Lz;
    const int64_t p = x + (int64_t)d.Lx * (y + (int64_t)d.Ly * z);
    if constexpr (LAST) {
        float(*ot)[4] = reinterpret_cast<float(*)[4]>(lds);  // ot[site][co]
        if (co < COUT) {
            const float bco = bias[co];
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) ot[16 * (4 * wave + m) + 4 * grp + i][co] = acc[m][i] + bco;
        }
        __syncthreads();
        if (inside) {
            float *u = static_cast<float *>(out) + (int64_t)g.z * COUT * d.P + p;
#pragma unroll
            for (int c = 0; c < COUT; ++c) u[(int64_t)c * d.P] = ot[t][c];
        }
    } else {
        // ot[site][8 channel pairs]; the two 16-byte halves of site s are
        // swapped when bit 3 of s is set, which spreads the one-half reads
        // of consecutive sites over the bank groups (of bits 2 and 3, bit 3
        // measured fewer conflict cycles).  Lanes co and co ^ 1 trade one
        // value so that each writes a channel pair of one site: the even
        // lane sites 4 grp + i, the odd lane 4 grp + i + 1.
        bf16x2(*ot)[8] = reinterpret_cast<bf16x2(*)[8]>(lds);
        const float bco = bias[co];
        const bool odd = co & 1;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                const float v0 = silu_bf16(acc[m][i] + bco), v1 = silu_bf16(acc[m][i + 1] + bco);
                const float got =
                    __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(odd ? v0 : v1), 0xB1, 0xF, 0xF, false));
                const int st = 16 * (4 * wave + m) + 4 * grp + i + (odd ? 1 : 0);
                const bf16x2 pr = odd ? bf16x2{(__bf16)got, (__bf16)v1} : bf16x2{(__bf16)v0, (__bf16)got};
                ot[st][(co >> 1) ^ (st & 8 ? 4 : 0)] = pr;
            }
        __syncthreads();
        if (inside) {
            const int sw = t & 8 ? 1 : 0;
            const bf16x8 lo = *reinterpret_cast<const bf16x8 *>(lds + 32 * t + 16 * sw);
            const bf16x8 hi = *reinterpret_cast<const bf16x8 *>(lds + 32 * t + 16 * (1 - sw));
            bf16x8 *dst = static_cast<bf16x8 *>(out) + ((int64_t)g.z * d.P + p) * 2;
            dst[0] = lo;
            dst[1] = hi;
        }
    }
}

// Lane-layout check of the 16x16x32 BF16 MFMA: D = A B for A [16][32],
// B [32][16], D [16][16] row-major FP32 (values exact in BF16).
__global__ void k_mfma16_probe(const float *__restrict__ A, const float *__restrict__ B, float *__restrict__ D) {
    const int l = threadIdx.x;
    bf16x8 a, b;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        a[j] = (__bf16)A[(l % 16) * 32 + 8 * (l / 16) + j];
        b[j] = (__bf16)B[(8 * (l / 16) + j) * 16 + l % 16];
    }
    const f32x4 c = mfma16(a, b, f32x4{});
#pragma unroll
    for (int i = 0; i < 4; ++i) D[(4 * (l / 16) + i) * 16 + l % 16] = c[i];
}

// Adam (Kingma & Ba) on n parameters, step t >= 1.
__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * kNT + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

}  // namespace

constexpr int kC[5] = {10, 16, 16, 16, 3};
constexpr int kMaxDilation = 64;

struct NetWork {
    int64_t cap_P = 0;
    int cap_B = 0;
    float *x = nullptr, *z[4] = {nullptr, nullptr, nullptr, nullptr};
    float *g[4] = {nullptr, nullptr, nullptr, nullptr};
    float *wt = nullptr;        // transposed weights of one layer
    double *part = nullptr;     // weight-gradient partials (FP64)
    size_t part_cap = 0;
    double *lpart = nullptr;
    size_t lpart_cap = 0;
    bf16x8 *frag = nullptr;     // BF16 MFMA weight fragments, [4 layers][14][64]
    bf16x8 *act[2] = {nullptr, nullptr};  // BF16 activations [B][P][16] (two 8-channel halves), ping-pong
    size_t act_cap = 0;                   // sites x images each holds
};

}  // namespace spx

using namespace spx;

struct spx_net {
    NetWork w;
    int dil[4] = {1, 1, 1, 1};  // per-layer dilation
    int prec = SPX_FP32;        // forward (inference) arithmetic: SPX_FP32 or SPX_BF16_MFMA
};

namespace {

int64_t net_nparams() {
    int64_t n = 0;
    for (int l = 0; l < 4; ++l) n += (int64_t)kC[l + 1] * kC[l] * 27 + kC[l + 1];
    return n;
}
int64_t layer_off(int l) {
    int64_t n = 0;
    for (int q = 0; q < l; ++q) n += (int64_t)kC[q + 1] * kC[q] * 27 + kC[q + 1];
    return n;
}

void net_free(NetWork &w) {
    for (void *p : {(void *)w.x, (void *)w.z[0], (void *)w.z[1], (void *)w.z[2], (void *)w.z[3], (void *)w.g[0],
                    (void *)w.g[1], (void *)w.g[2], (void *)w.g[3], (void *)w.wt, (void *)w.part, (void *)w.lpart,
                    (void *)w.frag, (void *)w.act[0], (void *)w.act[1]})
        if (p) (void)hipFree(p);
    w = NetWork{};
}

spx_status net_reserve(NetWork &w, int64_t P, int B, bool train) {
    if (P <= w.cap_P && B <= w.cap_B && (!train || w.g[0])) return SPX_OK;
    net_free(w);
    auto al = [](void **p, size_t bytes) {
        if (hipMalloc(p, bytes) != hipSuccess) {
            (void)hipGetLastError();
            *p = nullptr;
            return false;
        }
        return true;
    };
    bool ok = al((void **)&w.x, sizeof(float) * 10 * P * B);
    for (int l = 0; l < 4 && ok; ++l) ok = al((void **)&w.z[l], sizeof(float) * kC[l + 1] * P * B);
    for (int l = 0; l < 4 && ok && train; ++l) ok = al((void **)&w.g[l], sizeof(float) * kC[l + 1] * P * B);
    if (ok && train) ok = al((void **)&w.wt, sizeof(float) * 16 * 16 * 27);
    if (!ok) {
        net_free(w);
        return set_error(SPX_ERR_OUT_OF_MEMORY, "hipMalloc failed for network activations");
    }
    w.cap_P = P;
    w.cap_B = B;
    return SPX_OK;
}

// The dims of layer l: the lattice with that layer's dilation.
NetDims layer_dims(const NetDims &d, const int dil[4], int l) {
    NetDims e = d;
    e.dil = dil[l];
    e.Sx = (d.Lx + e.dil - 1) / e.dil;
    e.Sy = (d.Ly + e.dil - 1) / e.dil;
    e.Sz = (d.Lz + e.dil - 1) / e.dil;
    return e;
}

// Blocks of a layer: the tiles of one phase's sub-grid times the d^3 phases.
dim3 conv_grid(const NetDims &d, int B) {
    const int nbx = (d.Sx + kTXn - 1) / kTXn, nby = (d.Sy + kTYn - 1) / kTYn, nbz = (d.Sz + kTZn - 1) / kTZn;
    return dim3((unsigned)(nbx * nby * d.dil * d.dil), (unsigned)(nbz * d.dil), (unsigned)B);
}

// The box of a layer's FP32 kernels: the fewest tiles, then the smallest
// halo (what is staged per tile), then the longest rows.  Extents that split
// the sub-grid evenly are enough: a longer box with as many boxes per axis
// only pads.
NetBox conv_box(const NetDims &d, int B) {
    NetBox best{};
    for (int nx = (d.Sx + kBoxSites - 1) / kBoxSites, x = 0; x != 1; nx = x == 1 ? nx : (d.Sx + x - 2) / (x - 1)) {
        x = (d.Sx + nx - 1) / nx;
        const int ycap = kBoxSites / x;
        for (int ny = (d.Sy + ycap - 1) / ycap, y = 0; y != 1; ny = y == 1 ? ny : (d.Sy + y - 2) / (y - 1)) {
            y = (d.Sy + ny - 1) / ny;
            const int zcap = std::min(kBoxSites / (x * y), kBoxHalo / ((x + 2) * (y + 2)) - 2);
            if (zcap < 1) continue;
            NetBox b{};
            b.bx = x;
            b.by = y;
            b.nx = nx;
            b.ny = ny;
            b.nz = (d.Sz + zcap - 1) / zcap;
            b.bz = (d.Sz + b.nz - 1) / b.nz;
            b.hx = x + 2;
            b.hy = y + 2;
            b.halo = b.hx * b.hy * (b.bz + 2);
            b.vol = x * y * b.bz;
            b.tiles = (int64_t)b.nx * b.ny * b.nz;
            if (!best.vol || b.tiles < best.tiles || (b.tiles == best.tiles && b.halo < best.halo)) best = b;
        }
    }
    best.px = std::min(d.dil, d.Lx);
    best.py = std::min(d.dil, d.Ly);
    best.pz = std::min(d.dil, d.Lz);
    best.tiles *= (int64_t)best.px * best.py * best.pz * B;
    return best;
}

unsigned conv_blocks(const NetBox &b) { return (unsigned)std::min<int64_t>(b.tiles, kConvBlocks); }

// forward through the four layers as BF16 implicit GEMMs (inference), from
// the input states to the FP32 pre-activation u = z[3]
hipError_t net_forward_layers_mfma(NetWork &w, const float *params, const NetDims &d, const int dil[4], int B,
                                   const double *Sg, const double *SA, const double *SB, const float *t,
                                   int64_t ab_stride, hipStream_t st) {
    if (!w.frag) {
        hipError_t e = hipMalloc((void **)&w.frag, sizeof(bf16x8) * 4 * kTapPairs * 64);
        if (e != hipSuccess) return e;
    }
    const size_t need = (size_t)d.P * B;
    if (need > w.act_cap) {
        for (int k = 0; k < 2; ++k) {
            if (w.act[k]) (void)hipFree(w.act[k]);
            w.act[k] = nullptr;
        }
        w.act_cap = 0;
        for (int k = 0; k < 2; ++k) {
            hipError_t e = hipMalloc((void **)&w.act[k], sizeof(bf16x8) * 2 * need);
            if (e != hipSuccess) return e;
        }
        w.act_cap = need;
    }
    const int fb = (kTapPairs * 64 + 255) / 256;
    for (int l = 0; l < 4; ++l)
        k_wfrag<<<fb, 256, 0, st>>>(params + layer_off(l), kC[l], kC[l + 1], w.frag + l * kTapPairs * 64);
    const dim3 pg((unsigned)((d.P + kNT - 1) / kNT), (unsigned)B);
    k_net_input_bf16<<<pg, kNT, 0, st>>>(Sg, SA, SB, t, w.act[0], d.P, ab_stride);
    const NetDims d0 = layer_dims(d, dil, 0), d1 = layer_dims(d, dil, 1), d2 = layer_dims(d, dil, 2),
                  d3 = layer_dims(d, dil, 3);
    const float *b0 = params + layer_off(0) + 16 * 10 * 27, *b1 = params + layer_off(1) + 16 * 16 * 27;
    const float *b2 = params + layer_off(2) + 16 * 16 * 27, *b3 = params + layer_off(3) + 3 * 16 * 27;
    for (const NetDims *e : {&d0, &d1, &d2, &d3}) {
        const dim3 g = conv_grid(*e, B);
        if ((uint64_t)g.x * g.y * g.z >= ((uint64_t)1 << 31)) return hipErrorInvalidConfiguration;
    }
    bf16x8 *f = w.frag;
    k_conv_mfma<16, false><<<conv_grid(d0, B), kNT, 0, st>>>(w.act[0], f, b0, w.act[1], d0);
    k_conv_mfma<16, false><<<conv_grid(d1, B), kNT, 0, st>>>(w.act[1], f + kTapPairs * 64, b1, w.act[0], d1);
    k_conv_mfma<16, false><<<conv_grid(d2, B), kNT, 0, st>>>(w.act[0], f + 2 * kTapPairs * 64, b2, w.act[1], d2);
    k_conv_mfma<3, true><<<conv_grid(d3, B), kNT, 0, st>>>(w.act[1], f + 3 * kTapPairs * 64, b3, w.z[3], d3);
    return hipGetLastError();
}

// forward through the four layers; z[l] are pre-activations
hipError_t net_forward_layers(NetWork &w, const float *params, const NetDims &d, const int dil[4], int B,
                              hipStream_t st) {
    const NetDims d0 = layer_dims(d, dil, 0), d1 = layer_dims(d, dil, 1), d2 = layer_dims(d, dil, 2),
                  d3 = layer_dims(d, dil, 3);
    const float *W0 = params + layer_off(0), *W1 = params + layer_off(1);
    const float *W2 = params + layer_off(2), *W3 = params + layer_off(3);
    const NetBox b0 = conv_box(d0, B), b1 = conv_box(d1, B), b2 = conv_box(d2, B), b3 = conv_box(d3, B);
    k_conv<10, 16, false, false><<<conv_blocks(b0), kNT, 0, st>>>(w.x, W0, W0 + 16 * 10 * 27, nullptr, w.z[0], d0, b0);
    k_conv<16, 16, true, false><<<conv_blocks(b1), kNT, 0, st>>>(w.z[0], W1, W1 + 16 * 16 * 27, nullptr, w.z[1], d1, b1);
    k_conv<16, 16, true, false><<<conv_blocks(b2), kNT, 0, st>>>(w.z[1], W2, W2 + 16 * 16 * 27, nullptr, w.z[2], d2, b2);
    k_conv<16, 3, true, false><<<conv_blocks(b3), kNT, 0, st>>>(w.z[2], W3, W3 + 3 * 16 * 27, nullptr, w.z[3], d3, b3);
    return hipGetLastError();
}

spx_status check_dims(const int32_t *dims, int32_t batch, NetDims &d) {
    if (!dims || dims[0] < 1 || dims[1] < 1 || dims[2] < 1 || batch < 1)
        return set_error(SPX_ERR_INVALID_ARG, "bad network dims or batch");
    d.Lx = dims[0];
    d.Ly = dims[1];
    d.Lz = dims[2];
    d.P = (int64_t)dims[0] * dims[1] * dims[2];
    d.dil = 1;
    d.Sx = d.Lx;
    d.Sy = d.Ly;
    d.Sz = d.Lz;
    if (d.P * batch > ((int64_t)1 << 31)) return set_error(SPX_ERR_INVALID_ARG, "network batch too large");
    return SPX_OK;
}

}  // namespace

namespace spx {
// used by the GNEB learned initial path
spx_status net_apply(spx_net *net, const float *params, const int32_t dims[3], int32_t batch, const double *Sg,
                     const double *SA, const double *SB, int shared_ends, const float *t, double *Shat,
                     hipStream_t st) {
    NetDims d;
    spx_status s = check_dims(dims, batch, d);
    if (s != SPX_OK) return s;
    if ((s = net_reserve(net->w, d.P, batch, false)) != SPX_OK) return s;
    const dim3 pg((unsigned)((d.P + kNT - 1) / kNT), (unsigned)batch);
    const int64_t ab_stride = shared_ends ? 0 : 3 * d.P;
    hipError_t e;
    if (net->prec == SPX_BF16_MFMA) {
        e = net_forward_layers_mfma(net->w, params, d, net->dil, batch, Sg, SA, SB, t, ab_stride, st);
    } else {
        k_net_input<<<pg, kNT, 0, st>>>(Sg, SA, SB, t, net->w.x, d.P, ab_stride);
        e = net_forward_layers(net->w, params, d, net->dil, batch, st);
    }
    if (e == hipSuccess) {
        k_net_head<<<pg, kNT, 0, st>>>(net->w.z[3], Sg, nullptr, Shat, nullptr, nullptr, d.P, 0.0);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return set_hip_error(e, "network forward");
    return SPX_OK;
}
bool net_alive(spx_net *net) { return handle_alive(net); }
}  // namespace spx

extern "C" {

int64_t spx_net_nparams(void) { return net_nparams(); }

spx_status spx_net_create(const int32_t *channels, spx_net **out) {
    if (!out) return set_error(SPX_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (channels)
        for (int l = 0; l < 5; ++l)
            if (channels[l] != kC[l])
                return set_error(SPX_ERR_UNSUPPORTED, "only the 10-16-16-16-3 network is built");
    spx_net *n = new spx_net();
    register_handle(n);
    *out = n;
    return SPX_OK;
}

spx_status spx_net_set_dilation(spx_net *net, const int32_t *dil) {
    if (!handle_alive(net)) return set_error(SPX_ERR_BAD_HANDLE, "invalid spx_net handle");
    if (!dil) return set_error(SPX_ERR_INVALID_ARG, "dil is NULL");
    for (int l = 0; l < 4; ++l)
        if (dil[l] < 1 || dil[l] > kMaxDilation)
            return set_error(SPX_ERR_INVALID_ARG, "each dilation must be 1 .. 64");
    for (int l = 0; l < 4; ++l) net->dil[l] = dil[l];
    return SPX_OK;
}

spx_status spx_net_set_precision(spx_net *net, int32_t prec) {
    if (!handle_alive(net)) return set_error(SPX_ERR_BAD_HANDLE, "invalid spx_net handle");
    if (prec != SPX_FP32 && prec != SPX_BF16_MFMA)
        return set_error(SPX_ERR_INVALID_ARG, "the network runs in SPX_FP32 or SPX_BF16_MFMA");
    net->prec = prec;
    return SPX_OK;
}

spx_status spx_mfma16_probe(const float *A, const float *B, float *D, void *stream) {
    if (!A || !B || !D) return set_error(SPX_ERR_INVALID_ARG, "NULL argument");
    k_mfma16_probe<<<1, 64, 0, (hipStream_t)stream>>>(A, B, D);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_hip_error(e, "spx_mfma16_probe");
    return SPX_OK;
}

spx_status spx_net_destroy(spx_net *net) {
    if (!handle_alive(net)) return set_error(SPX_ERR_BAD_HANDLE, "invalid spx_net handle");
    unregister_handle(net);
    (void)hipDeviceSynchronize();
    net_free(net->w);
    delete net;
    return SPX_OK;
}

spx_status spx_net_forward(spx_net *net, const float *params, const int32_t *dims, int32_t batch, const double *Sg,
                           const double *SA, const double *SB, const float *t, double *Shat, void *stream) {
    if (!handle_alive(net)) return set_error(SPX_ERR_BAD_HANDLE, "invalid spx_net handle");
    if (!params || !Sg || !SA || !SB || !t || !Shat) return set_error(SPX_ERR_INVALID_ARG, "NULL argument");
    return net_apply(net, params, dims, batch, Sg, SA, SB, 0, t, Shat, (hipStream_t)stream);
}

spx_status spx_net_backward(spx_net *net, const float *params, const int32_t *dims, int32_t batch, const double *Sg,
                            const double *SA, const double *SB, const float *t, const double *Sstar, float *grad,
                            double *loss, void *stream) {
    if (!handle_alive(net)) return set_error(SPX_ERR_BAD_HANDLE, "invalid spx_net handle");
    if (!params || !Sg || !SA || !SB || !t || !Sstar || !grad) return set_error(SPX_ERR_INVALID_ARG, "NULL argument");
    hipStream_t st = (hipStream_t)stream;
    NetDims d;
    spx_status s = check_dims(dims, batch, d);
    if (s != SPX_OK) return s;
    NetWork &w = net->w;
    if ((s = net_reserve(w, d.P, batch, true)) != SPX_OK) return s;
    NetDims dl[4];
    NetBox box[4];
    size_t need = 0;  // doubles of the weight-gradient partials
    for (int l = 0; l < 4; ++l) {
        dl[l] = layer_dims(d, net->dil, l);
        box[l] = conv_box(dl[l], batch);
        need = std::max(need, (size_t)conv_blocks(box[l]) * (l == 3 ? 2 : 1) * (kC[l + 1] * kC[l] * 27 + kC[l + 1]));
    }
    const dim3 pg((unsigned)((d.P + kNT - 1) / kNT), (unsigned)batch);
    const size_t nl = (size_t)pg.x * pg.y;
    if (need > w.part_cap) {
        if (w.part) (void)hipFree(w.part);
        if (hipMalloc((void **)&w.part, need * sizeof(double)) != hipSuccess) {
            (void)hipGetLastError();
            w.part = nullptr;
            w.part_cap = 0;
            return set_error(SPX_ERR_OUT_OF_MEMORY, "hipMalloc failed for gradient partials");
        }
        w.part_cap = need;
    }
    if (nl > w.lpart_cap) {
        if (w.lpart) (void)hipFree(w.lpart);
        if (hipMalloc((void **)&w.lpart, nl * sizeof(double)) != hipSuccess) {
            (void)hipGetLastError();
            w.lpart = nullptr;
            w.lpart_cap = 0;
            return set_error(SPX_ERR_OUT_OF_MEMORY, "hipMalloc failed for loss partials");
        }
        w.lpart_cap = nl;
    }
    k_net_input<<<pg, kNT, 0, st>>>(Sg, SA, SB, t, w.x, d.P, 3 * d.P);
    hipError_t e = net_forward_layers(w, params, d, net->dil, batch, st);
    if (e != hipSuccess) return set_hip_error(e, "network backward (forward pass)");
    const double inv_count = 1.0 / ((double)d.P * batch);
    k_net_head<<<pg, kNT, 0, st>>>(w.z[3], Sg, Sstar, nullptr, w.g[3], w.lpart, d.P, inv_count);
    if (loss) k_loss_final<<<1, kNT, 0, st>>>(w.lpart, (int)nl, inv_count, loss);
    // layer 4 (16 -> 3), 3 (16 -> 16), 2 (16 -> 16), 1 (10 -> 16)
    for (int l = 3; l >= 0; --l) {
        const int cin = kC[l], cout = kC[l + 1];
        const int nw = cout * cin * 27 + cout;
        const float *Wl = params + layer_off(l);
        float *gl = grad + layer_off(l);
        const float *ain = l == 0 ? w.x : w.z[l - 1];
        const NetDims &d_l = dl[l];
        const NetBox &b_l = box[l];
        const unsigned gr = conv_blocks(b_l);
        if (l == 3) k_conv_wgrad<3, true, true, 2><<<gr, kNT, 0, st>>>(ain, w.g[3], w.part, d_l, b_l);
        else if (l == 0) k_conv_wgrad<10, false, false, 1><<<gr, kNT, 0, st>>>(ain, w.g[0], w.part, d_l, b_l);
        else k_conv_wgrad<16, false, true, 1><<<gr, kNT, 0, st>>>(ain, w.g[l], w.part, d_l, b_l);
        k_sum_partials<<<(nw + kSumW - 1) / kSumW, kNT, 0, st>>>(w.part, (int)gr * (l == 3 ? 2 : 1), nw, gl);
        if (l > 0) {
            // g_{l-1} = silu'(z_{l-1}) * conv(g_l, W^T flipped)
            k_transpose_flip<<<(cin * cout * 27 + 255) / 256, 256, 0, st>>>(Wl, w.wt, cin, cout);
            // the transposed convolution of layer l has layer l's dilation
            if (l == 3) k_conv<3, 16, false, true><<<gr, kNT, 0, st>>>(w.g[3], w.wt, nullptr, w.z[2], w.g[2], d_l, b_l);
            else k_conv<16, 16, false, true><<<gr, kNT, 0, st>>>(w.g[l], w.wt, nullptr, w.z[l - 1], w.g[l - 1], d_l, b_l);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return set_hip_error(e, "network backward");
    }
    return SPX_OK;
}

spx_status spx_net_adam_step(float *params, const float *grad, float *m, float *v, int64_t n, int64_t step,
                             double lr, double b1, double b2, double eps, void *stream) {
    if (!params || !grad || !m || !v || n < 0 || step < 1) return set_error(SPX_ERR_INVALID_ARG, "bad Adam arguments");
    const float c1 = (float)(1.0 - std::pow(b1, (double)step)), c2 = (float)(1.0 - std::pow(b2, (double)step));
    k_adam<<<(unsigned)((n + kNT - 1) / kNT), kNT, 0, (hipStream_t)stream>>>(params, grad, m, v, n, (float)lr,
                                                                            (float)b1, (float)b2, (float)eps, c1, c2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return set_hip_error(e, "spx_net_adam_step");
    return SPX_OK;
}

}  // extern "C"
